"""Code-generation guard for the loop bodies (CPU only): every instantiation
has the grid barrier and its sweeps inline.  Called out of line, each of them
saves most of the body's registers to memory and costs a sweep of a few
microseconds another one to four."""
import re

from test_codegen_cpu import asm, callees, function_body  # noqa: F401

LOOPS = r"^(_ZN12_GLOBAL__N_1\d+(?:map_loop_kernelI|map_body_gang_|map_body_async)[\w.$]*):"


def test_loop_bodies_inline_barriers_and_sweeps(asm):  # noqa: F811
    names = re.findall(LOOPS, asm, re.M)
    assert sum("map_loop_kernel" in x for x in names) >= 4 and sum("map_body_gang_filt" in x for x in names) == 1, names
    called = {x: [c for c in callees(function_body(asm, x)) if re.search("grid_sync|sweep_", c)] for x in names}
    assert not any(called.values()), called
