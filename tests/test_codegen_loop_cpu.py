"""Code-generation guard for the loop bodies (CPU only): every instantiation
that runs a barrier per sweep has the grid barrier inline.  Called out of line,
each barrier saved most of the body's registers to memory and cost a sweep of a
few microseconds another one or two."""
import re

from test_codegen_cpu import asm, callees, function_body  # noqa: F401

LOOPS = r"^(_ZN12_GLOBAL__N_1\d+(?:map_loop_kernelI|map_body_gang_|map_body_async)[\w.$]*):"


def test_loop_bodies_inline_the_grid_barrier(asm):  # noqa: F811
    names = re.findall(LOOPS, asm, re.M)
    assert sum("map_loop_kernel" in x for x in names) >= 4 and sum("map_body_gang_filt" in x for x in names) == 1, names
    called = {x: [c for c in callees(function_body(asm, x)) if "grid_sync" in c] for x in names}
    assert not any(called.values()), called
