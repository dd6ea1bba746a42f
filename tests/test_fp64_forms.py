"""Which FP64 kernel a product of two subcircuits takes (host only: launches are
recorded instead of run)."""
import json

import pytest

import launch_recorder
from workloads import synthetic as syn


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return launch_recorder.build(tmp_path_factory.mktemp("recorder"))


# cuts, outputs of each side (the longer one makes the rows), 128 x 128 tiles:
# 256 to 1024 columns and 2^27 outputs up with fewer than 8 labels, and a step
# beyond each of these
CASES = [(1, [19, 8], True), (0, [19, 8], True), (1, [17, 10], True), (1, [21, 9], True), (1, [20, 7], False),
         (1, [16, 11], False), (1, [18, 8], False), (2, [19, 8], False), (1, [8, 19], False), (1, [9, 18], False)]


@pytest.mark.parametrize("cuts,outs,tiled", CASES)
def test_tiles_of_short_products(recorder, cuts, outs, tiled):
    script = f"CASE = json.loads({json.dumps(syn.chain_cutmap([cuts], outs))!r})" + """
s = api._Subs(CASE)
assert L.cq_reconstruct_fd(len(CASE), s.ptr(), (C.c_void_p * len(CASE))(*[(i + 1) << 40 for i in range(len(CASE))]),
                           _lib.PRECISION["fp64"], None, C.c_void_p(1 << 50), C.c_void_p(1 << 51), 1 << 45, None) == 0
out = [[e["kernel"], e["ok"]] for e in events() if "gemm_" in e["kernel"]]
"""
    (kernel, ok), = launch_recorder.run(recorder, script)
    assert ok and ("gemm_f64_kernel" if tiled else "gemm_f64t_kernel") in kernel, kernel
