"""The largest sizes the limits admit stay within what a launch may ask for:
fewer than 2^32 threads in a dimension (host only, launches are recorded
instead of run, so nothing of these sizes is allocated)."""
import json

import pytest

import launch_recorder
from workloads import synthetic as syn


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return launch_recorder.build(tmp_path_factory.mktemp("recorder"))


FD = """
def fd(cm, perm, prec):
    s = api._Subs(cm)
    events()
    st = L.cq_reconstruct_fd(len(cm), s.ptr(), (C.c_void_p * len(cm))(*[(i + 1) << 40 for i in range(len(cm))]),
                             _lib.PRECISION[prec], (C.c_int32 * len(perm))(*perm), C.c_void_p(1 << 50),
                             C.c_void_p(1 << 51), 1 << 45, None)
    return [st, events()]
out = [fd(cm, perm, prec) for cm, perm, prec in json.loads(CASES)]
"""


@pytest.mark.parametrize("outs", [[16, 16], [16, 17], [17, 17], [17, 18], [18, 18]])
def test_permuted_full_definition(recorder, outs):
    n = sum(outs)
    cases = [(syn.chain_cutmap([1], outs), list(range(n))[::-1], prec)
             for prec in ("fp64", "fp32", "bf16", "bf16_split", "fp16_split")]
    for (_, _, prec), (status, ev) in zip(cases, launch_recorder.run(recorder, f"CASES = {json.dumps(cases)!r}\n" + FD)):
        assert any("permute" in e["kernel"] for e in ev)
        assert [e for e in ev if not e["ok"]] == [], prec
        assert status == 0, prec
