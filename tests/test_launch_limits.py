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


@pytest.mark.parametrize("outs", [[18, 18], [12, 12, 12], [7, 29], [3, 30]])
def test_tuned_full_definition(recorder, outs):
    """The autotuner tries only variants whose launch is possible."""
    n = sum(outs)
    cases = [(syn.chain_cutmap([1] * (len(outs) - 1), outs), list(range(n)), prec)
             for prec in ("fp32", "bf16", "bf16_split", "fp16_split")]
    script = f"L.cq_autotune_enable(1)\nCASES = {json.dumps(cases)!r}\n" + FD
    for (_, _, prec), (status, ev) in zip(cases, launch_recorder.run(recorder, script)):
        assert [e for e in ev if not e["ok"]] == [], prec
        assert status == 0, prec


VARIANTS = """
def variants(sub, states):
    s = api._Subs([sub])
    gates, n = api._gates([("u", q, [[0.6, 0.8], [0.8, -0.6]]) for q in range(sub[0])])
    events()
    st = L.cq_variant_probabilities(s.ptr(), gates, n, C.c_void_p(1 << 50), C.c_void_p(1 << 51), states << (sub[0] + 4),
                                    None)
    return [st, events()]
def simulate(n):
    gates, cnt = api._gates([("u", q, [[0.6, 0.8], [0.8, -0.6]]) for q in range(n)])
    events()
    st = L.cq_simulate_probabilities(n, gates, cnt, C.c_void_p(1 << 50), C.c_void_p(1 << 51), 1 << (n + 4), None)
    return [st, events()]
out = [variants(*c) for c in json.loads(CASES)] + [simulate(n) for n in range(32, 35)]
"""


def test_widest_registers(recorder):
    """32 slots with and without cut ends, one state of workspace and enough;
    34 qubits."""
    cases = []
    for w in (31, 32):
        for r, o in ((0, 0), (1, 0), (0, 1), (2, 2), (0, 8), (8, 0), (5, 3)):
            init = [c for c in range(r)] + [-1] * (w - r)
            meas = [-1] * (w - o) + [r + c for c in range(o)]
            cases += [((w, init, meas), 1), ((w, init, meas), 1 << r)]
    for c, (status, ev) in zip(cases + [(n, 1) for n in range(32, 35)],
                               launch_recorder.run(recorder, f"CASES = {json.dumps(cases)!r}\n" + VARIANTS)):
        assert ev and [e for e in ev if not e["ok"]] == [], c
        assert status == 0, c


STATES = """
def launches(sub, states):
    s = api._Subs([sub])
    gates, n = api._gates([("u", q, [[0.6, 0.8], [0.8, -0.6]]) for q in range(sub[0])] +
                          [("cz", q, q + 1) for q in range(sub[0] - 1)])
    events()
    assert L.cq_variant_probabilities(s.ptr(), gates, n, C.c_void_p(1 << 50), C.c_void_p(1 << 51),
                                      states << (sub[0] + 4), None) == 0
    return len(events())
def query(sub):
    s, b = api._Subs([sub]), C.c_size_t()
    assert L.cq_variants_workspace_size(s.ptr(), C.byref(b)) == 0
    return b.value
out = [[launches(sub, n) for n in states] + [query(sub)] for sub, states in json.loads(CASES)]
"""


def slots(w, r, o):
    return w, list(range(r)) + [-1] * (w - r), [-1] * (w - o) + list(range(r, r + o))


@pytest.mark.parametrize("w,r,o", [(6, 2, 1), (12, 1, 2), (12, 3, 2), (13, 2, 4), (14, 4, 0)])
def test_variants_use_what_the_workspace_holds(recorder, w, r, o):
    """2^s states of workspace take 4^(r - s) batches, each with the launches
    of a full one: its passes and one that writes every basis."""
    states = list(range(1, 2 ** r + 1))
    cases = [(slots(w, r, o), states)]
    *got, _ = launch_recorder.run(recorder, f"CASES = {json.dumps(cases)!r}\n" + STATES)[0]
    for n, launches in zip(states, got):
        assert launches <= 4 ** (r - (n.bit_length() - 1)) * (got[-1] + 1), n  # a prepared slot may cost a pass


def test_variants_workspace_leaves_room_for_the_variants(recorder):
    """The query asks for every computational init string, but not past 240 GiB
    with the variants: what fitted the card with one state still does."""
    cases = [(slots(w, r, o), []) for w, r, o in ((12, 3, 2), (22, 2, 2), (27, 4, 0), (29, 3, 0), (31, 1, 1), (32, 0, 0))]
    got = [q[0] for q in launch_recorder.run(recorder, f"CASES = {json.dumps(cases)!r}\n" + STATES)]
    assert got == [16 << 15, 16 << 24, 16 << 27, 16 << 29, 16 << 31, 16 << 32]


SHOTS = """
def kernels(rows, cols, shots):
    b = C.c_size_t()
    assert L.cq_sample_shots_workspace_size(rows, cols, shots, C.byref(b)) == 0
    events()
    assert L.cq_sample_shots(C.c_void_p(1 << 50), rows, cols, shots, 1, C.c_void_p(1 << 51), C.c_void_p(1 << 52), b, None) == 0
    return [e["kernel"] for e in events()]
out = [kernels(*c) for c in json.loads(CASES)]
"""


def test_small_tables_resolve_by_workgroups(recorder):
    """A wave a block only where the blocks fill the chip."""
    cases = [(52, 16320, 119), (255, 16320, 119), (256, 16320, 119), (144, 1 << 22, 8192), (144, 1 << 22, 1 << 16)]
    got = launch_recorder.run(recorder, f"CASES = {json.dumps(cases)!r}\n" + SHOTS)
    assert [any("resolve_sparse" in k for k in ks) for ks in got] == [False, False, True, True, False]


SMALL_SHOTS = """
def kernels(rows, cols, shots):
    up = lambda n: (n + 255) // 256 * 256
    blocks = rows * -(-cols // 2048)
    need = up(8 * blocks) + 3 * up(4 * blocks) + up(8 * rows * shots)
    b = C.c_size_t()
    assert L.cq_sample_shots_workspace_size(rows, cols, shots, C.byref(b)) == 0
    call = lambda n: L.cq_sample_shots(C.c_void_p(1 << 50), rows, cols, shots, 1, C.c_void_p(1 << 51),
                                       C.c_void_p(1 << 52), n, None)
    codes, sparse = [], []
    for n in (need - 1, need, b.value - 1, b.value):
        events()
        codes.append(call(n))
        sparse.append(any("resolve_sparse" in e["kernel"] for e in events()))
    return [b.value - need, codes, sparse]
out = [kernels(*c) for c in json.loads(CASES)]
"""


def test_shots_without_room_for_run_sums(recorder):
    """The run sums (256 bytes a block) are asked for where blocks resolve a wave
    each, up to 240 GiB with the tables; a workspace without room for them is
    taken as ever."""
    cases = [(144, 1 << 22, 8192), (2, 8, 100), (52, 16320, 119), (144, 1 << 22, 1 << 16), (64, 1 << 28, 8192)]
    got = launch_recorder.run(recorder, f"CASES = {json.dumps(cases)!r}\n" + SMALL_SHOTS)
    refused, plain = [-5, 0, -5, 0], [0, 0, 0, 0]
    assert got[0] == [144 * 2048 * 256, [-5] + plain[1:], [False, False, False, True]]
    assert got[1:] == [[0, refused, [False] * 4]] * 4
