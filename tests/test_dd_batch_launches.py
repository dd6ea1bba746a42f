"""A batch of dynamic-definition instances that advance together: what the
host launches for all of them fits what every member's device program says.
Members share a step sequence but not their sizes (host only, launches are
recorded instead of run)."""
import json

import pytest

import launch_recorder
from workloads import synthetic as syn

# active outputs of two subcircuits with two cuts between them: 2^13, 2^20
# (64 output tiles, up to which nothing is pruned) and 2^21 bins (128 tiles)
SIZES = {"one tile": ([7, 7], [6, 7]), "64 tiles": ([11, 11], [10, 10]), "128 tiles": ([11, 12], [10, 11])}

SCRIPT = """
import itertools
def batch(shapes, prec, R):
    subs = [api._Subs(cm) for cm, _ in shapes]
    arr = (_lib.cq_dd_instance * len(shapes))()
    keep, base = [], 1 << 40
    for a, s, (cm, M) in zip(arr, subs, shapes):
        n = len(cm)
        act = [(1 << m) - 1 for m in M]
        mer = [((1 << o) - 1) & ~x for o, x in zip(s.n_out, act)]
        u64 = C.c_uint64 * n
        f = [(C.c_void_p * n)(*[base + (i << 36) for i in range(n)]), u64(*act), u64(*mer), u64(), u64(),
             (C.c_int32 * n)(*M)]
        keep += f
        a.n_sub, a.subs = n, s.ptr()
        a.entries, a.active, a.merged, a.fixed, a.fixed_vals, a.max_active = f
        base += 1 << 39
    par = _lib.cq_dd_params(_lib.PRECISION[prec], R, _lib.DD_LAUNCH["direct"], 1, None, None)
    need = C.c_size_t()
    assert L.cq_dd_workspace_size(len(shapes), arr, C.byref(par), 0, C.byref(need)) == 0
    recs = (_lib.cq_dd_record * (len(shapes) * R))()
    done = (C.c_int32 * len(shapes))()
    events()
    st = L.cq_reconstruct_dd(len(shapes), arr, C.byref(par), recs, None, done, C.c_void_p(1 << 50), need, None)
    assert st == 0, L.cq_last_error()
    return events()
out = [batch(shapes, prec, R) for shapes, prec, R in json.loads(CASES)]
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return launch_recorder.build(tmp_path_factory.mktemp("recorder"))


def record(recorder, cases):
    return launch_recorder.run(recorder, f"CASES = {json.dumps(cases)!r}\n" + SCRIPT)


def shape(name):
    ns, M = SIZES[name]
    return syn.chain_cutmap([2], ns), M


def kernels(events):
    return [e["kernel"] for e in events if "kernel" in e]


def programs(events):
    return next(e["programs"] for e in events if "programs" in e)


ORDERS = [["one tile"], ["64 tiles"], ["128 tiles"], ["one tile", "128 tiles"], ["128 tiles", "one tile"],
          ["64 tiles", "128 tiles", "one tile"], ["one tile", "64 tiles"]]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16_split"])
def test_members_are_pruned_together(recorder, prec):
    """Tiles are pruned for all members or for none, as the largest asks for,
    and the launches that pruning needs are there exactly then."""
    for names, ev in zip(ORDERS, record(recorder, [([shape(n) for n in names], prec, 4) for names in ORDERS])):
        prune = [p["prune"] for p in programs(ev)]
        assert prune == [int("128 tiles" in names)] * len(names), names
        for part in ("tile_bound_kernel", "tile_warm_kernel", "warm_tau_kernel", "tile_compact_kernel"):
            assert any(part in k for k in kernels(ev)) == bool(prune[0]), (names, part)


def test_selection_is_staged_for_the_largest_candidate_list(recorder):
    """One workgroup selects from at most 4096 candidates; a member that can
    hold more (128 tiles of 64 keys) has them staged, whatever its place."""
    for names, ev in zip(ORDERS, record(recorder, [([shape(n) for n in names], "fp32", 16) for names in ORDERS])):
        staged = any("topk_kernel" in k for k in kernels(ev))
        assert staged == ("128 tiles" in names), names


def uncut(ns, M):
    return syn.chain_cutmap([0], ns), M


@pytest.mark.parametrize("prec", ["bf16", "bf16_split", "fp16", "fp16_split"])
def test_members_take_the_same_preparation(recorder, prec):
    """Label balance needs a cut and column scaling an output axis a
    subcircuit: members launched together agree on both, and one that is
    balanced finds its balance launched, whichever comes first."""
    cut, bare = shape("one tile"), uncut([7, 7], [6, 7])
    for ev in record(recorder, [([bare, cut], prec, 4), ([cut, bare], prec, 4), ([bare], prec, 4), ([cut], prec, 4)]):
        progs = programs(ev)
        for flag, part in (("balance", "balance_ind_kernel"), ("cscale", "colmax_ind_kernel")):
            launches = sum(part in k for k in kernels(ev))
            groups = sum("dd_init_kernel" in k for k in kernels(ev))
            sets = {p[flag] for p in progs}
            assert launches == (groups if sets == {1} else 0 if sets == {0} else 1), (flag, progs)
            assert len(sets) <= groups
