"""Instances of different sizes that advance together take the records that
each takes alone, in either order of the batch.

Entries are integers, or all equal, or all zero (every bin a tie), so bins are
exact and the records must agree field by field.  Whether a small member's
tiles are pruned follows the largest member, so tiles_run is left out."""
import numpy as np
import pytest

from oracle import dd
from workloads import synthetic as syn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# one output tile, 64 tiles (the most that run unpruned alone) and 128
SIZES = [([7, 7], [6, 7]), ([11, 11], [10, 10]), ([11, 12], [10, 11])]


def entries(kind, ns):
    rng = np.random.default_rng(sum(ns))
    ks = syn.chain_ks([2], 2)
    if kind == "integer":
        return [syn.integer_entries(rng, k, n, lo=-2, hi=3) for k, n in zip(ks, ns)]
    return [np.full((4 ** k, 2 ** n), 1.0 if kind == "equal" else 0.0) for k, n in zip(ks, ns)]


def instance(kind, ns, M):
    st = dd.initial_states(syn.chain_cutmap([2], ns), M)
    return dict(subs=syn.chain_cutmap([2], ns),
                entries=[torch.from_numpy(np.ascontiguousarray(e)).to(DEV) for e in entries(kind, ns)],
                active=[sum(1 << int(i) for i in s.active) for s in st],
                merged=[sum(1 << int(i) for i in s.merged) for s in st],
                fixed=[0] * len(ns), fixed_vals=[0] * len(ns), max_active=M)


def fields(rec):
    return {k: v for k, v in rec.items() if k != "tiles_run"}


def check(kind, R, prec, launch, order):
    import paper_2205_05836_amd as m
    print(f"mixed batch {kind} R={R} {prec} {launch} {order}", flush=True)
    insts = [instance(kind, *SIZES[q]) for q in order]
    alone = [m.cq_reconstruct_dd([x], prec, R, launch=launch) for x in insts]
    recs, done = m.cq_reconstruct_dd(insts, prec, R, launch=launch)
    assert done == [d[0] for _, d in alone]
    for got, (want, _) in zip(recs, alone):
        assert [fields(r) for r in got] == [fields(r) for r in want[0]]


@pytest.mark.parametrize("order", [(0, 2), (2, 0), (1, 2, 0), (0, 1)])
@pytest.mark.parametrize("launch", ["graph", "direct"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16_split", "fp16"])
def test_records_follow_no_other_member(prec, launch, order):
    check("integer", 4, prec, launch, order)


@pytest.mark.parametrize("order", [(0, 2), (2, 0), (1, 2, 0)])
@pytest.mark.parametrize("kind", ["integer", "equal", "zero"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16_split"])
def test_most_candidates(prec, kind, order):
    """With ties everywhere the largest member holds 8192 candidates."""
    check(kind, 16, prec, "graph", order)


@pytest.mark.parametrize("prec", ["bf16", "fp16", "fp16_split"])
@pytest.mark.parametrize("cut_first", [False, True])
def test_with_and_without_cuts(prec, cut_first):
    """An instance without cuts is not balanced; one with cuts is, whichever
    comes first.  The workspace starts as bytes of ones, so an exponent that
    no launch has written would show."""
    import paper_2205_05836_amd as m
    print(f"mixed batch {prec} cut_first={cut_first}", flush=True)
    rng = np.random.default_rng(3)
    insts = []
    for bonds in ([0], [2]):
        cm, ks = syn.chain_cutmap(bonds, [6, 7]), syn.chain_ks(bonds, 2)
        st = dd.initial_states(cm, [4, 4])
        insts.append(dict(subs=cm, entries=[torch.from_numpy(syn.integer_entries(rng, k, n, lo=-2, hi=3)).to(DEV)
                                            for k, n in zip(ks, [6, 7])],
                          active=[sum(1 << int(i) for i in s.active) for s in st],
                          merged=[sum(1 << int(i) for i in s.merged) for s in st],
                          fixed=[0, 0], fixed_vals=[0, 0], max_active=[4, 4]))
    if cut_first:
        insts.reverse()
    alone = [m.cq_reconstruct_dd([x], prec, 3)[0][0] for x in insts]
    ws = torch.full((m.cq_dd_workspace_size(insts, prec, 3),), 255, dtype=torch.uint8, device=DEV)
    recs, _ = m.cq_reconstruct_dd(insts, prec, 3, workspace=ws)
    assert [[fields(r) for r in rec] for rec in recs] == [[fields(r) for r in rec] for rec in alone]


@pytest.mark.parametrize("order", [(0, 2), (2, 0)])
@pytest.mark.parametrize("launch", ["graph", "direct"])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16_split"])
def test_resumed_at_different_recursions(prec, launch, order):
    """Members resume at recursions of their own; those at their end are
    launched along with the others, on a workspace of bytes of ones, and run
    nothing."""
    import paper_2205_05836_amd as m
    print(f"resume {prec} {launch} {order}", flush=True)
    R, insts = 5, [instance("integer", *SIZES[q]) for q in order]
    full = [m.cq_reconstruct_dd([x], prec, R, launch=launch) for x in insts]
    for cut in ((5, 1), (1, 5), (4, 1), (1, 4)):
        cks = [m.cq_reconstruct_dd([x], prec, R, launch=launch, recursions=c, checkpoint=True)[2]
               for x, c in zip(insts, cut)]
        ws = torch.full((m.cq_dd_workspace_size(insts, prec, R),), 255, dtype=torch.uint8, device=DEV)
        recs, done = m.cq_reconstruct_dd(insts, prec, R, launch=launch, resume=b"".join(cks), workspace=ws)
        for got, n, (want, total), c in zip(recs, done, full, cut):
            assert n == max(total[0] - c, 0)
            assert [fields(r) for r in got] == [fields(r) for r in want[0][c:]]
