"""Top-C selection of the fused path at the sizes where its launches change:
one tile, partial tiles, the 64 tiles up to which nothing is pruned, and more;
one candidate, few, and the most a recursion keeps.

Entries are integers (or all equal, or all zero: every bin a tie), so every
bin is exact and the fused records must equal those of the stored-bins path,
which selects by a scan of the bins, field by field."""
import numpy as np
import pytest

from oracle import dd
from workloads import synthetic as syn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def entries(kind, bonds, ns):
    rng = np.random.default_rng(sum(ns))
    ks = syn.chain_ks(bonds, len(ns))
    if kind == "integer":
        return [syn.integer_entries(rng, k, n, lo=-2, hi=3) for k, n in zip(ks, ns)]
    if kind == "few":  # a handful of nonzero bins
        return [(rng.random((4 ** k, 2 ** n)) < 0.02).astype(np.float64) for k, n in zip(ks, ns)]
    return [np.full((4 ** k, 2 ** n), 1.0 if kind == "equal" else 0.0) for k, n in zip(ks, ns)]


# active outputs per subcircuit: 2^2 bins, 2^13 (one tile, partial), 2^20 (64
# tiles) and 2^21 (128)
@pytest.mark.parametrize("bonds,ns,M", [([1], [3, 4], [1, 1]), ([1, 1], [6, 6, 6], [4, 4, 5]),
                                        ([2], [11, 11], [10, 10]), ([1, 1], [8, 8, 8], [7, 7, 7])])
@pytest.mark.parametrize("kind", ["integer", "few", "equal", "zero"])
@pytest.mark.parametrize("R", [1, 3, 16])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16_split"])
def test_fused_selection_equals_stored(bonds, ns, M, kind, R, prec):
    import paper_2205_05836_amd as m
    cm, E = syn.chain_cutmap(bonds, ns), entries(kind, bonds, ns)
    st = dd.initial_states(cm, M)
    inst = dict(subs=cm, entries=[torch.from_numpy(np.ascontiguousarray(e)).to(DEV) for e in E],
                active=[sum(1 << int(i) for i in s.active) for s in st],
                merged=[sum(1 << int(i) for i in s.merged) for s in st],
                fixed=[0] * len(ns), fixed_vals=[0] * len(ns), max_active=M)
    dt = torch.float64 if prec == "fp64" else torch.float32
    bins = [torch.empty(2 ** sum(M), dtype=dt, device=DEV) for _ in range(R)]
    stored, done_s = m.cq_reconstruct_dd([inst], prec, R, bins=bins)
    fused, done_f = m.cq_reconstruct_dd([inst], prec, R)
    assert done_s == done_f
    for a, b in zip(fused[0], stored[0]):
        for key in b:
            if key not in ("tiles", "tiles_run"):
                assert a[key] == b[key], (key, a["recursion"])
        if a["tiles"] <= 64:
            assert a["tiles_run"] == a["tiles"]
