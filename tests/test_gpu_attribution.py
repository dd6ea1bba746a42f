"""Attribution with three or four cut ends on a side against the FP64 oracle.

Variants are integers of magnitude at most 8, so every sum (at most 16 outcome
values, then 16 combinations of them with weights of magnitude at most 16 per
digit) is an integer far below 2^53 and the device must match the oracle
exactly, whatever the order of the additions."""
import numpy as np
import pytest

from oracle import attribution as at

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def make_sub(r, o, n, where, rng):
    """Measured slots last, first, or at random places; init slots among the rest."""
    w = n + o
    ms = {"last": list(range(n, w)), "first": list(range(o)),
          "mixed": sorted(rng.choice(w, size=o, replace=False).tolist())}[where]
    cuts = list(rng.permutation(r + o))
    init, meas = [-1] * w, [-1] * w
    for s in ms:
        meas[s] = int(cuts.pop())
    for s in sorted(rng.choice(w, size=r, replace=False).tolist()):
        init[s] = int(cuts.pop())
    # a slot may be initialised and measured, by different cuts
    return w, init, meas


@pytest.mark.parametrize("r,o,n,where", [
    (0, 3, 6, "last"), (0, 3, 5, "mixed"), (1, 3, 7, "mixed"), (2, 3, 8, "first"), (2, 3, 6, "last"),
    (0, 4, 7, "last"), (0, 4, 6, "mixed"), (1, 4, 6, "first"), (1, 4, 1, "last"), (3, 3, 2, "mixed"),
    (4, 0, 5, "last"), (4, 0, 4, "last"), (4, 1, 6, "mixed"), (4, 1, 3, "first"), (4, 2, 4, "mixed")])
@pytest.mark.parametrize("offset", [0, 1])
def test_three_and_four_cut_ends_exact(r, o, n, where, offset):
    """``offset`` 1: the variants start 8 bytes past a 16-byte boundary."""
    import paper_2205_05836_amd as cq
    rng = np.random.default_rng(1000 * r + 100 * o + n)
    sub = make_sub(r, o, n, where, rng)
    V = rng.integers(-8, 9, size=(4 ** r, 3 ** o, 2 ** sub[0])).astype(np.float64)
    buf = torch.empty(V.size + offset, dtype=torch.float64, device=DEV)
    dev = buf[offset:].view(V.shape)
    dev.copy_(torch.from_numpy(V))
    got = cq.cq_attribute(sub, dev).cpu().numpy()
    assert np.array_equal(got, at.attribute(sub, V))


@pytest.mark.parametrize("r,o,n,cols", [(4, 3, 10, 8), (3, 3, 12, 64)])
def test_sampled_columns_of_large_entries(r, o, n, cols):
    """Entries of many workgroups: sampled columns equal those of a subcircuit
    that has only them (attribution acts on every output column by itself)."""
    import paper_2205_05836_amd as cq
    sub = (n + o, list(range(r)) + [-1] * (n + o - r), [-1] * n + [r + u for u in range(o)])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    V = torch.randint(-8, 9, (4 ** r, 3 ** o, 2 ** (n + o)), device=DEV, generator=gen).to(torch.float64)
    E = cq.cq_attribute(sub, V)
    rng = np.random.default_rng(4)
    bs = np.sort(rng.choice(2 ** n, size=cols, replace=False))
    bs[-1] = 2 ** n - 1
    m = cols.bit_length() - 1
    Vs = V.view(4 ** r, 3 ** o, 2 ** n, 2 ** o)[:, :, torch.from_numpy(bs).to(DEV)].reshape(4 ** r, 3 ** o, -1)
    got = E[:, torch.from_numpy(bs).to(DEV)].cpu().numpy()
    # measured ends by the oracle per init string, then the init butterflies
    # (I, X, Y, Z) = (d0 + d1, 2 d2 - d0 - d1, 2 d3 - d0 - d1, d0 - d1)
    Vh = Vs.cpu().numpy()
    meas = (m + o, [-1] * (m + o), [-1] * m + list(range(o)))
    U = np.stack([at.attribute(meas, Vh[j:j + 1]) for j in range(4 ** r)])
    for t in range(r):
        d = U.reshape(4 ** t, 4, -1)
        U = np.stack([d[:, 0] + d[:, 1], 2 * d[:, 2] - d[:, 0] - d[:, 1], 2 * d[:, 3] - d[:, 0] - d[:, 1],
                      d[:, 0] - d[:, 1]], 1)
    assert np.array_equal(got, U.reshape(4 ** (r + o), -1))
