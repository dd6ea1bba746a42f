"""The state-vector passes that touch qubits as late as possible, and the
variants combined from computational init strings, against the oracle.

Amplitudes outside the touched set are never stored, so every workspace and
output starts as NaN: reading one that no pass wrote would show.  Values are
sums of products of factors of magnitude at most 1 over at most a few hundred
gates: the bar is the state-vector tests' 1e-12 absolute."""
import numpy as np
import pytest

from oracle import statevector as sv
from workloads import circuits as wc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def nan_bytes(n):
    return torch.full((max(n // 8, 1),), float("nan"), dtype=torch.float64, device=DEV).view(torch.uint8)


def line(n, layers, rng, qubits=None):
    qs = list(range(n)) if qubits is None else qubits
    ops = []
    for t in range(layers):
        ops += [wc.Op("u", (q,), wc.haar_u2(rng)) for q in qs]
        ops += [wc.Op("cz", (qs[i], qs[i + 1])) for i in range(t % 2, len(qs) - 1, 2)]
    return ops


def pairs(n, layers, rng):
    ops = []
    for _ in range(layers):
        ops += [wc.Op("u", (q,), wc.haar_u2(rng)) for q in range(n)]
        p = rng.permutation(n)
        ops += [wc.Op("cz", (int(p[i]), int(p[i + 1]))) for i in range(0, n - 1, 2)]
    return ops


CIRCUITS = [
    ("line", 12, lambda r: line(12, 3, r)), ("line", 13, lambda r: line(13, 12, r)),
    ("line", 18, lambda r: line(18, 8, r)), ("line", 19, lambda r: line(19, 3, r)),
    ("random pairs", 18, lambda r: pairs(18, 5, r)),
    ("highest index bits idle", 18, lambda r: line(18, 6, r, list(range(7, 18)))),
    ("lowest index bits idle", 18, lambda r: line(18, 6, r, list(range(0, 12)))),
    ("every third qubit", 18, lambda r: line(18, 5, r, list(range(0, 18, 3)))),
    ("one gate", 18, lambda r: [wc.Op("u", (4,), wc.haar_u2(r))]),
    ("signs only", 14, lambda r: [wc.Op("cz", (0, 13)), wc.Op("cz", (3, 4))]),
    ("signs last", 12, lambda r: line(12, 2, r) + [wc.Op("cz", (a, b)) for a in range(12) for b in range(a)]),
    # more one-qubit gates, and more gates, on one tile than a pass takes
    ("many on a tile", 18, lambda r: line(18, 40, r, list(range(8, 18)))),
    ("long sign runs", 12, lambda r: line(12, 1, r) + [wc.Op("cz", (int(a), int(a + 1) % 12)) for a in
                                                      r.integers(0, 12, 400)] + line(12, 1, r)),
]


@pytest.mark.parametrize("name,n,make", CIRCUITS, ids=[f"{c[0]}-{c[1]}" for c in CIRCUITS])
def test_touched_set_growth(name, n, make):
    import paper_2205_05836_amd as cq
    print(f"{name} n={n}", flush=True)
    ops = make(np.random.default_rng(n))
    out = torch.full((2 ** n,), float("nan"), dtype=torch.float64, device=DEV)
    cq.cq_simulate_probabilities(n, ops, out=out, workspace=nan_bytes(cq.cq_simulate_workspace_size(n)))
    got, want = out.cpu().numpy(), sv.probabilities(n, ops)
    assert np.max(np.abs(got - want)) < 1e-12


def spec_of(w, r, o, rng, where):
    init, meas = [-1] * w, [-1] * w
    cuts = list(rng.permutation(r + o))
    for s in sorted(rng.choice(w, size=r, replace=False).tolist()):
        init[s] = int(cuts.pop())
    ms = range(w - o, w) if where == "last" else sorted(rng.choice(w, size=o, replace=False).tolist())
    for s in ms:
        meas[s] = int(cuts.pop())
    return wc.SubcircuitSpec(w, init, meas, [(q, 0) for q in range(w)], line(w, 3, rng))


@pytest.mark.parametrize("w,r,o,where", [
    (1, 1, 1, "last"), (4, 0, 1, "last"), (4, 2, 0, "last"), (6, 1, 3, "mixed"), (5, 3, 3, "last"),
    (8, 0, 5, "mixed"), (8, 5, 0, "mixed"), (9, 3, 2, "last"), (9, 2, 4, "mixed"), (10, 1, 2, "last"),
    (11, 2, 3, "last"), (12, 3, 1, "mixed"), (13, 2, 2, "last"), (18, 1, 1, "mixed"), (18, 0, 2, "last")])
@pytest.mark.parametrize("offset", [0, 1])
def test_variants_from_computational_strings(w, r, o, where, offset):
    """``offset`` 1: the output starts 8 bytes past a 16-byte boundary."""
    import paper_2205_05836_amd as cq
    print(f"w={w} r={r} o={o} {where}", flush=True)
    spec = spec_of(w, r, o, np.random.default_rng(100 * w + 10 * r + o), where)
    want = sv.variant_probabilities(spec)
    buf = torch.full((want.size + offset,), float("nan"), dtype=torch.float64, device=DEV)
    out = buf[offset:].view(want.shape)
    cq.cq_variant_probabilities(spec, out=out, workspace=nan_bytes(cq.cq_variants_workspace_size(spec)))
    assert np.max(np.abs(out.cpu().numpy() - want)) < 1e-12


@pytest.mark.parametrize("w,r,o", [(6, 2, 1), (12, 1, 2), (12, 1, 8)])
def test_variants_one_state_at_a_time(w, r, o):
    """A workspace of one state, with the results of the full one."""
    import paper_2205_05836_amd as cq
    from paper_2205_05836_amd import _lib
    from paper_2205_05836_amd.api import _Subs, _dev_ptr, _gates, _stream
    spec = spec_of(w, r, min(o, 7), np.random.default_rng(w + r + o), "mixed")
    want = cq.cq_variant_probabilities(spec)
    out = torch.full_like(want, float("nan"))
    ws = nan_bytes(16 << w)
    subs, (arr, cnt) = _Subs([spec]), _gates(spec.ops)
    assert _lib.lib().cq_variant_probabilities(subs.ptr(), arr, cnt, _dev_ptr(out), _dev_ptr(ws), 16 << w,
                                               _stream(None)) == 0
    assert float((out - want).abs().max()) < 1e-12


def matrix(kind, rng):
    """One-qubit matrices around the edges of the normalised form."""
    z = np.exp(1j * rng.uniform(0, 2 * np.pi, 4))
    if kind == "small pivot":  # |u00| = |u11| about a 16th, below and above, and next to nothing
        c = float(rng.choice([1 / 16 * 0.99, 1 / 16 * 1.01, 1e-3, 1e-30]))
        s = np.sqrt(1 - c * c)
        return np.array([[c, -s], [s, c]]) * z[0] * np.array([[1, z[1]], [1, z[1]]])
    if kind == "exchange":  # zero diagonal or zero off-diagonal
        return np.array([[0, z[0]], [z[1], 0]]) if rng.random() < 0.5 else np.diag(z[:2])
    if kind == "not unitary":  # unequal rows, up to a factor of 64 each
        return (rng.normal(size=(2, 2)) + 1j * rng.normal(size=(2, 2))) * np.exp2(rng.uniform(-3, 3, (2, 1)))
    return np.outer(rng.normal(size=2), rng.normal(size=2)) + 0j  # rank one: a measured branch


@pytest.mark.parametrize("kind", ["small pivot", "exchange", "not unitary", "rank one"])
@pytest.mark.parametrize("n,layers", [(11, 3), (12, 40), (14, 9)])
def test_matrix_forms(kind, n, layers):
    """Matrices that the normalised form takes, just takes and does not, mixed
    with Haar ones, deep enough that the factors it holds back reach their
    bound.  Errors are compared with the largest probability (the matrices of
    two kinds do not keep the norm); the bar is that of the tests above."""
    import paper_2205_05836_amd as cq
    rng = np.random.default_rng(n + layers)
    ops = []
    for t in range(layers):
        ops += [wc.Op("u", (q,), matrix(kind, rng) if rng.random() < 0.5 else wc.haar_u2(rng)) for q in range(n)]
        ops += [wc.Op("cz", (i, i + 1)) for i in range(t % 2, n - 1, 2)]
    want = sv.probabilities(n, ops)
    got = cq.cq_simulate_probabilities(n, ops).cpu().numpy()
    assert np.abs(got - want).max() <= 1e-12 * want.max()
