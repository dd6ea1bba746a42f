"""Variants with every size of workspace, from one state to one for each
computational init string, against the oracle.

Workspace and output start as NaN, so an amplitude that no pass wrote would
show; the bar is the state-vector tests' 1e-12 absolute."""
import ctypes as C

import numpy as np
import pytest

from oracle import statevector as sv
from workloads import circuits as wc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def spec_of(w, r, o, rng):
    init, meas = [-1] * w, [-1] * w
    cuts = [int(c) for c in rng.permutation(r + o)]
    for s in sorted(rng.choice(w, size=r, replace=False).tolist()):
        init[s] = cuts.pop()
    for s in sorted(rng.choice(w, size=o, replace=False).tolist()):
        meas[s] = cuts.pop()
    ops = []
    for t in range(9):  # deep enough that the unitaries are rewritten
        ops += [wc.Op("u", (q,), wc.haar_u2(rng)) for q in range(w)]
        ops += [wc.Op("cz", (q, q + 1)) for q in range(t % 2, w - 1, 2)]
    return wc.SubcircuitSpec(w, init, meas, [(q, 0) for q in range(w)], ops)


@pytest.mark.parametrize("w,r,o", [(1, 1, 0), (5, 2, 1), (6, 3, 3), (10, 1, 2), (11, 2, 2), (12, 3, 1), (13, 2, 3),
                                   (11, 5, 0), (18, 1, 1)])
def test_every_workspace(w, r, o):
    import paper_2205_05836_amd as cq
    from paper_2205_05836_amd import _lib
    from paper_2205_05836_amd.api import _Subs, _dev_ptr, _gates, _stream
    spec = spec_of(w, r, o, np.random.default_rng(100 * w + 10 * r + o))
    want = sv.variant_probabilities(spec)
    subs, (arr, cnt) = _Subs([spec]), _gates(spec.ops)
    sizes = sorted({1, 2, 3, 2 ** r // 2, 2 ** r - 1, 2 ** r, 2 ** r + 1} - {0})
    for states in sizes:
        print(f"w={w} r={r} o={o} states={states}", flush=True)
        out = torch.full(want.shape, float("nan"), dtype=torch.float64, device=DEV)
        ws = torch.full((2 * states << w,), float("nan"), dtype=torch.float64, device=DEV)
        assert _lib.lib().cq_variant_probabilities(subs.ptr(), arr, cnt, _dev_ptr(out), _dev_ptr(ws),
                                                   C.c_size_t(16 * states << w), _stream(None)) == 0
        assert np.max(np.abs(out.cpu().numpy() - want)) < 1e-12


def test_python_workspaces(monkeypatch):
    """Any workspace of one state or more is taken, and one state is what is
    left when memory does not hold the rest."""
    import paper_2205_05836_amd as cq
    from paper_2205_05836_amd import api
    spec = spec_of(12, 2, 1, np.random.default_rng(4))
    want = sv.variant_probabilities(spec)
    for n in (16 << 12, (16 << 12) + 8, 3 * (16 << 12)):
        got = cq.cq_variant_probabilities(spec, workspace=torch.empty(n, dtype=torch.uint8, device=DEV))
        assert np.max(np.abs(got.cpu().numpy() - want)) < 1e-12
    with pytest.raises(ValueError):
        cq.cq_variant_probabilities(spec, workspace=torch.empty((16 << 12) - 1, dtype=torch.uint8, device=DEV))
    real, asked = api._workspace, []

    def short(nbytes, device, workspace=None):
        asked.append(nbytes)
        if nbytes > 16 << 12:
            raise torch.OutOfMemoryError("no room")
        return real(nbytes, device, workspace)

    monkeypatch.setattr(api, "_workspace", short)
    got = cq.cq_variant_probabilities(spec)
    assert asked == [16 << 14, 16 << 12]
    assert np.max(np.abs(got.cpu().numpy() - want)) < 1e-12
