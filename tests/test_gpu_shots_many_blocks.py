"""Shot resolution in tables of about 2048 blocks and more, from which a wave
resolves a block with few shots, bit for bit against the oracle."""
import numpy as np
import pytest

from oracle import shots

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def table(rows, cols, kind):
    rng = np.random.default_rng(rows + cols)
    p = rng.exponential(size=(rows, cols)) ** 2
    if kind == "runs":  # whole runs of 64 without probability, block ends among them
        p[:, (np.arange(cols) // 64) % 3 != 1] = 0.0
        p[:, -1] = 1.0
    if kind == "crowded":  # most shots of a row on neighbouring entries: blocks with more than 64
        p[:, 63:66] += p.sum() / 4
    p[rows // 2] = 0.0
    return p / np.maximum(p.sum(axis=1, keepdims=True), 1e-300)


# 2046, 2048 and 2050 blocks (the line), and more
@pytest.mark.parametrize("rows,cols,n,kind", [
    (1023, 2049, 32, "runs"), (1024, 2049, 32, "runs"), (410, 5 * 2048, 5, "plain"), (410, 5 * 2048, 80, "plain"),
    (410, 5 * 2048, 81, "plain"), (700, 3 * 2048 + 64, 48, "runs"), (60, 40 * 2048 + 2, 640, "crowded"),
    (33, 64 * 2048, 1000, "runs")])
@pytest.mark.parametrize("offset", [0, 1])
def test_forms_bit_exact(rows, cols, n, kind, offset):
    import paper_2205_05836_amd as cq
    print(f"rows={rows} cols={cols} shots={n} {kind} offset={offset}", flush=True)
    P = table(rows, cols, kind)
    buf = torch.full((2, P.size + offset), float("nan"), dtype=torch.float64, device=DEV)
    src, out = (b[offset:].view(P.shape) for b in (buf[0].clone(), buf[1].clone()))
    src.copy_(torch.from_numpy(P))
    got = cq.cq_sample_shots(src, n, 2 ** 33 + n, out=out).cpu().numpy()
    assert np.array_equal(got, shots.sample_frequencies(P, n, 2 ** 33 + n))


@pytest.mark.parametrize("rows,cols,n", [(1024, 2049, 32), (410, 5 * 2048, 80)])
def test_no_room_for_run_sums(rows, cols, n):
    """Workspaces from what every call needs up to a byte below what is asked for."""
    import paper_2205_05836_amd as cq
    print(f"rows={rows} cols={cols} shots={n}", flush=True)
    P = table(rows, cols, "plain")
    src, want = torch.from_numpy(P).to(DEV), shots.sample_frequencies(P, n, 5)
    up = lambda b: (b + 255) // 256 * 256
    blocks = rows * -(-cols // 2048)
    need = up(8 * blocks) + 3 * up(4 * blocks) + up(8 * rows * n)
    asked = cq.cq_sample_shots_workspace_size(rows, cols, n)
    assert asked == need + 256 * blocks
    for size in (need, asked - 1, asked):
        got = cq.cq_sample_shots(src, n, 5, workspace=torch.empty(size, dtype=torch.uint8, device=DEV))
        assert np.array_equal(got.cpu().numpy(), want)
    with pytest.raises(ValueError):
        cq.cq_sample_shots(src, n, 5, workspace=torch.empty(need - 1, dtype=torch.uint8, device=DEV))
