"""Shot resolution at the edges of its forms, bit for bit against the oracle,
and the chi-square loss on odd sizes and alignments.

The form is chosen by the shots per block of 2048 outcomes: up to 16 on
average a wave per block, then a workgroup per block in registers, from 64 on
in LDS; single blocks above 64 shots are listed.  Outputs start as NaN."""
import numpy as np
import pytest

from oracle import shots

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def on_device(a, offset):
    """A copy that starts 8 * offset bytes past a 16-byte boundary."""
    buf = torch.full((a.size + offset,), float("nan"), dtype=torch.float64, device=DEV)
    return buf[offset:].view(a.shape).copy_(torch.from_numpy(np.ascontiguousarray(a)))


def rows_of(rng, rows, cols, kind):
    p = rng.exponential(size=(rows, cols)) ** 2
    if kind == "runs":      # whole runs of 64 without probability, block ends among them
        p[:, (np.arange(cols) // 64) % 3 != 1] = 0.0
        p[:, -1] = 1.0
    if kind == "crowded":   # most shots of a block on neighbouring entries
        p[:, 63:66] += p.sum() / 4
    if kind == "dead":      # a row without probability between live ones
        p[rows // 2] = 0.0
    return p / np.maximum(p.sum(axis=1, keepdims=True), 1e-300)


@pytest.mark.parametrize("rows,cols,n,kind", [
    (3, 5 * 2048, 5, "plain"), (3, 5 * 2048, 5 * 16, "plain"), (3, 5 * 2048, 5 * 16 + 1, "plain"),
    (3, 5 * 2048, 5 * 64 - 1, "runs"), (3, 5 * 2048, 5 * 64, "runs"), (2, 3 * 2048 + 64, 48, "runs"),
    (4, 2047, 16, "plain"), (4, 2047, 17, "plain"), (5, 2049, 32, "runs"), (3, 65, 16, "crowded"),
    (7, 33, 15, "dead"), (3, 40 * 2048 + 2, 640, "crowded"), (2, 64 * 2048, 1000, "runs"), (3, 1, 16, "plain")])
@pytest.mark.parametrize("offset", [0, 1])
def test_forms_bit_exact(rows, cols, n, kind, offset):
    import paper_2205_05836_amd as cq
    print(f"rows={rows} cols={cols} shots={n} {kind} offset={offset}", flush=True)
    P = rows_of(np.random.default_rng(rows + cols + n), rows, cols, kind)
    out = on_device(np.full(P.shape, np.nan), offset)
    got = cq.cq_sample_shots(on_device(P, offset), n, 2 ** 33 + n, out=out).cpu().numpy()
    assert np.array_equal(got, shots.sample_frequencies(P, n, 2 ** 33 + n))


@pytest.mark.parametrize("n", [1, 2, 3, 1023, 2 ** 20 + 1, 3 * 2 ** 20])
def test_chi2_sizes_and_alignments(n):
    """Within 1e-12 of the sum of the terms' magnitudes (the additions' order
    differs from the oracle's), and the same bits whatever the alignment."""
    import paper_2205_05836_amd as cq
    rng = np.random.default_rng(n)
    a, b = rng.random(n), rng.random(n)
    a[::5], b[::5] = 0.0, 0.0
    vals = [float(cq.cq_chi2(on_device(a, i), on_device(b, j))[0]) for i, j in ((0, 0), (1, 0), (1, 1))]
    assert vals[0] == vals[1] == vals[2]
    assert abs(vals[0] - shots.chi2(a, b)) <= 1e-12 * max(shots.chi2(a, b), 1e-300)


@pytest.mark.parametrize("rows,cols,n,kind", [
    (1, 2048, 6144, "plain"), (1, 2048, 6145, "plain"), (3, 1, 8193, "plain"), (5, 17, 2 ** 18 + 3, "dead"),
    (2, 1233, 4096 * 9, "crowded"), (1023, 64, 8000, "runs"), (1024, 64, 8000, "plain"), (300, 100, 40000, "dead")])
def test_rows_of_one_block_bit_exact(rows, cols, n, kind):
    """Rows of one block: whole in a workgroup, or their shots spread over
    several, at the lines between the two and with a last part that is short."""
    import paper_2205_05836_amd as cq
    print(f"rows={rows} cols={cols} shots={n} {kind}", flush=True)
    P = rows_of(np.random.default_rng(rows + cols + n), rows, cols, kind)
    out = on_device(np.full(P.shape, np.nan), 1)
    got = cq.cq_sample_shots(on_device(P, 0), n, n, out=out).cpu().numpy()
    assert np.array_equal(got, shots.sample_frequencies(P, n, n))
