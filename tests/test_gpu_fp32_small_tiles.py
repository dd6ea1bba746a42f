"""FP32 64 x 64 tiles of products with fewer labels than a stage holds, on both
sides of the line from which their ring is four stages (512 tiles): the sums
are those of the tiled kernel bit for bit."""
import pytest

from workloads import synthetic as syn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# cuts of each bond, outputs: 4 labels at 512 and 1024 tiles, ragged sides, no
# cut at all, and three subcircuits
@pytest.mark.parametrize("bonds,outs", [([1], [11, 10]), ([1], [11, 11]), ([1], [18, 5]), ([1], [4, 18]), ([1], [17, 9]),
                                        ([0], [12, 11]), ([1, 1], [9, 3, 10])])
@pytest.mark.parametrize("variant", [2, 3])
def test_bits_of_the_tiled_kernel(bonds, outs, variant):
    import paper_2205_05836_amd as cq
    print(f"{bonds} {outs} variant {variant}", flush=True)
    cm, ks = syn.chain_cutmap(bonds, outs), syn.chain_ks(bonds, len(outs))
    E = [torch.randn((4 ** k, 2 ** n), dtype=torch.float64, device=DEV) for k, n in zip(ks, outs)]
    try:
        cq.cq_autotune_enable(variant=0)
        want = cq.cq_reconstruct_fd(cm, E, "fp32")
        cq.cq_autotune_enable(variant=variant)
        out = torch.full_like(want, float("nan"))
        cq.cq_reconstruct_fd(cm, E, "fp32", out=out)
    finally:
        cq.cq_autotune_enable(True)
    assert torch.equal(out, want)
