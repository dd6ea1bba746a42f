"""Long FP64 outputs of products with fewer labels than a stage holds, on both
sides of the line from which they take 128 x 128 tiles."""
import pytest

from workloads import synthetic as syn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# 2^27 outputs with 128, 256 and 1024 columns, half as many, and no cut
@pytest.mark.parametrize("cuts,outs", [(1, [20, 7]), (1, [19, 8]), (1, [17, 10]), (1, [18, 8]), (0, [19, 8])])
def test_long_outputs(cuts, outs):
    """K products of 0..1 values round to within K eps of their sum each way."""
    import paper_2205_05836_amd as cq
    print(f"{cuts} {outs}", flush=True)
    cm = syn.chain_cutmap([cuts], outs)
    E = [torch.rand((4 ** cuts, 2 ** n), dtype=torch.float64, device=DEV) for n in outs]
    out = torch.full((2 ** sum(outs),), float("nan"), dtype=torch.float64, device=DEV)
    cq.cq_reconstruct_fd(cm, E, "fp64", out=out)
    got = out.view(2 ** outs[0], 2 ** outs[1])
    want = torch.zeros_like(got)
    for a, b in zip(E[0], E[1]):
        want.addr_(a, b)
    want *= 0.5 ** cuts
    assert ((got - want).abs() <= 2 * 4 ** cuts * 2.0 ** -52 * want).all()
