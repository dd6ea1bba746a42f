"""Output orders of a full definition: tiles of a bit permutation and the
generic form below them, bit for bit against the unpermuted call.

A permutation only moves values.  FP64 and FP32 calls keep the last GEMM's
results as they are, so every order must equal the unpermuted call (one kernel
variant is fixed).  The 16-bit forms store those results in their planes before
the permutation: there every order, undone, must equal every other bit for bit,
and lie within the planes' rounding of the unpermuted call (all terms are
positive: 2^-15 relative for BF16 split planes, 2^-20 for FP16 ones, whose lo
plane may be subnormal, 2^-10 for FP16).  Sizes lie around the smallest tile
(2^10), the change of tile (2^22) and between; the orders are the identity with
its ends exchanged, a reversal (runs of one element), a rotation by one
subcircuit and a random one."""
import numpy as np
import pytest

from oracle import reconstruct as rc
from workloads import synthetic as syn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def orders(n, first):
    rng = np.random.default_rng(n)
    return {"ends": [n - 1] + list(range(1, n - 1)) + [0], "reversed": list(range(n))[::-1],
            "rotated": list(range(first, n)) + list(range(first)), "random": list(rng.permutation(n))}


@pytest.mark.parametrize("outs", [[4, 5], [5, 5], [6, 5], [7, 6, 4], [10, 11], [11, 11], [8, 9, 6]])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16_split", "fp16", "fp16_split"])
def test_orders_move_values_only(outs, prec):
    import paper_2205_05836_amd as cq
    rng = np.random.default_rng(3)
    bonds = [1] * (len(outs) - 1)
    cm = syn.chain_cutmap(bonds, outs)
    ents = [torch.from_numpy(rng.uniform(0.1, 1.0, size=(4 ** k, 2 ** n))).cuda()
            for k, n in zip(syn.chain_ks(bonds, len(outs)), outs)]
    n = sum(outs)
    cq.cq_autotune_enable(0)
    try:
        plain = cq.cq_reconstruct_fd(cm, ents, prec=prec).cpu().numpy()
        first = None
        for name, perm in orders(n, outs[0]).items():
            got = cq.cq_reconstruct_fd(cm, ents, prec=prec, out_perm=[int(q) for q in perm]).cpu().numpy()
            got = rc.apply_out_perm(got, np.argsort(perm))  # concatenated order again
            print(f"{prec} {outs} {name}: {np.array_equal(got, plain)}", flush=True)
            if first is None:
                first = plain if prec in ("fp64", "fp32") else got
            assert np.array_equal(got, first), name
        tol = {"bf16_split": 2.0 ** -15, "fp16_split": 2.0 ** -20, "fp16": 2.0 ** -10}.get(prec, 0.0)
        assert (np.abs(first - plain) <= tol * np.abs(plain)).all()
    finally:
        cq.cq_autotune_enable(1)
