"""16-bit label GEMMs with a short side (subcircuits of one to three outputs),
against the oracle.

Entries are integers of magnitude at most 2 and every label sum has at most 4^4
terms of at most three factors.  Single-plane formats hold every operand exactly;
intermediate results reach 4^4 * 4 = 2^10, which needs split planes (16 bits of
significand and more) where a subcircuit of three contracts twice, so those run
in split planes only.  All sums are then exact: the device must match exactly."""
import numpy as np
import pytest

from oracle import reconstruct as rc
from workloads import synthetic as syn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# short sides of 1, 2, 4 and 8 columns or rows; long ones at the smallest size
# taken (128), at partial and whole workgroups (512), and below; labels from 1
# (outer product) over part of a step of 16 to several
CASES = [([1], [7, 1]), ([1], [1, 7]), ([1], [6, 2]), ([2], [2, 9]), ([0], [10, 1]), ([1], [10, 2]), ([2], [11, 2]),
         ([4], [3, 8]), ([0], [13, 0])]
CHAINS = [([1, 1], [1, 8, 2]), ([2, 1], [8, 3, 1]), ([1, 2], [2, 2, 9]), ([0, 2], [1, 8, 2])]


def run(bonds, outs, prec, offset):
    import paper_2205_05836_amd as cq
    rng = np.random.default_rng(sum(outs) + 10 * len(bonds))
    cm, ks = syn.chain_cutmap(bonds, outs), syn.chain_ks(bonds, len(outs))
    ents = [syn.integer_entries(rng, k, n, lo=-2, hi=2) for k, n in zip(ks, outs)]
    out = torch.empty(2 ** sum(outs) + offset, dtype=torch.float32, device="cuda:0")
    got = cq.cq_reconstruct_fd(cm, [torch.from_numpy(e).cuda() for e in ents], prec=prec, out=out[offset:])
    return got.cpu().numpy().reshape(-1), rc.fd_contract(cm, ents).reshape(-1)


@pytest.mark.parametrize("bonds,outs", CASES)
@pytest.mark.parametrize("prec", ["bf16", "fp16", "bf16_split", "fp16_split"])
@pytest.mark.parametrize("offset", [0, 1])
def test_integer_pairs_exact(bonds, outs, prec, offset):
    """``offset`` 1: the output starts 4 bytes past a 16-byte boundary."""
    got, want = run(bonds, outs, prec, offset)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("bonds,outs", CHAINS)
@pytest.mark.parametrize("prec", ["bf16_split", "fp16_split"])
def test_integer_chains_exact(bonds, outs, prec):
    got, want = run(bonds, outs, prec, 0)
    assert np.array_equal(got, want)
