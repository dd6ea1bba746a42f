"""The FP64 label GEMM on its tile edges, against the oracle.

Entries are integers of magnitude at most 8 and every label sum has at most
4^5 terms of at most 4 factors, so all sums are integers far below 2^53 (then
scaled by a power of two): the device must match the oracle exactly."""
import numpy as np
import pytest

from oracle import reconstruct as rc
from workloads import synthetic as syn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# labels per contraction 1 (outer product), 4 (half a stage), 16, 64 and 256;
# rows and columns from 1 and 2 to several 64 x 128 tiles, partial ones among them
CASES = [([0], [1, 1]), ([0], [7, 6]), ([1], [1, 6]), ([1], [6, 1]), ([1], [5, 8]), ([2], [4, 4]), ([2], [9, 7]),
         ([3], [3, 9]), ([4], [7, 7]), ([4], [8, 5]), ([0, 2], [3, 4, 5]), ([1, 2], [2, 6, 3]), ([2, 3], [5, 3, 8]),
         ([2, 1, 2], [4, 2, 3, 4])]


@pytest.mark.parametrize("bonds,outs", CASES)
@pytest.mark.parametrize("offset", [0, 1])
def test_integer_chains_exact(bonds, outs, offset):
    """``offset`` 1: every entry tensor starts 8 bytes past a 16-byte
    boundary, which the aligned kernel does not take."""
    import paper_2205_05836_amd as cq
    print(f"bonds {bonds} outputs {outs} offset {offset}", flush=True)
    rng = np.random.default_rng(sum(outs) + 10 * len(bonds))
    cm, ks = syn.chain_cutmap(bonds, outs), syn.chain_ks(bonds, len(outs))
    ents = [syn.integer_entries(rng, k, n) for k, n in zip(ks, outs)]
    dev = []
    for e in ents:
        buf = torch.empty(e.size + offset, dtype=torch.float64, device=DEV)
        dev.append(buf[offset:].view(e.shape).copy_(torch.from_numpy(e)))
    got = cq.cq_reconstruct_fd(cm, dev).cpu().numpy()
    assert np.array_equal(got, rc.fd_contract(cm, ents).reshape(-1))
