"""Operand preparation of a full-definition call: every operand in one launch a
stage, at the shapes where its kernels change form -- one and two columns
(rows share a wave, no four-element groups), columns in the thousands under
few rows (a row split over waves), rows below and above a column fold, inputs
that are only 8-byte aligned -- against the FP64 oracle.

Tolerance, relative to the bin's scale sum_l prod_c |E_c[l, b]|: entries are
uniform in +-[0.5, 1) before exact powers of two per label that cancel in every
term, so each operand and each intermediate is rounded by u (2^-24 FP32, 2^-20
split planes, whose lo plane may be subnormal, 2^-10 FP16, 2^-8 BF16): 2 n_C
roundings of 2 u each, and n_C FP32 sums of at most 4^3 terms of 2^-23 each.
A wrong power of two in any row or column is an error of the scale itself."""
import numpy as np
import pytest

from oracle import cutmap
from oracle import reconstruct as rc
from workloads import synthetic as syn

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

U = {"fp32": 2.0 ** -24, "fp16_split": 2.0 ** -20, "bf16_split": 2.0 ** -15, "fp16": 2.0 ** -10, "bf16": 2.0 ** -8}
SHIFT = [0, 9, -7, 4]


def label_shift(cm, E):
    out = []
    for sub, e in zip(cm, E):
        cuts, meas = cutmap.incident_cuts(sub), sub[2]
        ex = np.zeros(e.shape[0], dtype=np.int64)
        for l in range(e.shape[0]):
            for p, cut in enumerate(cuts):
                d = (l >> (2 * (len(cuts) - 1 - p))) & 3
                ex[l] += SHIFT[d] if cut in meas else -SHIFT[d]
        out.append(np.ldexp(e, ex[:, None]))
    return out


def device(a, offset):
    """`a` on the device, `offset` doubles past an allocation's start."""
    buf = torch.empty(a.size + offset, dtype=torch.float64, device="cuda:0")
    t = buf[offset:].view(a.shape)
    t.copy_(torch.from_numpy(np.ascontiguousarray(a)))
    return t


@pytest.mark.parametrize("bonds,ns", [([1], [1, 1]), ([1], [2, 13]), ([2], [14, 3]), ([3], [3, 6]), ([2, 3], [7, 6, 9]),
                                      ([1, 1, 2], [3, 11, 1, 4])])
@pytest.mark.parametrize("prec", sorted(U))
@pytest.mark.parametrize("balance,offset", [(1, 0), (1, 1), (0, 0)])
def test_prepared_operands_match_oracle(bonds, ns, prec, balance, offset):
    import paper_2205_05836_amd as m
    rng = np.random.default_rng(len(ns) * 100 + ns[0])
    cm = syn.chain_cutmap(bonds, ns)
    E = [np.copysign(rng.uniform(0.5, 1.0, size=(4 ** k, 2 ** n)), rng.uniform(-1, 1, size=(4 ** k, 2 ** n)))
         for k, n in zip(syn.chain_ks(bonds, len(ns)), ns)]
    ref = rc.fd_contract(cm, E)
    scale = rc.fd_contract(cm, [np.abs(e) for e in E])
    # the 16-bit range needs the balance (FP32 and BF16 carry the labels as they are)
    if balance or not prec.startswith("fp16"):
        E = label_shift(cm, E)
    dev = [device(e, offset) for e in E]
    try:
        m.cq_label_balance_enable(balance)
        out = m.cq_reconstruct_fd(cm, dev, prec=prec).cpu().numpy().astype(np.float64)
    finally:
        m.cq_label_balance_enable(1)
    tol = 4 * len(ns) * U[prec] + len(ns) * 4 ** 3 * 2.0 ** -23
    worst = (np.abs(out - ref) / scale).max()
    print(f"{prec} {bonds} {ns}: {worst:.2e} of {tol:.2e}", flush=True)
    assert worst <= tol


@pytest.mark.parametrize("outs", [[1, 3], [6, 3]])
def test_bf16_operands_are_rounded_through_fp32(outs):
    """FP64 values a little off a BF16 tie that FP32 rounds onto it: the
    operand is the BF16 of the FP32 value, which goes to the even neighbour.
    One cut whose only nonzero label pairs each value with a one, so every
    output is half an operand exactly."""
    import paper_2205_05836_amd as m
    cm = syn.chain_cutmap([1], outs)
    base = 1.0 + 2.0 ** -7 * np.arange(2 ** outs[0])  # BF16 values of [1, 2)
    off = np.where(np.arange(2 ** outs[0]) % 2 == 0, 2.0 ** -40, -2.0 ** -40)  # towards the odd neighbour
    E = [np.zeros((4, 2 ** n)) for n in outs]
    E[0][0] = base + 2.0 ** -8 + off
    E[1][0] = 1.0
    want = torch.from_numpy(E[0][0]).float().bfloat16().double().numpy()
    assert not np.array_equal(want, base + 2.0 ** -7 * (off > 0))  # one rounding would differ
    out = m.cq_reconstruct_fd(cm, [torch.from_numpy(e).cuda() for e in E], prec="bf16").cpu().numpy()
    assert np.array_equal(out.reshape(2 ** outs[0], -1), np.repeat(0.5 * want[:, None], 2 ** outs[1], 1))
