"""The autotuner's report names the kernel that runs (host only: launches are
recorded instead of run, so every trial ties and variant 0 is kept)."""
import json

import pytest

import launch_recorder
from workloads import synthetic as syn


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return launch_recorder.build(tmp_path_factory.mktemp("recorder"))


SCRIPT = """
L.cq_autotune_enable(1)
def fd(cm, prec, shift):
    s = api._Subs(cm)
    call = lambda: L.cq_reconstruct_fd(
        len(cm), s.ptr(), (C.c_void_p * len(cm))(*[((i + 1) << 40) + shift for i in range(len(cm))]),
        _lib.PRECISION[prec], None, C.c_void_p(1 << 50), C.c_void_p(1 << 51), 1 << 45, None)
    before = {json.dumps([e[k] for k in "MNKZ"]) for e in cq.cq_autotune_json() if e["prec"] == prec}
    assert call() == 0
    events()
    assert call() == 0
    new = [e for e in cq.cq_autotune_json() if e["prec"] == prec and json.dumps([e[k] for k in "MNKZ"]) not in before]
    return [[e["kernel"] for e in events() if "gemm_" in e["kernel"]], new]
out = [fd(*c) for c in json.loads(CASES)]
"""

KERNELS = {"gemm_f64t_kernel": "occupancy", "gemm_f64s_kernel": "small-tile", "gemm_f64_kernel": "tiled",
           "gemm_f32_kernel": "tiled", "gemm_h16a_kernel": "async", "gemm_h16n_kernel": "short-side",
           "gemm_h16_kernel": "register"}
# outputs of two subcircuits with two cuts: long and even, one side of 2, 4 and
# 1, and a few hundred a side
OUTS = [[12, 12], [1, 14], [2, 13], [14, 1], [10, 10], [0, 15]]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16", "bf16_split"])
@pytest.mark.parametrize("shift", [0, 8])
def test_report_names_what_runs(recorder, prec, shift):
    for outs in OUTS:  # a process each: the cache is keyed by shape
        cases = [(syn.chain_cutmap([0 if 0 in outs else 1], outs), prec, shift)]
        (launched, entries), = launch_recorder.run(recorder, f"CASES = {json.dumps(cases)!r}\n" + SCRIPT)
        for e in entries:
            names = {next(v for n, v in KERNELS.items() if n in k) for k in launched}
            assert names == {e["schedule"]["kernel"]}, (outs, launched, e)


def test_small_fp32_tiles_of_short_products(recorder):
    """The ring of forced 64 x 64 tiles: four stages' LDS below 16 labels where
    there are many tiles, whole ones."""
    cases = [(syn.chain_cutmap([b], outs), "fp32", 0)
             for b, outs in ((1, [10, 10]), (1, [12, 12]), (2, [12, 12]), (1, [18, 6]), (1, [18, 5]), (1, [5, 18]))]
    script = SCRIPT.replace("L.cq_autotune_enable(1)", "L.cq_autotune_enable(4)")
    got = launch_recorder.run(recorder, f"CASES = {json.dumps(cases)!r}\n" + script)
    assert [int(k[0].split(", ")[1].split(">")[0]) for k, _ in got] == [8, 4, 2, 4, 2, 2]


def test_report_of_loaded_choices(recorder, tmp_path):
    """FP32 64 x 64 tiles run an eight-deep ring up to 512 of them and a two-
    or four-deep one beyond; FP64 rows of 2 or 4 columns take the aligned
    kernels."""
    ms = " ".join(["0.5"] * 12)
    rows = [(1, 1, 1024, 2048, 2), (1, 1, 2048, 2048, 2), (0, 0, 4, 1 << 15, 0), (0, 0, 4, 1 << 17, 0),
            (0, 0, 1024, 1024, 0), (0, 1, 1024, 1024, 0)]
    path = tmp_path / "tune.txt"
    path.write_text("".join(f"cq-tune-1 gfx950-256cu {p} {p} 0 1 1 {al} {M} {N} 16 1 {v} 15 {ms}\n"
                            for p, al, M, N, v in rows))
    got = launch_recorder.run(recorder, f"cq.cq_autotune_load({str(path)!r})\nout = cq.cq_autotune_json()\n")
    sched = {(e["prec"], e["M"], e["N"]): e["schedule"] for e in got if (e["M"], e["N"]) != (1024, 1024)}
    assert sched["fp32", 1024, 2048]["ring"] == 8 and sched["fp32", 2048, 2048]["ring"] == 2
    assert sched["fp64", 4, 1 << 15]["kernel"] == "small-tile" and sched["fp64", 4, 1 << 17]["kernel"] == "occupancy"
    both = [e["schedule"]["kernel"] for e in got if (e["M"], e["N"]) == (1024, 1024)]
    assert sorted(both) == ["small-tile", "tiled"]
