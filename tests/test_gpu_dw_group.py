"""Weight gradients of a layer in one launch, and GEMMs whose reduction is no
multiple of 64, against the one-problem launches and the register-staged kernel."""
import numpy as np
import pytest

import synth
from parity import to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _cfg(name, **kw):
    return synth.PartitionConfig(name, **dict(dict(layers=2, d_model=192, d_ff=328, heads=3, seq=32, batch=3, micro=3,
                                                   dtype="bf16"), **kw))


CASES = [
    # one micro-batch of 32 rows: less than one k-tile; widths with partial tiles; d_ff % 64 = 8
    _cfg("rows32"),
    # pairs of 2 x 96 rows and a last single 96 (K = 64 + 32); d_ff % 64 = 40
    _cfg("rows96", seq=96, d_ff=424),
    # the groups' problems differ in K (memory rows), ragged and whole; 1, 2, 3 .. whole tiles of width
    _cfg("decoder", kind="decoder", mem_seq=64, batch=4, micro=2, d_model=128, heads=2, d_ff=392),
    _cfg("decoder_m1", kind="decoder", seq=64, mem_seq=32, batch=3, micro=1, loss="xent_ls", vocab=136,
         label_smoothing=0.1),
    # a group large enough to be handed over before the layer's end
    _cfg("wide", layers=1, d_model=1024, heads=16, d_ff=8192 + 8, seq=32, batch=2, micro=2),
]




def _step(cfg, case):
    from paper_1811_06965_amd.runtime import Partition
    with Partition(cfg) as part:
        part.load_params(case["layers"], case["head"])
        inp = part.device_inputs(case)
        for _ in range(2):  # the second step accumulates afresh
            out = part.step(inp["x"], inp["mem"], inp["dy"])
        gl, gh = part.grads()
    res = {"y": to_np(out["y"]), "dx": to_np(out["dx"])}
    for l, g in enumerate(gl + [gh]):
        res.update({f"{l}.{k}": v for k, v in g.items()})
    return res


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_grouped_weight_gradients_equal_single_launches(cfg, monkeypatch):
    """Fewer than eight k-tiles per reduction over rows: no launch splits it, so
    the grouping changes no bit."""
    case = synth.make_case(cfg, 5, perturb=True)
    ref = _step(cfg, case)
    for flush in ("0", "2"):
        monkeypatch.setenv("GP_DW_FLUSH", flush)
        res = _step(cfg, case)
        for k, v in ref.items():
            assert np.array_equal(v, res[k]), (flush, k)


@pytest.mark.parametrize("cfg", [c for c in CASES if c.d_ff < 512], ids=lambda c: c.name)
def test_ragged_reductions_equal_the_register_staged_kernel(cfg, monkeypatch):
    """Every width is below 512 (no split-K), and both kernels add an element's
    products in the same order: equal bits, except the bias gradients, whose
    column sums are fp32 sums of at most 192 rows in another order (error bound
    192 * 2^-24 of the sum of magnitudes, which is within 10 of the result's
    norm here: 1.2e-4)."""
    case = synth.make_case(cfg, 5, perturb=True)
    ref = _step(cfg, case)
    monkeypatch.setenv("GP_GEMM_TILE", "3")
    monkeypatch.setenv("GP_GEMM_SPLITS", "1")
    res = _step(cfg, case)
    for k, v in ref.items():
        if k.split(".")[-1] in ("bq", "bv", "bo", "b1", "b2", "xbq", "xbv", "xbo", "bout"):
            assert np.linalg.norm(v - res[k]) <= 1.2e-4 * np.linalg.norm(v), k
        elif k.split(".")[-1] not in ("bk", "xbk"):  # zero but for rounding
            assert np.array_equal(v, res[k]), k
