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
    # reductions over 2 x 1024 and 768 rows that single launches split
    _cfg("rows2048", layers=1, d_model=256, heads=4, d_ff=512, seq=256, batch=8, micro=2),
    _cfg("rows768_m3", layers=1, d_model=128, heads=2, d_ff=512, seq=256, batch=9, micro=3),
    # jobs large enough to be handed over alone, and a group of the rest
    _cfg("wide", layers=1, d_model=1024, heads=16, d_ff=8192 + 8, seq=32, batch=2, micro=2),
    # jobs that are large enough only together: a group handed over in the middle of the layer, and one of the rest
    _cfg("two_groups", layers=1, d_model=1024, heads=16, d_ff=4096 + 8, seq=32, batch=2, micro=2),
    _cfg("two_groups_decoder", layers=1, d_model=1024, heads=16, d_ff=4096 - 40, seq=32, mem_seq=64, batch=2, micro=2,
         kind="decoder"),
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
    """A group adds up each reduction as its own launch does, split over workgroups
    or not, so neither the grouping nor the time of the hand-over changes a bit."""
    case = synth.make_case(cfg, 5, perturb=True)
    ref = _step(cfg, case)
    for flush in ("0", "1", "2"):
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


def test_timed_groups_are_the_launches_of_an_untimed_step():
    """A selected role times the grouped launch itself: the roles share its time
    by their FLOPs (o : qkv : ffn = 1 : 3 : 4), each counts one launch per layer and
    pair, and the gradients keep their bits."""
    from paper_1811_06965_amd.runtime import Partition
    cfg = _cfg("timed", d_model=256, heads=4, d_ff=1024, seq=256, batch=8, micro=4)
    case = synth.make_case(cfg, 5, perturb=True)
    ref = _step(cfg, case)
    with Partition(cfg) as part:
        part.load_params(case["layers"], case["head"])
        inp = part.device_inputs(case)
        part.timer_select("all")
        part.step(inp["x"], inp["mem"], inp["dy"])
        torch.cuda.synchronize()
        got = {r: part.timer_read(r + ".dw") for r in ("o", "qkv", "ffn1", "ffn2")}
        part.timer_reset()
        part.timer_select("o.dw")
        part.timer_sample(2)
        out = part.step(inp["x"], inp["mem"], inp["dy"])
        torch.cuda.synchronize()
        part.timer_select(None)
        sampled = part.timer_read("o.dw")
        gl, _ = part.grads()
    for role, n in (("o", 1), ("qkv", 3), ("ffn1", 4), ("ffn2", 4)):
        assert got[role]["launches"] == 4
        assert got[role]["flops"] == pytest.approx(n * 4 * 2 * 1024 * 256 * 256)
        assert got[role]["ms"] == pytest.approx(n * got["o"]["ms"]) and got[role]["ms"] > 0
    assert sampled["launches"] == 2 and 0 < sampled["ms"]
    assert np.array_equal(to_np(out["dx"]), ref["dx"])
    for l, g in enumerate(gl):
        for k, v in g.items():
            assert np.array_equal(v, ref[f"{l}.{k}"]), (l, k)
