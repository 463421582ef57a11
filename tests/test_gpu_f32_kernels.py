"""fp32 kernels at the edges of their tiles, against the fp64 oracle and each other."""
import numpy as np
import pytest

import synth
from parity import compare_grads, rel_err, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _step(cfg, case):
    from paper_1811_06965_amd.runtime import Partition
    with Partition(cfg) as part:
        part.load_params(case["layers"], case["head"])
        inp = part.device_inputs(case)
        out = part.step(inp["x"], inp["mem"], inp["dy"])
        torch.cuda.synchronize()
        gl, gh = part.grads()
    return dict(y=to_np(out["y"]), dx=to_np(out["dx"]), loss=out["loss"], grads=gl, head=gh)


def _against_oracle(cfg, case, res):
    """The fp32 parity bound of 1e-4 that every fp32 partition is held to."""
    from oracle import gpipe
    ref = gpipe.gpipe_step(cfg, case, cfg.micro)
    assert rel_err(res["y"], ref["y"]) <= 1e-4
    assert rel_err(res["dx"], ref["dx"]) <= 1e-4
    assert abs(res["loss"] - ref["loss"]) <= 1e-4 * abs(ref["loss"])
    compare_grads(res["grads"], res["head"], ref["grads"], ref["head_grads"], "rel", 1e-4)


# widths and rows that are no multiples of a tile or of a 32-deep k-tile, and
# rows of several 128-row tiles; the reductions end 4, 8, 12, 16 .. past a k-tile
GEMM_CASES = {
    "edges": synth.PartitionConfig("edges", layers=1, d_model=72, d_ff=200, heads=6, seq=20, batch=6, micro=3,
                                   dtype="f32", kind="decoder", loss="xent_ls", vocab=104, label_smoothing=0.1,
                                   mem_seq=12),
    "wide": synth.PartitionConfig("wide", layers=2, d_model=144, d_ff=328, heads=4, seq=68, batch=10, micro=2,
                                  dtype="f32", loss="mse"),
}


@pytest.mark.parametrize("name", sorted(GEMM_CASES))
def test_f32_gemm_tiles_agree_bit_for_bit(name, monkeypatch):
    """Every tile sums each element in the same order, so forcing any of them
    gives the same bits; one of them against the oracle."""
    cfg = GEMM_CASES[name]
    case = synth.make_case(cfg, 1, perturb=True)
    res = []
    for tile in (32, 33, 34):
        monkeypatch.setenv("GP_GEMM_TILE", str(tile))
        res.append(_step(cfg, case))
    _against_oracle(cfg, case, res[0])
    for r in res[1:]:
        assert np.array_equal(r["y"], res[0]["y"]) and np.array_equal(r["dx"], res[0]["dx"])
        assert r["loss"] == res[0]["loss"]
        for a, b in zip(r["grads"] + [r["head"]], res[0]["grads"] + [res[0]["head"]]):
            for k in a:
                assert np.array_equal(a[k], b[k]), k


# the block-per-row LayerNorm backward: one, two and a partial second chunk per
# thread; several rows per block (2052 rows: rows per wave 2, a short last block)
@pytest.mark.parametrize("d_model,heads,seq,batch,micro", [(1024, 16, 513, 4, 1), (1280, 20, 12, 2, 2),
                                                           (1792, 28, 20, 1, 1), (2048, 32, 8, 3, 3)])
def test_layernorm_backward_of_wide_rows(d_model, heads, seq, batch, micro):
    cfg = synth.PartitionConfig("wide", layers=1, d_model=d_model, d_ff=64, heads=heads, seq=seq, batch=batch,
                                micro=micro, dtype="f32", loss="mse")
    case = synth.make_case(cfg, 4, perturb=True)
    _against_oracle(cfg, case, _step(cfg, case))


# 16-row blocks with remainders, score rows of each length class (up to 128,
# 320 and 1024 columns) and their edges, head widths of one to four 16-column
# blocks with remainders; causal self-attention and cross-attention of another
# length (at least two keys: over one the query gradients are zero and have no relative error)
@pytest.mark.parametrize("heads,dh,seq,mem_seq", [(2, 64, 16, 0), (3, 4, 20, 0), (2, 20, 132, 0), (1, 48, 320, 0),
                                                  (1, 36, 324, 0), (2, 64, 17, 129), (2, 12, 128, 2),
                                                  (1, 40, 1024, 3)])
def test_f32_attention_lengths_and_widths(heads, dh, seq, mem_seq):
    dec = mem_seq > 0
    cfg = synth.PartitionConfig("attn", layers=1, d_model=heads * dh * (1 if heads * dh % 8 == 0 else 2), d_ff=64,
                                heads=heads * (1 if heads * dh % 8 == 0 else 2), seq=seq, mem_seq=mem_seq, batch=4,
                                micro=1, dtype="f32", kind="decoder" if dec else "encoder", loss="mse")
    case = synth.make_case(cfg, 6, perturb=True)
    _against_oracle(cfg, case, _step(cfg, case))


# Infinities and NaN stay on their side of the causal mask, also inside the 16-row
# block that shares its products: a token's bad input reaches no earlier output, and
# its bad gradient no later one.  Blocks within the 128 rows that are loaded ahead
# and beyond them, whole and cut off by the sequence's end, all head-width classes.
@pytest.mark.parametrize("dh,seq,at", [(64, 40, 21), (12, 40, 37), (32, 36, 32), (48, 204, 149), (64, 1024, 1018)])
def test_f32_causal_mask_holds_for_nonfinite_values(dh, seq, at):
    from paper_1811_06965_amd.runtime import Partition
    cfg = synth.PartitionConfig("mask", layers=1, d_model=2 * dh, d_ff=64, heads=2, seq=seq, mem_seq=8, batch=2, micro=1,
                                dtype="f32", kind="decoder")
    case = synth.make_case(cfg, 6, perturb=True)
    with Partition(cfg) as part:
        def step(x_at=None, dy_at=None):
            part.load_params(case["layers"], case["head"])  # a bad gradient leaves bad weights, at any rate
            inp = part.device_inputs(case)
            if x_at is not None:
                inp["x"][0, x_at, 3] = float("inf")
            if dy_at is not None:
                inp["dy"][0, dy_at, 5] = float("inf")
            out = part.step(inp["x"], inp["mem"], inp["dy"])
            return to_np(out["y"]), to_np(out["dx"])
        y, dx = step()
        y_bad, _ = step(x_at=at)
        _, dx_bad = step(dy_at=at)
    assert np.isfinite(y).all() and np.isfinite(dx).all()
    assert not np.isfinite(y_bad[0, at]).any()
    assert np.array_equal(y[0, :at], y_bad[0, :at]) and np.array_equal(y[1], y_bad[1])
    assert not np.isfinite(dx_bad[0, at]).any()
    assert np.array_equal(dx[0, at + 1:], dx_bad[0, at + 1:]) and np.array_equal(dx[1], dx_bad[1])
