"""The bits of a step's outputs.  A result of the library does not depend on the
kernel form that a size takes: where a wider or grouped form took a simpler one's
place, it adds in the simpler one's order.  tests/golden/step_bits.json holds
digests of each output as the simpler forms gave them (a wave per row in LayerNorm
and cross-entropy, one launch and its split-K reduce per weight gradient, the
register-staged GEMM for reductions that are no multiple of 64)."""
import hashlib
import json
import os

import numpy as np
import pytest

import synth
from parity import to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "step_bits.json")


def _cfg(name, **kw):
    return synth.PartitionConfig(name, **dict(dict(layers=2, d_model=64, d_ff=128, heads=1, seq=32, batch=3, micro=3,
                                                   dtype="bf16"), **kw))


CASES = [
    # the update: weights in whole tiles, biases and gains; SGD and RMSProp in both types
    _cfg("sgd", d_model=128, heads=2, d_ff=256),
    _cfg("rmsprop", d_model=128, heads=2, d_ff=256, loss="mse", optimizer="rmsprop"),
    _cfg("sgd_f32", d_model=72, heads=6, d_ff=200, seq=20, dtype="f32"),
    _cfg("rmsprop_f32", d_model=72, heads=6, d_ff=200, seq=20, dtype="f32", loss="mse", optimizer="rmsprop"),
    # LayerNorm backward of wide rows, a block per row: one and two chunks per
    # thread, the second one for some of the waves only; odd row counts
    _cfg("ln1024", d_model=1024, heads=16, batch=6),
    _cfg("ln2048", layers=1, d_model=2048, heads=32, batch=6),
    _cfg("ln1280_f32", layers=1, d_model=1280, heads=20, seq=12, batch=2, micro=2, dtype="f32", loss="mse"),
    _cfg("ln1536", layers=1, d_model=1536, heads=24, batch=2, micro=2),
    _cfg("ln1792_f32", layers=1, d_model=1792, heads=28, seq=20, batch=1, micro=1, dtype="f32", loss="mse"),
    # several rows per run of the parameter sums, the last run and block cut off
    _cfg("ln1024_rows", layers=1, d_model=1024, heads=16, d_ff=64, seq=513, batch=4, micro=1, dtype="f32", loss="mse"),
    _cfg("ln2048_rows", layers=1, d_model=2048, heads=32, d_ff=64, seq=1023, batch=4, micro=1, dtype="f32", loss="mse"),
    # its input still in split-K partial sums
    _cfg("ln1024_partials", d_model=1024, heads=16, d_ff=8192, seq=128, batch=2, micro=2),
] + [
    # cross-entropy rows: register chunks of one to sixteen times 2048 logits and their edges
    _cfg("xent%d" % v, layers=1, batch=6, loss="xent_ls", vocab=v, label_smoothing=0.1, logit_clip=c)
    for v, c in ((64, 0.0), (264, 0.3), (2048, 0.3), (2112, 0.0), (4160, 0.3), (8256, 0.0), (16448, 0.0), (32000, 0.0),
                 (32768, 0.3))
] + [
    # weight gradients whose single launches split the reduction over rows, accumulated over pairs
    _cfg("dw_split", d_model=1024, heads=16, d_ff=1024, seq=256, batch=32, micro=4),
    _cfg("dw_split_odd", layers=1, d_model=512, heads=8, d_ff=512, seq=256, batch=24, micro=3),
    _cfg("dw_split_decoder", layers=1, d_model=512, heads=8, d_ff=512, seq=256, mem_seq=128, batch=32, micro=2,
         kind="decoder"),
    _cfg("dw_split768", layers=1, d_model=768, heads=12, d_ff=768, seq=192, batch=24, micro=2),
    # reductions that are no multiple of 64: over widths, over rows, over both; split and not
    _cfg("rag", d_model=320, heads=5, d_ff=1000, seq=96, batch=15, micro=5, loss="mse"),
    _cfg("rag_wide", d_model=512, heads=8, d_ff=2056, batch=2, micro=2),
    _cfg("rag_rows", layers=1, d_model=256, heads=4, d_ff=520, seq=96, batch=21, micro=1),
    _cfg("rag_decoder", d_model=256, heads=4, d_ff=1000, seq=96, mem_seq=32, batch=21, micro=1, kind="decoder",
         loss="xent_ls", vocab=1000, label_smoothing=0.1),
    _cfg("rag_tiles", layers=1, d_model=1024, heads=16, d_ff=8200, seq=224, batch=3, micro=1),
    _cfg("rag_head", layers=1, loss="xent_ls", vocab=8200, label_smoothing=0.1, logit_clip=0.3),
    _cfg("rag_m3", layers=1, d_model=128, heads=2, d_ff=264, seq=224, batch=9, micro=3),
]


def digests(cfg):
    from paper_1811_06965_amd.runtime import Partition
    case = synth.make_case(cfg, 9, perturb=True)
    with Partition(cfg) as part:
        part.load_params(case["layers"], case["head"])
        inp = part.device_inputs(case)
        for _ in range(2):  # the second step accumulates afresh, on updated weights
            out = part.step(inp["x"], inp["mem"], inp["dy"], lr=1e-2 if cfg.optimizer == "sgd" else 1e-3)
        gl, gh = part.grads()
        pl, ph = part.params()
    res = {k: to_np(out[k]) for k in ("y", "dx", "dmem") if out[k] is not None}
    if out["loss"] is not None:
        res["loss"] = np.float32([out["loss"]])
    for l, g in enumerate(gl + [gh]):
        res.update({f"{l}.{k}": v for k, v in g.items()})
    for l, w in enumerate(pl + [ph]):
        res.update({f"{l}.{k}.updated": v for k, v in w.items()})
    # + 0: a zero has one sign
    return {k: hashlib.sha256(np.ascontiguousarray(v + v.dtype.type(0)).tobytes()).hexdigest()[:12]
            for k, v in res.items()}


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_outputs_keep_their_bits(cfg):
    with open(GOLDEN) as f:
        want = json.load(f)[cfg.name]
    got = digests(cfg)
    assert sorted(got) == sorted(want)
    assert [k for k in want if got[k] != want[k]] == []
