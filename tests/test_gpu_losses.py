"""The loss heads at the edges of their kernels' ranges, against the fp64 oracle."""
import pytest

import synth
from parity import cosine, to_np

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _run(cfg, case, shift=0):
    from oracle import gpipe
    from paper_1811_06965_amd.runtime import Partition
    ref = gpipe.gpipe_step(cfg, case, cfg.micro)
    with Partition(cfg) as part:
        part.load_params(case["layers"], case["head"])
        inp = part.device_inputs(case)
        if shift:  # a target that starts `shift` elements past an aligned address
            buf = torch.empty(inp["dy"].numel() + shift, dtype=inp["dy"].dtype, device="cuda")
            view = buf[shift:].view_as(inp["dy"])
            view.copy_(inp["dy"])
            inp["dy"] = view
        losses = []
        for _ in range(2):
            out = part.step(inp["x"], inp["mem"], inp["dy"])
            losses.append(out["loss"])
        gl, gh = part.grads()
    assert losses[0] == losses[1]
    assert abs(losses[0] - ref["loss"]) <= 2e-2 * abs(ref["loss"])
    assert cosine(to_np(out["dx"]), ref["dx"]) >= 0.999
    return ref, gh


# one, two, four, eight and sixteen 2048-logit chunks per thread, their edges
# and the range beyond them
@pytest.mark.parametrize("vocab,clip", [(16, 0.0), (2048, 0.3), (2056, 0.0), (8192, 0.0), (8200, 0.3), (16392, 0.0),
                                        (32768, 0.0), (32776, 0.3)])
def test_xent_rows_by_vocabulary(vocab, clip):
    cfg = synth.PartitionConfig("v", layers=1, d_model=64, d_ff=128, heads=1, seq=32, batch=3, micro=3, dtype="bf16",
                                loss="xent_ls", vocab=vocab, label_smoothing=0.1, logit_clip=clip)
    case = synth.make_case(cfg, 2, perturb=True)
    case["labels"].reshape(-1)[:2] = (0, vocab - 1)
    ref, gh = _run(cfg, case)
    assert cosine(gh["bout"], ref["head_grads"]["bout"]) >= 0.999
    assert cosine(gh["wout"], ref["head_grads"]["wout"]) >= 0.999


@pytest.mark.parametrize("dtype,micro,shift", [("f32", 1, 1), ("f32", 4, 0), ("bf16", 2, 1), ("bf16", 4, 2)])
def test_mse_by_micro_batches_and_target_alignment(dtype, micro, shift):
    cfg = synth.PartitionConfig("m", layers=1, d_model=64, d_ff=128, heads=1, seq=32, batch=4, micro=micro,
                                dtype=dtype, loss="mse")
    _run(cfg, synth.make_case(cfg, 3, perturb=True), shift)
