"""``specdec_step_noalloc`` beyond the small steps (more than 256 logit rows of at
most 16 KB): verification in one launch on the library's completion counts,
eager and replayed from a HIP graph, against ``specdec_step`` bit for bit."""
import numpy as np
import pytest
import torch

from paper_2510_22876_amd import workloads as wl
from tests.gpu_util import alloc_outputs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", ["oop", "inplace"])
@pytest.mark.parametrize("dtype,V", [("bf16", 8192), ("f32", 4096), ("f16", 777)])
def test_large_batches_verify_in_one_launch(variant, dtype, V):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2510_22876_amd import specdec as sd
    sd.timing_enable(False)
    w = wl.WORKLOADS["vicuna7b"].scaled(B=70, V=V, L=1, H=2, D=16, logit_dtype=dtype, prompt=("uniform", 16, 120))
    n, W_in, pad_in, cap = wl.initial_geometry(w, 3)
    src0 = wl.make_kv(w, pad_in, W_in, cap, 3, device="cuda")
    pad = torch.as_tensor(np.asarray(pad_in, np.int32), device="cuda")
    inputs = [wl.logits_and_drafts(w, 3, t, device="cuda")[:2] for t in range(3)]
    lg, dr, src = inputs[0][0].clone(), inputs[0][1].clone(), src0.clone()
    dst = src if variant == "inplace" else torch.zeros_like(src)
    o = alloc_outputs(w.B, w.k, w.V, W_in + w.k + 1)

    def step():
        sd.specdec_step_noalloc(lg, dr, pad, W_in, src, dst, o.tokens, o.n_acc, o.bonus, o.pad_out, o.w_new, o.pos,
                                o.mask, o.dev_status)

    def check(t, what):
        say(f"noalloc large {what} {variant} {dtype} inputs={t}")
        e = alloc_outputs(w.B, w.k, w.V, W_in + w.k + 1)
        s = src0.clone()
        d = s if variant == "inplace" else torch.zeros_like(s)
        sd.specdec_step(inputs[t][0], inputs[t][1], pad, W_in, s, d, e.tokens, e.n_acc, e.bonus, e.pad_out, e.w_new,
                        e.pos, e.mask, e.workspace, e.dev_status)
        torch.cuda.synchronize()
        W = int(e.w_new)
        for name in ("tokens", "n_acc", "bonus", "pad_out", "w_new", "dev_status"):
            assert torch.equal(getattr(o, name), getattr(e, name)), (t, name)
        for name in ("pos", "mask"):
            assert torch.equal(getattr(o, name)[:, :W + w.k + 1], getattr(e, name)[:, :W + w.k + 1]), (t, name)
        assert torch.equal(dst[..., :W, :].view(torch.int16), d[..., :W, :].view(torch.int16)), (t, "kv")

    def load(t):
        lg.copy_(inputs[t][0])
        dr.copy_(inputs[t][1])
        src.copy_(src0)
        torch.cuda.synchronize()

    for t in (0, 1, 2, 0):
        load(t)
        step()
        torch.cuda.synchronize()
        check(t, "eager")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for t in (1, 2, 1, 0):
        load(t)
        g.replay()
        torch.cuda.synchronize()
        check(t, "replay")
