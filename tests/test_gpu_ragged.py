"""Stages whose token count, widths or vocabulary are no multiple of any tile: every product runs
with partial tiles, partial k-slices or padded rows.  Forward, backward of two microbatches (the
second accumulates) against the float64 oracle, bf16 at the repository's 2e-2 bar, fp32 at 1e-4,
norm-wise per tensor."""
import numpy as np
import pytest

import datagen
import oracle
from gpu_common import log, rel, shape_of, to_device

pytestmark = pytest.mark.gpu

# name: (dtype, role, blocks, d, heads, kv, hd, ffn, vocab, seq, mb)
CASES = {
    # T = 17 < one tile; the widths are single k-slices; K = 96 (a half slice) in the products over
    # the packed heads
    "tiny": ("bf16", "middle", 1, 64, 1, 1, 32, 64, 0, 17, 1),
    # T = 129: one row into the second tile, one k past the second slice; d_ffn = 192 (half a tile)
    "129-tokens": ("bf16", "middle", 2, 128, 2, 1, 64, 192, 0, 43, 3),
    # T = 127, head dim 128 (delta and RoPE in kernels of their own), d_model 192
    "127-tokens": ("bf16", "middle", 1, 192, 2, 2, 128, 320, 0, 127, 1),
    # split-K over a ragged K: T = 2057 tokens in the weight-gradient products
    "2057-tokens": ("bf16", "first", 1, 128, 2, 2, 64, 320, 333, 2057, 1),
    "vocab-129": ("bf16", "last", 1, 128, 2, 2, 64, 192, 129, 33, 3),
    "vocab-1003": ("bf16", "last", 1, 192, 3, 1, 64, 256, 1003, 128, 1),
    # vocabulary a multiple of 8 but not of a slice; K = 2056 deep activation-gradient product
    "vocab-2056": ("bf16", "last", 1, 64, 1, 1, 64, 64, 2056, 65, 2),
    "f32-vocab-1003": ("f32", "last", 1, 128, 2, 2, 64, 192, 1003, 61, 3),
    "f32-129-tokens": ("f32", "middle", 1, 192, 6, 2, 32, 320, 0, 43, 3),
    "f32-head-128": ("f32", "middle", 1, 128, 2, 1, 128, 64, 0, 67, 1),
    # dk/dv items split 5 and 2 ways over their queries
    "split-hd64": ("bf16", "middle", 1, 256, 4, 1, 64, 64, 0, 650, 1),
    "split-hd128": ("bf16", "middle", 1, 256, 4, 2, 128, 64, 0, 515, 1),
    # the same over several sequences (the batch term of the partial sums' layout)
    "split-hd64-3-sequences": ("bf16", "middle", 1, 256, 4, 1, 64, 64, 0, 650, 3),
    "split-hd128-2-sequences": ("bf16", "middle", 1, 256, 4, 2, 128, 64, 0, 515, 2),
    # the last key block has one tile of queries for two shares: one share adds nothing
    "split-empty-share": ("bf16", "middle", 1, 128, 1, 1, 128, 64, 0, 1025, 1),
    # 11 norms: more than one batch of column sums
    "f32-five-blocks": ("f32", "last", 5, 64, 2, 2, 32, 64, 97, 33, 2),
}


@pytest.mark.parametrize("name", list(CASES))
def test_ragged_stage_against_oracle(name):
    import torch
    from paper_2606_30634_amd.stage import Stage
    dt, role, blocks, d, heads, kv, hd, ffn, vocab, seq, mb = CASES[name]
    w = datagen.SMALL.with_(name=name, dtype=dt, n_blocks=blocks, d_model=d, n_heads=heads, n_kv_heads=kv,
                            head_dim=hd, d_ffn=ffn, vocab=vocab, first_stage=role == "first",
                            last_stage=role == "last", tie_embedding=False, seq_len=seq, micro_batch=mb,
                            microbatches_per_step=2, max_inflight=1)
    log(f"ragged stage {name}")
    dev = torch.device("cuda:0")
    st = Stage(shape_of(w), "cuda:0")
    p0 = datagen.init_params(w)
    st.load_master(p0)
    inputs = [datagen.step_inputs(w, 0, i) for i in range(2)]
    ys, losses, dxs = [], [], []
    for inp in inputs:
        t = to_device(inp, w, dev)
        loss = torch.zeros(1, device=dev)
        y = None if role == "last" else torch.empty_like(t["dy"])
        dx = None if role == "first" else torch.empty_like(t["x_in"])
        st.forward(0, 0, tokens=t.get("tokens"), x_in=t.get("x_in"), targets=t.get("targets"), y_out=y, loss=loss)
        st.backward(0, dy=t.get("dy"), dx_out=dx, microbatches_per_step=2)
        ys.append(y)
        dxs.append(dx)
        losses.append(float(loss.item()))
    torch.cuda.synchronize()
    gref, outs = {}, []
    for inp in inputs:
        o, saves = oracle.model.stage_forward(p0, inp, w)
        g, o["dx_in"] = oracle.model.stage_backward(p0, inp, saves, w, loss_scale=0.5)
        outs.append(o)
        gref = {n: gref.get(n, 0.0) + v for n, v in g.items()}
    errs = {f"grad.{n}": rel(st.view(f"grad0.{n}").double().cpu().numpy().reshape(p0[n].shape), gref[n]) for n in p0}
    for i, o in enumerate(outs):
        if role == "last":
            errs[f"loss{i}"] = abs(losses[i] - float(o["loss"])) / float(o["loss"])
        else:
            errs[f"y{i}"] = rel(ys[i].double().cpu().numpy().reshape(o["y"].shape), o["y"])
        if role != "first":
            errs[f"dx{i}"] = rel(dxs[i].double().cpu().numpy().reshape(o["dx_in"].shape), o["dx_in"])
    st.close()
    worst = max(errs, key=errs.get)
    log(f"{name}: worst {worst} {errs[worst]:.2e}")
    tol = 2e-2 if dt == "bf16" else 1e-4
    assert errs[worst] < tol, {k: v for k, v in errs.items() if not v < tol}


def test_large_ragged_tiles_against_float64():
    # the 256 x 256 tiles with partial rows and columns (17 x 32 tiles of T = 4099, 2 d_ffn = 8064 at
    # K = 1536): the gate/up product and its SwiGLU from the stage's own n2 and weights.  One
    # rounding to bf16 of an fp32 value: at most 2^-9 per element, checked norm-wise at twice that.
    import torch
    from paper_2606_30634_amd.stage import Stage
    w = datagen.SMALL.with_(name="large-ragged", dtype="bf16", n_blocks=1, d_model=1536, n_heads=12, n_kv_heads=4,
                            head_dim=128, d_ffn=4032, vocab=0, first_stage=False, last_stage=False, seq_len=4099,
                            micro_batch=1, max_inflight=1)
    log("large ragged tiles")
    dev = torch.device("cuda:0")
    st = Stage(shape_of(w), "cuda:0")
    st.load_master(datagen.init_params(w))
    t = to_device(datagen.step_inputs(w, 0), w, dev)
    st.forward(0, 0, x_in=t["x_in"], y_out=torch.empty_like(t["x_in"]))
    torch.cuda.synchronize()
    n2 = st.view("act0.blk0.n2").double().view(-1, w.d_model)
    gate = n2 @ st.view("w0.blk0.wgate").double().view(-1, w.d_model).t()
    up = n2 @ st.view("w0.blk0.wup").double().view(-1, w.d_model).t()
    gu = st.view("act0.blk0.gu").double().view(-1, 2 * w.d_ffn)
    z = st.view("act0.blk0.z").double().view(-1, w.d_ffn)
    err = lambda a, b: float((a - b).norm() / b.norm())  # noqa: E731
    errs = dict(gate=err(gu[:, :w.d_ffn], gate), up=err(gu[:, w.d_ffn:], up),
                z=err(z, torch.nn.functional.silu(gate) * up))
    # the last rows and columns by themselves: they sit in the partial tiles
    errs.update(rows=err(z[-3:], (torch.nn.functional.silu(gate) * up)[-3:]), cols=err(gu[:, -64:], up[:, -64:]))
    st.close()
    log(str(errs))
    assert max(errs.values()) < 2.0 ** -8, errs
