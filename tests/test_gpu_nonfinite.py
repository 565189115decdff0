"""Infinities and NaNs stay where the computation puts them: a masked or zero-weight element reaches
nothing, whatever it holds."""
import pytest

pytestmark = pytest.mark.gpu


def _stage(hd, bf16, S, heads=2, kv=1, d=64, ffn=64, vocab=0):
    import torch
    from paper_2606_30634_amd.stage import Stage, make_shape
    st = Stage(make_shape(1 if not vocab else 0, d, heads, kv, hd, ffn, vocab, False, vocab > 0, False, S, 1, 1, bf16=bf16),
               "cuda:0")
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    st.view("flat.master").normal_(0.0, 0.1, generator=gen)
    st.resume(0, 0)
    dt = torch.bfloat16 if bf16 else torch.float32
    x = torch.randn(1, S, d, generator=gen, device="cuda:0").to(dt)
    dy = torch.randn(1, S, d, generator=gen, device="cuda:0").to(dt)
    return st, x, dy


def _step(st, x, dy):
    import torch
    y, dx = torch.empty_like(x), torch.empty_like(x)
    st.forward(0, 0, x_in=x, y_out=y)
    st.backward(0, dy=dy, dx_out=dx)
    torch.cuda.synchronize()
    return y[0].double(), dx[0].double()


# The head dimensions of the kernels that multiply fp32 weights; S ends inside a tile of 32 rows.
@pytest.mark.parametrize("bf16,hd", [(False, 32), (False, 64), (False, 128), (True, 32)])
@pytest.mark.parametrize("j", [40, 74])
def test_attention_is_causal_for_nonfinite_rows(bf16, hd, j):
    # a token with an infinity reaches the outputs from its own position on, its output gradient the input
    # gradients up to it; the other rows differ from a clean run by the order of fp32 sums at most
    import torch
    st, x, dy = _stage(hd, bf16, 75)
    y0, dx0 = _step(st, x, dy)
    bad = x.clone()
    bad[0, j, 3] = float("inf")
    y1, _ = _step(st, bad, dy)
    bad = dy.clone()
    bad[0, j, 3] = float("inf")
    _, dx1 = _step(st, x, bad)
    st.close()
    assert not bool(torch.isfinite(y1[j]).all()) and not bool(torch.isfinite(dx1[j]).all())
    tol = 2.0 ** -8 if bf16 else 1e-5
    for a, b in ((y1[:j], y0[:j]), (dx1[j + 1:], dx0[j + 1:])):
        assert a.numel() == 0 or float((a - b).norm() / b.norm()) < tol


def test_attention_scores_of_minus_infinity():
    # keys 32..63 score below every float against any query (the product overflows): weight 0, also
    # for the queries whose tile of 32 keys holds nothing else
    import torch
    hd, S = 32, 130
    st, x, dy = _stage(hd, False, S, heads=1)
    w = {n: st.view(f"w0.blk0.{n}") for n in ("wq", "wk")}
    for v in w.values():
        v.zero_()
    w["wq"].view(hd, 64)[15, 0] = 1e20  # the slowest pair of the rotary embedding: cos about 1
    w["wk"].view(hd, 64)[15, 1] = -1e20
    st.view("w0.blk0.attn_norm").fill_(1.0)
    x.normal_()
    x[..., 0] = 1.0
    x[..., 1] = 0.0
    x[:, 32:64, 1] = 1.0
    st.forward(0, 0, x_in=x, y_out=torch.empty_like(x))
    torch.cuda.synchronize()
    v = st.view("act0.blk0.qkv").view(S, 3 * hd)[:, 2 * hd:].double()
    p = torch.ones(S, S, device="cuda:0", dtype=torch.float64).tril()
    p[:, 32:64] = 0.0
    ref = (p / p.sum(1, keepdim=True)) @ v
    o = st.view("act0.blk0.o").view(S, hd).double()
    st.close()
    assert float((o - ref).norm() / ref.norm()) < 1e-6


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("vocab", [7, 1003, 1004])
def test_cross_entropy_with_logits_of_minus_infinity(bf16, vocab):
    # the first four logits of every row overflow to -inf: probability 0, and a finite loss
    import torch
    S, d = 33, 64
    st, x, _ = _stage(32, bf16, S, vocab=vocab)
    st.view("w0.final_norm").fill_(1.0)
    st.view("w0.head").view(vocab, d)[:4] = -3e38
    x = x.abs() + 0.5
    tg = torch.arange(S, device="cuda:0", dtype=torch.int32).view(1, S) % (vocab - 4) + 4
    loss, dx = torch.zeros(1, device="cuda:0"), torch.empty_like(x)
    st.forward(0, 0, x_in=x, targets=tg, loss=loss)
    st.backward(0, dx_out=dx)
    torch.cuda.synchronize()
    z = st.view("act0.logits").view(S, vocab).double()
    assert bool(torch.isinf(z[:, :4]).all())
    ref = float(torch.nn.functional.cross_entropy(z, tg[0].long()))
    got = float(loss)
    fin = bool(torch.isfinite(dx).all())
    st.close()
    assert abs(got - ref) < 1e-5 * ref and fin, (got, ref, fin)
