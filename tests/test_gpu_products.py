"""Products and passes whose kernel depends on the shape, each against torch in float64 on the GPU from
the stage's own operands: the tile choices of the weight-gradient products, split activation products,
the fp32 tilings, and the two token sorts."""
import pytest

pytestmark = pytest.mark.gpu


def _stage(d, ffn, T, bf16=True, blocks=1, vocab=0, first=False, heads=2, hd=64, seed=3):
    """A middle (or first) stage of one sequence with random weights, in place on the GPU."""
    import torch
    from paper_2606_30634_amd.stage import Stage, make_shape
    st = Stage(make_shape(blocks, d, heads, heads, hd, ffn, vocab, first, False, False, T, 1, 1, bf16=bf16), "cuda:0")
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    st.view("flat.master").normal_(0.0, 0.02, generator=gen)
    st.resume(0, 0)
    dt = torch.bfloat16 if bf16 else torch.float32
    x = torch.randn(1, T, d, generator=gen, device="cuda:0").to(dt)
    dy = torch.randn(1, T, d, generator=gen, device="cuda:0").to(dt)
    return st, x, dy


def _err(a, b):
    return float((a.double() - b).norm() / b.norm())


def _worst(a, b):
    """Norm-wise error of the whole, and of the worst row and the worst column by themselves (an edge tile
    or a tile that was summed elsewhere is a share of the whole that its norm hides)."""
    e = a.double() - b
    return max([_err(a, b)] + [float((e.norm(dim=k) / b.norm(dim=k)).max()) for k in (0, 1)])


# fp32 sums of K terms of independent signs: the rounding of each partial sum (at most 2^-24 of it, in
# either direction) adds up to at most about sqrt(K) 2^-24 / 2 of the result's size norm-wise, measured over
# a row or column of 64 elements or more twice that at most.  Sums or partial sums of 16 bits (2^-9), or
# products of 11-bit mantissas (2^-12), are far above.
def _sum_tol(K):
    return 2.0 * K ** 0.5 * 2.0 ** -24


# d, ffn, T: dWdown [d, ffn] over K = T
@pytest.mark.parametrize("d,ffn,T", [
    (768, 3072, 2048),    # 144 tiles of 128 x 128 in 4 splits just past a round: 128 x 192 tiles
    (2048, 5632, 2048),   # 176 tiles of 256 x 256: one round of them
    (4096, 14336, 2048),  # 896 tiles of 256 x 256, 3.5 rounds: not deep enough to split the last 128
    (2560, 6912, 2048),   # 270 tiles of 256 x 256: the last 14 split over K
    (3200, 8704, 2048),   # whole 128 x 128 tiles, 256 x 256 ones partial at the edge
    (768, 3072, 2056),    # the widths of the first over a ragged K: 3 splits, one round
    (128, 10752, 4104),   # 84 tiles over a ragged K: 5 splits (6 would be 80 blocks each)
], ids=["wide", "one-round", "half-round", "tail", "edge", "ragged", "ragged-84"])
def test_weight_gradient_tiles(d, ffn, T):
    import torch
    st, x, dy = _stage(d, ffn, T)
    out = {}
    for rep in range(2):  # the second microbatch accumulates
        st.forward(0, 0, x_in=x, y_out=torch.empty_like(x))
        st.backward(0, dy=dy, microbatches_per_step=2)
        torch.cuda.synchronize()
        out[rep] = st.view("grad0.blk0.wdown").view(d, ffn).clone()
    z = st.view("act0.blk0.z").view(T, ffn)
    ref = torch.cat([dy[0].double().t() @ z[:, c:c + 2048].double() for c in range(0, ffn, 2048)], 1)
    st.close()
    tol = _sum_tol(T)  # the products of bf16 values are exact in fp32
    errs = _worst(out[0], ref), _worst(out[1], 2 * ref)
    assert max(errs) < tol, (errs, tol)


@pytest.mark.parametrize("d,ffn,T", [(256, 4096, 300), (64, 2112, 17), (768, 3072, 999)], ids=["6-tiles", "1-tile", "48-tiles"])
def test_split_activation_product(d, ffn, T):
    # y = h + z Wd^T, K = ffn split over the idle blocks, summed in fp32 and rounded to bf16 once: the sums'
    # own error moves few roundings (its size against the 2^-8 between neighbours, and four times that for
    # the elements where h and the product cancel); a second rounding anywhere would move half of them
    import torch
    st, x, dy = _stage(d, ffn, T)
    y = torch.empty_like(x)
    st.forward(0, 0, x_in=x, y_out=y)
    torch.cuda.synchronize()
    z, h = st.view("act0.blk0.z").double().view(T, ffn), st.view("act0.blk0.h").double().view(T, d)
    ref = h + z @ st.view("w0.blk0.wdown").double().view(d, ffn).t()
    e = _worst(y[0], ref)
    moved = float((y[0] != ref.to(torch.bfloat16)).double().mean())
    st.close()
    assert e < 2.0 ** -8 and moved < 4 * _sum_tol(ffn) / 2.0 ** -8, (e, moved)


def test_swiglu_backward_of_partial_tiles():
    # dgate and dup of a ragged product as the gate | up weight gradient shows them: one-hot rows of n2 and
    # dy = e_0, so that dWgu[r, t] = dgu[t, r] and dz = row 0 of Wdown, exact in bf16.  In fp32 with an
    # exponential of 1 ulp the formula's eight roundings stay below 2^-20.8 of the result, which moves at
    # most 2^-20.8 / 2^-8 = 1.4e-4 of its bf16 roundings.
    import torch
    d, ffn, T = 64, 8192, 63
    st, x, dy = _stage(d, ffn, T)
    st.forward(0, 0, x_in=x, y_out=torch.empty_like(x))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(11)
    gu = st.view("act0.blk0.gu").view(T, 2 * ffn)
    gu[:, :ffn] = torch.empty(T, ffn, device="cuda:0").uniform_(-80.0, -64.0, generator=gen)
    gu[:, ffn:] = torch.empty(T, ffn, device="cuda:0").uniform_(1.0, 2.0, generator=gen)
    st.view("act0.blk0.n2").view(T, d).copy_(torch.eye(d, device="cuda:0")[:T])
    dy.zero_()
    dy[..., 0] = 1.0
    w = st.view("w0.blk0.wdown").view(d, ffn)
    w[0] = torch.empty(ffn, device="cuda:0").uniform_(1.0, 2.0, generator=gen)
    st.backward(0, dy=dy)
    torch.cuda.synchronize()
    a, b, dz = gu[:, :ffn].double(), gu[:, ffn:].double(), w[0].double()
    s = torch.sigmoid(a)
    moved = 0
    for name, ref in (("wgate", dz * b * s * (1.0 + a * (1.0 - s))), ("wup", dz * a * s)):
        got = st.view(f"grad0.blk0.{name}").view(ffn, d)[:, :T].t()
        ref16 = ref.float().to(torch.bfloat16).float()
        moved += int((got != ref16).sum())
        assert float(((got - ref16).abs() / ref16.abs()).max()) <= 2.0 ** -7  # the neighbouring value at most
    st.close()
    assert moved < 1.4e-4 * 2 * T * ffn, moved


def test_gate_and_up_rows_past_a_tile_offset():
    # d_ffn x d_model above 2^30: the up rows are out of reach of the gate rows' tile offsets, so the
    # product runs first and the SwiGLU after it
    import torch
    d, ffn, T = 4096, 262208, 128
    st, x, dy = _stage(d, ffn, T)
    st.forward(0, 0, x_in=x, y_out=torch.empty_like(x))
    torch.cuda.synchronize()
    n2 = st.view("act0.blk0.n2").view(T, d).double()
    cols = torch.tensor([0, 1, 63, 64, 131071, ffn - 65, ffn - 1], device="cuda:0")
    g = n2 @ st.view("w0.blk0.wgate").view(ffn, d)[cols].double().t()
    u = n2 @ st.view("w0.blk0.wup").view(ffn, d)[cols].double().t()
    gu, z = st.view("act0.blk0.gu").view(T, 2 * ffn), st.view("act0.blk0.z").view(T, ffn)
    errs = (_err(gu[:, cols], g), _err(gu[:, ffn + cols], u), _err(z[:, cols], torch.nn.functional.silu(g) * u))
    st.close()
    assert max(errs) < 2.0 ** -8, errs


@pytest.mark.parametrize("d,ffn,T", [(64, 64, 31), (128, 512, 1000), (512, 2048, 2100)], ids=["32x32", "64x64", "128x128"])
def test_fp32_tilings(d, ffn, T):
    # gate | up = n2 Wgu^T (the SwiGLU in its epilogue): fp32 sums of K = d products; z from both, with
    # half a dozen roundings of its own
    import torch
    st, x, dy = _stage(d, ffn, T, bf16=False, heads=2, hd=32)
    st.forward(0, 0, x_in=x, y_out=torch.empty_like(x))
    torch.cuda.synchronize()
    n2 = st.view("act0.blk0.n2").double().view(T, d)
    g = n2 @ st.view("w0.blk0.wgate").double().view(ffn, d).t()
    u = n2 @ st.view("w0.blk0.wup").double().view(ffn, d).t()
    gu = st.view("act0.blk0.gu").view(T, 2 * ffn)
    z = st.view("act0.blk0.z").view(T, ffn)
    errs = (_worst(gu[:, :ffn], g), _worst(gu[:, ffn:], u), _worst(z, torch.nn.functional.silu(g) * u))
    st.close()
    tol = _sum_tol(d)
    assert max(errs[:2]) < tol and errs[2] < 2 * tol + 6 * 2.0 ** -24, (errs, tol)


@pytest.mark.parametrize("n", [1, 2, 65, 128, 129, 1000, 4095, 4096, 4097, 8191, 8192, 8193])
def test_token_sort_lengths(n):
    # a first stage without blocks: the embedding's gradient is the scatter of dy itself.  Ids and
    # counts exact; each row the fp32 sum of its positions (50 ids, so up to n / 10 of them).
    import torch
    st, x, dy = _stage(64, 64, n, blocks=0, vocab=50, first=True)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n)
    tok = torch.randint(0, 50, (1, n), generator=gen, device="cuda:0", dtype=torch.int32)
    st.forward(0, 0, tokens=tok, y_out=torch.empty_like(x))
    st.backward(0, dy=dy)
    torch.cuda.synchronize()
    ids, counts = st.embed_indices(0)
    rid, rc = torch.unique(tok.cpu(), return_counts=True)
    assert list(ids) == rid.tolist() and list(counts) == rc.tolist()
    ref = torch.zeros(50, 64, dtype=torch.float64, device="cuda:0").index_add_(0, tok[0].long(), dy[0].double())
    e = _err(st.view("grad0.embed").view(50, 64), ref)
    st.close()
    assert e < n * 2.0 ** -24 + 1e-7, e
