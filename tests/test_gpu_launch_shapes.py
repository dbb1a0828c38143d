"""Kernels at the sizes where a variant begins, ends or leaves a remainder."""
import numpy as np
import pytest
import torch

import synth_inputs as Y
from oracle import mlp as OM

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_02550_amd as S
    from paper_2503_02550_amd import params as P
    from paper_2503_02550_amd.session import Session, mlp_shape
    from gpu_util import DEV, f32, up, assert_f32_close, stream_beside


def _bf16(gen, *shape):
    return torch.randn(shape, device=DEV, generator=gen).to(torch.bfloat16)


@pytest.mark.parametrize("batch,hidden", [(1, 8), (16, 512), (16, 528), (32, 1024), (32, 1056), (33, 2048), (512, 1024), (520, 1024), (2048, 1024), (2080, 1024)])
def test_last_block_is_found_whatever_the_grid(batch, hidden):
    """A launch is reported done by its last block; grids at the edges of the counting tree must all be, twice in a row (the
    counters are re-armed), with every kernel counted.  Blocks of the first product: 1, 32, 33, 128, 132, 384 (tiles of
    16 x 16), 512, 544, 2048, 2080 (32 x 32); of the second 1 to 65.  Products of fp32 values: the bound of the other fp32 tests, 1e-4 of the largest value."""
    shape = mlp_shape(8, hidden, 32, batch)
    p = Y.mlp_params(3, 8, hidden, 32)
    with Session() as s:
        m = s.register_inference(shape, P.pack(shape, p))
        for turn in range(2):
            x = Y.activations(10 + turn, batch, 8)
            X, out = f32(x), torch.zeros((batch, 32), device=DEV)
            torch.cuda.synchronize()
            s.wait(s.submit_offline(m, X, out, batch), 10.0)
            y, _ = OM.mlp_forward({k: v.astype(np.float64) for k, v in p.items()}, x)
            assert_f32_close(up(out), y, f"turn {turn}")
        assert s.stats().kernels_run == 4


@pytest.mark.parametrize("batch,hidden", [(8, 32), (64, 1056)])
def test_training_kernels_are_counted(batch, hidden):
    """The count of training kernels that ran, as the kernels report it, is the number launched."""
    shape = mlp_shape(16, hidden, 16, batch)
    with Session() as s:
        s.register_training(shape, P.pack(shape, Y.mlp_params(4, 16, hidden, 16)))
        n = 0
        while S.sif_train_op_name(s.ctx, s.train["handle"], n) is not None:
            n += 1
        x, t = Y.mlp_batch(0, 0, batch, 16, 16)
        X, T = f32(x), f32(t)
        torch.cuda.synchronize()
        for k in range(1, 4):
            s.step(X, T)
            s.sync()
            assert s.stats().train_kernels == k * n
            assert s.stats().steps == k


@pytest.mark.parametrize("bubble", [False, True])
@pytest.mark.parametrize("d_in,hidden,d_out,batch", [(5, 7, 3, 1), (16, 17, 33, 15), (70, 530, 517, 600), (640, 512, 516, 512)])
def test_mlp_step_of_shared_launches_matches_the_oracle(d_in, hidden, d_out, batch, bubble):
    """The step with its update in the last gradient's launch (no bubble) and as a launch of its own (bubble), at sizes
    of one tile, of remainders and of the wide tile; three steps, tolerances of the other fp32 model tests."""
    shape = mlp_shape(d_in, hidden, d_out, batch)
    p0 = Y.mlp_params(6, d_in, hidden, d_out)
    p0["b1"], p0["b2"] = p0["b1"] + 0.01, p0["b2"] - 0.02
    ref = {k: v.astype(np.float64) for k, v in p0.items()}
    with Session() as s:
        s.register_training(shape, P.pack(shape, p0), par_mode=S.SIF_PAR_FIXED if bubble else S.SIF_PAR_NONE, lr=0.05,
                            fixed_bubble_ns=50_000 if bubble else 0)
        loss = torch.zeros(1, device=DEV)
        for step in range(3):
            x, t = Y.mlp_batch(1, step, batch, d_in, d_out)
            X, T = f32(x), f32(t)
            torch.cuda.synchronize()
            s.step(X, T, loss)
            s.sync()
            rl, ref, rg = OM.mlp_train_step(ref, x, t, 0.05)
            assert abs(loss.item() - rl) <= 1e-4 * abs(rl), step
            got_g = P.unpack(shape, up(s.train_tensor("grads", dtype=torch.float32)))
            got_p = P.unpack(shape, up(s.train["master"]))
            for k in ref:
                assert_f32_close(got_g[k], rg[k], f"step {step} grad {k}")
                assert_f32_close(got_p[k], ref[k], f"step {step} param {k}", 1e-5)


@pytest.mark.parametrize("k_contig_a", [True, False])
@pytest.mark.parametrize("k_contig_b", [True, False])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (16, 16, 16), (17, 33, 65), (31, 50, 3), (8, 256, 256), (512, 512, 64), (515, 517, 68), (513, 1030, 130)])
def test_gemm_f32_tiles_and_remainders(m, n, k, k_contig_a, k_contig_b):
    """Both tile sizes, with 16-byte loads (K contiguous and a multiple of 4) and without, at remainders of M, N and K.
    Bound: an fp32 sum of k products in any order errs by at most (k + 4) 2^-24 times the sum of their magnitudes."""
    rng = np.random.default_rng(m * 7 + n * 3 + k)
    a, b = rng.standard_normal((m, k)).astype(np.float32), rng.standard_normal((n, k)).astype(np.float32)
    A, Bt = f32(a if k_contig_a else a.T), f32(b if k_contig_b else b.T)
    c = torch.full((m, n), float("nan"), device=DEV)
    S.sif_k_gemm_f32(A, *((k, 1) if k_contig_a else (1, m)), Bt, *((1, k) if k_contig_b else (n, 1)), c, n, m, n, k)
    torch.cuda.synchronize()
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    bound = (k + 4) * 2.0 ** -24 * (np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64).T)
    assert np.all(np.abs(up(c) - ref) <= bound)


@pytest.mark.parametrize("al", [0, 1])
@pytest.mark.parametrize("bl", [0, 1])
@pytest.mark.parametrize("m,n,k", [(1, 8, 8), (31, 72, 64), (33, 64, 136), (64, 64, 256), (65, 200, 520), (300, 3080, 320), (1000, 768, 200),
                                   (1000, 2304, 456), (2008, 1536, 520), (4100, 768, 328), (2056, 2048, 1032), (8192, 776, 72), (4096, 3072, 512)])
def test_gemm_bf16_picks_tiles_that_give_the_bits_of_the_128_ones(m, n, k, al, bl):
    """Products of a few rows to ones that fill the chip: whichever kernel the launcher takes (32x64 with one K step, fetching
    32x32 and 64x64, 128x128 with one and two per CU, 256x128, 256x256; the tests below have the others and name them), at ragged M, N and K, the
    result has the bits of the 128x128 tiles and is the product.  Bound:
    one rounding to bf16 (2^-9 of the value) and the fp32 sum of k exact products ((k + 4) 2^-24 of their magnitudes)."""
    gen = torch.Generator(device=DEV).manual_seed(m + 3 * n + 5 * k + al + 2 * bl)
    mp, np_ = (m + 7) // 8 * 8, n
    a, b = torch.zeros((mp, k), device=DEV, dtype=torch.bfloat16), _bf16(gen, n, k)
    a[:m] = _bf16(gen, m, k)
    A, Bt = (a if al == 0 else a.t().contiguous()), (b if bl == 0 else b.t().contiguous())
    out = [torch.full((m, n), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(2)]
    torch.cuda.synchronize()
    for c, tile in zip(out, (0, 128)):
        S.sif_k_gemm_bf16(A, Bt, c, m, n, k, A.shape[1], Bt.shape[1], n, a_layout=al, b_layout=bl, tile=tile)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
    ref = a[:m].double() @ b.double().t()
    bound = 2.0 ** -8 * ref.abs() + (k + 4) * 2.0 ** -24 * (a[:m].double().abs() @ b.double().abs().t())
    assert bool(((out[0].double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("d,da,f,k,apart", [(1920, 1920, 7680, 1024, True), (1744, 192, 3976, 8200, True), (2048, 2048, 8192, 256, False), (520, 512, 2056, 8200, False), (768, 768, 3072, 1000, False)])
@pytest.mark.parametrize("acc", [0, 1])
def test_bias_gradients_that_would_begin_another_round_follow_with_the_same_bits(d, da, f, k, apart, acc):
    """The one-row products of a layer's group, in it and as launches of their own, onto a stored gradient too; sizes on both
    sides of the rule, ragged tokens.  Bound: one rounding to bf16 and fp32 sums of k terms."""
    from tile_choice import part
    gen = torch.Generator(device=DEV).manual_seed(d + k)
    lay = dict(a_layout=S.SIF_A_ROW_M, b_layout=S.SIF_B_ROW_N)
    ones = torch.zeros((k, 8), device=DEV, dtype=torch.bfloat16)
    ones[:, 0] = 1
    rows = [(_bf16(gen, k, n), _bf16(gen, n)) for n in (f, 3 * da)]
    wide = [(_bf16(gen, k, m), _bf16(gen, k, n), torch.zeros((m, n), device=DEV, dtype=torch.bfloat16)) for m, n in ((d, f), (f, d), (d, da), (3 * da, d))]
    out = [[c.clone() for _, c in rows] for _ in range(2)]
    onto = lambda c: dict(lay, **(dict(epilogue=S.SIF_EPI_RESIDUAL, res=c) if acc else {}))
    prods = [S.gemm_args(a, b, c, *c.shape, k, c.shape[0], c.shape[1], c.shape[1], **lay) for a, b, c in wide]
    prods += [S.gemm_args(ones, b, c, 1, c.numel(), k, 8, c.numel(), c.numel(), **onto(c)) for (b, _), c in zip(rows, out[0])]
    assert part(prods, 4) == (4 if apart else 6)
    records = torch.zeros(S.sif_k_gemm_bf16_group_bytes(6) + 16, device=DEV, dtype=torch.uint8)
    torch.cuda.synchronize()
    S.sif_k_gemm_bf16_group(prods, records)
    for (b, _), c in zip(rows, out[1]):
        S.sif_k_gemm_bf16(ones, b, c, 1, c.numel(), k, 8, c.numel(), c.numel(), **onto(c))
    torch.cuda.synchronize()
    for (b, c0), x, y in zip(rows, *out):
        assert torch.equal(x, y)
        ref = b.double().sum(0) + acc * c0.double()
        assert bool(((x.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + (k + 2) * 2.0 ** -24 * (b.double().abs().sum(0) + c0.double().abs())).all())


# (rows, columns, K, kernel): K shorter than the kernel's ring (six steps of 128 with 32 rows, eight of 64 with 64x64, six of 64
# with 128x64, which no shorter K gets), as long as it, whole turns of it and some steps more, ragged at the end of either
# half of a step
FETCHING = [(m, n, k, "fetching " + name) for name, sizes, ks in (
    ("32x32", [(33, 72), (72, 2312)], (72, 128, 200, 640, 648, 704, 768, 1480, 1544)), ("32x64", [(848, 520), (77, 3072)], (72, 128, 200, 640, 648, 704, 768, 1480, 1544)),
    ("64x64", [(280, 1992)], (72, 128, 448, 456, 512, 640, 648, 704, 1024, 1480)), ("128x64", [(580, 2440)], (328, 384, 392, 640, 648, 704, 768, 1480)))
    for m, n in sizes for k in ks]
OTHERS = ([(m, n, k, name) for m, n, name in ((33, 72, "32x64"), (72, 2312, "32x64"), (280, 1992, "64x64"), (848, 520, "32x64")) for k in (8, 64)] + [(580, 2440, k, "32x64") for k in (8, 64, 72, 128)] +
          [(1100, 3080, k, "128x64" if k < 200 else "128x128 one") for k in (8, 64, 72, 128, 640, 648, 704, 1480)])


@pytest.mark.parametrize("al", [0, 1])
@pytest.mark.parametrize("bl", [0, 1])
@pytest.mark.parametrize("m,n,k,name", FETCHING + OTHERS)
def test_gemm_bf16_fed_tiles_give_the_bits_of_the_128_ones(m, n, k, name, al, bl):
    """Kernels with wavefronts that only fetch (FETCHING), and the ring beside them at the same sizes and short K."""
    from tile_choice import kernel
    gen = torch.Generator(device=DEV).manual_seed(m + 3 * n + 5 * k + al + 2 * bl)
    a, b, bias = torch.zeros(((m + 7) // 8 * 8, k), device=DEV, dtype=torch.bfloat16), _bf16(gen, n, k), _bf16(gen, n)
    a[:m] = _bf16(gen, m, k)
    A, Bt = (a if al == 0 else a.t().contiguous()), (b if bl == 0 else b.t().contiguous())
    out = [torch.full((m, n), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(2)]
    assert name is None or kernel(S.gemm_args(A, Bt, out[0], m, n, k, A.shape[1], Bt.shape[1], n, a_layout=al, b_layout=bl)) == name
    torch.cuda.synchronize()
    for c, tile in zip(out, (0, 128)):
        S.sif_k_gemm_bf16(A, Bt, c, m, n, k, A.shape[1], Bt.shape[1], n, a_layout=al, b_layout=bl, epilogue=S.SIF_EPI_BIAS, bias=bias, tile=tile)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
    ref = a[:m].double() @ b.double().t() + bias.double()
    bound = 2.0 ** -8 * ref.abs() + (k + 5) * 2.0 ** -24 * (a[:m].double().abs() @ b.double().abs().t() + bias.double().abs())
    assert bool(((out[0].double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("al", [0, 1])
@pytest.mark.parametrize("bl", [0, 1])
@pytest.mark.parametrize("m,n,k,name", [(72, 200, 1160, "fetching 32x32"), (600, 1544, 776, "fetching 64x64"), (600, 2440, 1160, "fetching 128x64"),
                                        (400, 2440, 1160, "32x64"), (792, 2440, 1160, "64x64"), (1576, 2440, 1160, "128x64"), (1032, 2440, 776, "128x128 one"),
                                        (4104, 2440, 776, "128x128 two"), (2008, 2440, 1160, "256x128"), (4360, 4104, 64, "256x256"), (4360, 4104, 192, "256x256")])
def test_gemm_bf16_long_rings_and_more_tiles_than_blocks_give_the_bits_of_the_128_ones(m, n, k, name, al, bl):
    """Every ring over more K steps than its unrolled body has, with a ragged step behind them; and 256x256 tiles, of which
    256 blocks work through 306 (one and three K steps): the next tile's operands travel while the last one is stored."""
    from tile_choice import kernel
    gen = torch.Generator(device=DEV).manual_seed(m + 3 * n + 5 * k + al + 2 * bl)
    a, b = _bf16(gen, m, k), _bf16(gen, n, k)
    A, Bt = (a if al == 0 else a.t().contiguous()), (b if bl == 0 else b.t().contiguous())
    out = [torch.full((m, n), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(2)]
    chosen = 256 if name == "256x256" else 0
    assert kernel(S.gemm_args(A, Bt, out[0], m, n, k, A.shape[1], Bt.shape[1], n, a_layout=al, b_layout=bl, tile=chosen)) == name
    torch.cuda.synchronize()
    for c, tile in zip(out, (chosen, 128)):
        S.sif_k_gemm_bf16(A, Bt, c, m, n, k, A.shape[1], Bt.shape[1], n, a_layout=al, b_layout=bl, tile=tile)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
    ref = a.double() @ b.double().t()
    bound = 2.0 ** -8 * ref.abs() + (k + 4) * 2.0 ** -24 * (a.double().abs() @ b.double().abs().t())
    assert bool(((out[0].double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("what,s,batch,dh,name", [("scores", 200, 6, 136, "fetching 32x64"), ("scores", 264, 6, 128, "fetching 64x64"), ("pv", 200, 6, 136, "fetching 32x32"),
                                                  ("pv", 776, 3, 136, "fetching 32x64"), ("pv", 776, 4, 136, "fetching 64x64"), ("pv", 776, 8, 136, "fetching 128x64"),
                                                  ("ptdo", 200, 6, 136, "fetching 32x32"), ("ptdo", 776, 3, 136, "fetching 32x64"), ("ptdo", 776, 4, 136, "fetching 64x64"),
                                                  ("ptdo", 776, 8, 136, "fetching 128x64"), ("slices", 520, 5, 200, "fetching 64x64"), ("slices", 200, 4, 192, "fetching 32x32")])
def test_batched_causal_and_sliced_products_on_fetching_kernels_give_the_bits_of_the_128_ones(what, s, batch, dh, name):
    """Causal scores (tiles above the diagonal are not written), products that stop at or begin with the diagonal, so that
    their first or last tiles have fewer K steps than the ring, and slices of one long K with a shorter, ragged last one.
    Bits of the 128x128 tiles, and the product: fp32 sums of at most s terms, one rounding where it is stored as bf16."""
    from tile_choice import kernel
    gen = torch.Generator(device=DEV).manual_seed(s + batch)
    p = torch.tril(_bf16(gen, batch, s, s))
    x, y = _bf16(gen, batch, s, dh), _bf16(gen, batch, s, dh)
    if what == "scores":
        m, n, k, a, b, ref, dtype = s, s, dh, x, y, x.double() @ y.double().transpose(1, 2).contiguous(), torch.float32
        kw = dict(epilogue=S.SIF_EPI_OUT_F32 | S.SIF_EPI_CAUSAL_SKIP, a_strides=(0, s * dh), b_strides=(0, s * dh), c_strides=(0, s * s))
        lda, ldb = dh, dh
    elif what == "slices":
        m, n, k, total, dtype = s, 264, dh, dh * (batch - 1) + 77, torch.float32
        lda = ldb = (total + 7) // 8 * 8
        a, b = _bf16(gen, m, lda), _bf16(gen, n, lda)
        a[:, total:] = 0
        cut = [slice(i * dh, min(total, (i + 1) * dh)) for i in range(batch)]
        ref = torch.stack([a[:, c].double() @ b[:, c].double().t() for c in cut])
        kw = dict(epilogue=S.SIF_EPI_OUT_F32, a_strides=(0, dh), b_strides=(0, dh), c_strides=(0, m * n), k_limit=total)
    else:
        m, n, k, a, b, dtype, lda, ldb = s, dh, s, p, x, torch.bfloat16, s, dh
        left = p.double() if what == "pv" else p.double().transpose(1, 2).contiguous()
        ref = left @ x.double()
        kw = dict(a_layout=S.SIF_A_ROW_K if what == "pv" else S.SIF_A_ROW_M, b_layout=S.SIF_B_ROW_N, k_causal=1 if what == "pv" else 2,
                  a_strides=(0, s * s), b_strides=(0, s * dh), c_strides=(0, s * dh))
    out = [torch.full((batch, m, n), 9.0, device=DEV, dtype=dtype) for _ in range(2)]
    assert kernel(S.gemm_args(a, b, out[0], m, n, k, lda, ldb, n, batch_inner=batch, **kw)) == name
    torch.cuda.synchronize()
    for c, tile in zip(out, (0, 128)):
        S.sif_k_gemm_bf16(a, b, c, m, n, k, lda, ldb, n, batch_inner=batch, tile=tile, **kw)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
    got = out[0].double()
    if what == "scores":
        at = torch.arange(s, device=DEV) // 128
        above = at[None, :] > at[:, None]
        assert bool((got[:, above] == 9.0).all())
        got, ref = got[:, ~above], ref[:, ~above]
    assert float((got - ref).norm() / ref.norm()) <= (2.0 ** -8 if dtype == torch.bfloat16 else 1e-5)


@pytest.mark.parametrize("al,bl", [(0, 0), (0, 1), (1, 1)])
def test_products_with_fetching_wavefronts_give_the_same_bits_beside_copies(al, bl):
    """What a fetching wavefront has waited for is what the others read behind the barrier: many times beside copies on another
    stream that keep the memory system busy, the bits of the quiet run."""
    from tile_choice import kernel
    gen = torch.Generator(device=DEV).manual_seed(5)
    cases = []
    for m, n, k, name in ((77, 768, 768, "fetching 32x32"), (512, 768, 3072, "fetching 32x64"), (600, 1544, 776, "fetching 64x64"), (600, 2440, 1160, "fetching 128x64")):
        a, b = _bf16(gen, *((m, k) if al == 0 else (k, (m + 7) // 8 * 8))), _bf16(gen, *((n, k) if bl == 0 else (k, n)))
        cases.append((a, b, m, n, k))
        assert kernel(S.gemm_args(a, b, a, m, n, k, a.shape[1], b.shape[1], n, a_layout=al, b_layout=bl)) == name

    side, big = torch.cuda.Stream(), torch.zeros(64 * 2 ** 20, device=DEV)

    def copy(times):
        with torch.cuda.stream(side):
            for _ in range(times):
                big.add_(1.0)                      # 256 MB read and written per pass, beside the kernels under test

    main = stream_beside(side, lambda: copy(32))

    def run(copies):
        out = [[torch.full((m, n), float("nan"), device=DEV, dtype=torch.bfloat16) for _, _, m, n, _ in cases] for _ in range(5)]
        torch.cuda.synchronize()
        copy(copies)
        for turn in out:
            for c, (a, b, m, n, k) in zip(turn, cases):
                S.sif_k_gemm_bf16(a, b, c, m, n, k, a.shape[1], b.shape[1], n, a_layout=al, b_layout=bl, stream=main)
        main.synchronize()
        beside = not side.query()
        torch.cuda.synchronize()
        return out, beside

    quiet, _ = run(0)
    for _ in range(6):
        got, beside = run(32)
        assert beside                          # copies were still to come when the last product was done
        assert all(torch.equal(x, y) for turn in got for x, y in zip(quiet[0], turn))


@pytest.mark.parametrize("shapes,k,tiles", [([(512, 128), (128, 512), (1, 512)], 1032, "128x128 one"), ([(1032, 776), (776, 3080), (1, 3080)], 1160, "256x128"),
                                            ([(4104, 4616), (2056, 2568), (1, 8200)], 512, "256x256")])
def test_groups_give_the_bits_of_the_128_tiles_on_every_tile(shapes, k, tiles):
    """Groups whose products' tile counts are no multiples of eight (the padding has nothing to do), with one-row products,
    a ragged K where the tiles allow it, and 256x256 tiles that are more than the chip's CUs, so that a block goes from one
    product's tile to another's."""
    from tile_choice import group
    gen = torch.Generator(device=DEV).manual_seed(k)
    lay = dict(a_layout=S.SIF_A_ROW_M, b_layout=S.SIF_B_ROW_N)
    prods, pairs = [], []
    for m, n in shapes:
        a, b = torch.zeros((k, (m + 7) // 8 * 8), device=DEV, dtype=torch.bfloat16), _bf16(gen, k, n)
        a[:, :m] = _bf16(gen, k, m)
        c = [torch.full((m, n), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(2)]
        prods.append(S.gemm_args(a, b, c[0], m, n, k, a.shape[1], n, n, **lay))
        pairs.append((a, b, c))
    assert group(prods)[1] == tiles
    records = torch.zeros(S.sif_k_gemm_bf16_group_bytes(len(prods)) + 16, device=DEV, dtype=torch.uint8)
    torch.cuda.synchronize()
    S.sif_k_gemm_bf16_group(prods, records)
    for a, b, c in pairs:
        S.sif_k_gemm_bf16(a, b, c[1], *c[1].shape, k, a.shape[1], b.shape[1], b.shape[1], tile=128, **lay)
    torch.cuda.synchronize()
    for a, b, c in pairs:
        assert torch.equal(c[0], c[1])
        ref = a[:, :c[0].shape[0]].double().t() @ b.double()
        assert float((c[0].double() - ref).norm() / ref.norm()) <= 2.0 ** -8


@pytest.mark.parametrize("m,n,k", [(77, 200, 136), (1000, 768, 256), (1032, 2304, 192)])
@pytest.mark.parametrize("epi", ["bias_residual", "gelu_aux", "gelu_grad", "f32"])
def test_gemm_bf16_epilogues_on_every_tile_width(m, n, k, epi):
    """The staged epilogues through the staging areas of tiles 64 and 128 columns wide against the 128x128 ones."""
    gen = torch.Generator(device=DEV).manual_seed(m + n + k)
    a, b, bias, res, z = _bf16(gen, m, k), _bf16(gen, n, k), _bf16(gen, n), _bf16(gen, m, n), _bf16(gen, m, n)
    got = []
    for tile in (0, 128):
        c = torch.zeros((m, n), device=DEV, dtype=torch.float32 if epi == "f32" else torch.bfloat16)
        aux = z.clone()
        kw = {"bias_residual": dict(epilogue=S.SIF_EPI_BIAS | S.SIF_EPI_RESIDUAL, bias=bias, res=res), "gelu_aux": dict(epilogue=S.SIF_EPI_GELU, bias=bias, aux=aux),
              "gelu_grad": dict(epilogue=S.SIF_EPI_GELU_GRAD, aux=aux), "f32": dict(epilogue=S.SIF_EPI_OUT_F32)}[epi]
        torch.cuda.synchronize()
        S.sif_k_gemm_bf16(a, b, c, m, n, k, k, k, n, tile=tile, **kw)
        torch.cuda.synchronize()
        got.append((c, aux))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    acc = a.double() @ b.double().t()
    ref = {"bias_residual": acc + bias.double() + res.double(), "gelu_aux": torch.nn.functional.gelu(acc + bias.double()), "f32": acc,
           "gelu_grad": acc * (0.5 * (1 + torch.erf(z.double() / 2 ** 0.5)) + z.double() * torch.exp(-z.double() ** 2 / 2) / (2 * torch.pi) ** 0.5)}[epi]
    assert float((got[0][0].double() - ref).norm() / ref.norm()) <= 2.0 ** -8


@pytest.mark.parametrize("m,n,k", [(256, 256, 64), (300, 520, 192), (513, 264, 128), (31, 777, 64)])
@pytest.mark.parametrize("epi", ["residual", "grad", "grad_residual", "grad_bias_residual", "gelu_aux_residual", "f32_residual"])
def test_gemm_bf16_staged_epilogues_on_256_tiles(m, n, k, epi):
    """What an epilogue reads is requested 32 or 64 rows ahead of its staging passes, a second tensor with its pass (of eight rows on
    256x256 tiles, of 32 on 128x128): whole and ragged tiles, an auxiliary tensor, a residual and both, vectors and (777 columns)
    single elements: the same bits, and the product (one rounding to bf16 of the result, and of fp32 sums that GELU' or GELU
    scales)."""
    gen = torch.Generator(device=DEV).manual_seed(m + n + k)
    a, b, bias, res, z = _bf16(gen, m, k), _bf16(gen, n, k), _bf16(gen, n), _bf16(gen, m, n), _bf16(gen, m, n)
    f32out = epi.startswith("f32")
    epilogue = sum(flag for name, flag in (("gelu", S.SIF_EPI_GELU), ("grad", S.SIF_EPI_GELU_GRAD), ("bias", S.SIF_EPI_BIAS), ("residual", S.SIF_EPI_RESIDUAL),
                                           ("f32", S.SIF_EPI_OUT_F32)) if name in epi.split("_"))
    got = []
    for tile in (256, 128):
        c, aux = torch.full((m, n), float("nan"), device=DEV, dtype=torch.float32 if f32out else torch.bfloat16), z.clone()
        torch.cuda.synchronize()
        S.sif_k_gemm_bf16(a, b, c, m, n, k, k, k, n, epilogue=epilogue, bias=bias if "bias" in epi else None, aux=None if f32out or epi == "residual" else aux,
                          res=(res.float() if f32out else res) if "residual" in epi else None, tile=tile)
        torch.cuda.synchronize()
        got.append((c, aux))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    ref = a.double() @ b.double().t() + (bias.double() if "bias" in epi else 0.0)
    if "grad" in epi:
        ref = ref * (0.5 * (1 + torch.erf(z.double() / 2 ** 0.5)) + z.double() * torch.exp(-z.double() ** 2 / 2) / (2 * torch.pi) ** 0.5)
    if "gelu" in epi:
        ref = torch.nn.functional.gelu(ref)
    ref = ref + (res.double() if "residual" in epi else 0.0)
    assert float((got[0][0].double() - ref).norm() / ref.norm()) <= 2.0 ** -8


EPILOGUES = ["plain", "gelu", "residual", "gelu_aux", "gelu_grad", "f32", "gelu_residual", "gelu_aux_residual", "grad_residual", "grad_bias_residual", "f32_residual",
             "f32_gelu", "f32_grad", "f32_grad_residual", "f32_gelu_aux_residual"]


def _epilogue(name, acc, bias, res, z):
    """(flags, bias?, residual?, auxiliary tensor?, result, auxiliary output or None) of a named epilogue over the product acc;
    everything in 64 bits.  GELU and a residual alone come with a bias."""
    words = name.split("_")
    grad, gelu = "grad" in words, "gelu" in words and "grad" not in words
    biased = gelu or "bias" in words or name in ("plain", "residual")
    flags = (S.SIF_EPI_GELU * gelu | S.SIF_EPI_GELU_GRAD * grad | S.SIF_EPI_RESIDUAL * ("residual" in words) | S.SIF_EPI_OUT_F32 * ("f32" in words) |
             S.SIF_EPI_BIAS * (biased and not gelu))
    x = acc + bias if biased else acc
    pre = x if gelu and "aux" in words else None
    if gelu:
        x = torch.nn.functional.gelu(x)
    if grad:
        x = x * (0.5 * (1 + torch.erf(z / 2 ** 0.5)) + z * torch.exp(-z ** 2 / 2) / (2 * torch.pi) ** 0.5)
    if "residual" in words:
        x = x + res
    return flags, biased, "residual" in words, grad or "aux" in words, x, pre


@pytest.mark.parametrize("m,n,far,k,tile,name",
                         [(m, n, far, 64, tile, None) for m, n, far in ((1, 8, False), (33, 200, False), (129, 136, False), (257, 328, False), (33, 200, True),
                                                                        (33, 77, False), (257, 333, False), (33, 77, True)) for tile in (0, 128, 256)] +
                         [(m, n + more, False, k, 0, name) for m, n, k, name in ((33, 200, 136, "fetching 32x32"), (847, 520, 136, "fetching 32x64"), (281, 1992, 136, "fetching 64x64"),
                                                                                 (581, 2440, 392, "fetching 128x64"), (401, 2440, 136, "32x64"), (793, 2440, 136, "64x64"),
                                                                                 (1577, 2440, 136, "128x64"), (1033, 2440, 776, "128x128 one"), (4105, 2440, 136, "128x128 two"),
                                                                                 (2009, 2440, 1160, "256x128")) for more in (0, -3)])
@pytest.mark.parametrize("epi", EPILOGUES)
def test_gemm_bf16_epilogues_write_their_rows_and_columns_only(m, n, far, k, tile, name, epi):
    """Rows further apart than their columns (by 24 elements, and by more than 2 M), the last rows and columns of a tile
    missing: what lies between the rows and behind the last one keeps its value, in the result and in the auxiliary tensor, and
    what lies there in the tensors that are read (NaN) reaches no result.  Bound: one rounding to bf16 of the result, and of
    fp32 sums that GELU' or GELU scales."""
    from tile_choice import kernel
    gen = torch.Generator(device=DEV).manual_seed(m + n)
    ld, below = (1 << 21) + 8 if far else n + 24, 2 if far else 256
    a, b, bias, res, z = _bf16(gen, m, k), _bf16(gen, n, k), _bf16(gen, n), _bf16(gen, m, n), _bf16(gen, m, n)
    flags, biased, residual, has_aux, ref, pre = _epilogue(epi, a.double() @ b.double().t(), bias.double(), res.double(), z.double())
    dtype = torch.float32 if "f32" in epi else torch.bfloat16
    c, aux, other = torch.full((m + below, ld), 7.0, device=DEV, dtype=dtype), None, None
    if has_aux:
        aux = torch.full((m + below, ld), float("nan"), device=DEV, dtype=torch.bfloat16)
        aux[:m, :n] = z
    if residual:
        other = torch.full((m + below, ld), float("nan"), device=DEV, dtype=dtype)
        other[:m, :n] = res
    assert name is None or kernel(S.gemm_args(a, b, c, m, n, k, k, k, ld)) == name
    torch.cuda.synchronize()
    S.sif_k_gemm_bf16(a, b, c, m, n, k, k, k, ld, epilogue=flags, bias=bias if biased else None, res=other, aux=aux, tile=tile)
    torch.cuda.synchronize()
    assert bool((c[m:] == 7.0).all()) and bool((c[:, n:] == 7.0).all())
    assert aux is None or bool(aux[m:].isnan().all()) and bool(aux[:, n:].isnan().all())
    assert float((c[:m, :n].double() - ref).norm() / ref.norm()) <= 2.0 ** -8
    if pre is not None:
        assert float((aux[:m, :n].double() - pre).norm() / pre.norm()) <= 2.0 ** -8


@pytest.mark.parametrize("m,k,tiles", [(136, 136, "128x128 one"), (776, 136, "128x128 two"), (776, 1160, "256x128"), (1032, 512, "256x256"), (2056, 1024, "256x256")])
@pytest.mark.parametrize("ragged", [False, True])
def test_a_group_whose_products_have_all_epilogues_gives_each_its_bits(m, k, tiles, ragged):
    """One launch over products with the common epilogues and with the others, ragged columns among them: the bits of each by
    itself."""
    from tile_choice import group
    gen = torch.Generator(device=DEV).manual_seed(m + k)
    lay = dict(a_layout=S.SIF_A_ROW_M, b_layout=S.SIF_B_ROW_N)
    prods, outs = [], []
    for i, epi in enumerate(EPILOGUES):
        n, pitch = m // 2 + 8 * i - (3 if ragged and i % 4 == 3 else 0), m + 512
        a, b, bias = _bf16(gen, k, m), _bf16(gen, k, m + 512), _bf16(gen, m + 512)
        flags, biased, residual, has_aux, _, _ = _epilogue(epi, *[torch.zeros(1, device=DEV)] * 4)
        dtype = torch.float32 if "f32" in epi else torch.bfloat16
        res, z = torch.randn((m, pitch), device=DEV, generator=gen).to(dtype), _bf16(gen, m, pitch)
        pair = [(torch.full((m, pitch), 7.0, device=DEV, dtype=dtype), z.clone()) for _ in range(2)]
        call = lambda c, aux, **kw: ((a, b, c, m, n, k, m, m + 512, pitch), dict(lay, epilogue=flags, bias=bias if biased else None, res=res if residual else None,
                                                                              aux=aux if has_aux else None, **kw))
        args, kw = call(*pair[0])
        prods.append(S.gemm_args(*args, **kw))
        args, kw = call(*pair[1], tile=128)
        outs.append((pair, a, b, bias, res))
        torch.cuda.synchronize()
        S.sif_k_gemm_bf16(*args, **kw)
    assert group(prods)[1] == tiles
    records = torch.zeros(S.sif_k_gemm_bf16_group_bytes(len(prods)) + 16, device=DEV, dtype=torch.uint8)
    torch.cuda.synchronize()
    S.sif_k_gemm_bf16_group(prods, records)
    torch.cuda.synchronize()
    for epi, (pair, *_) in zip(EPILOGUES, outs):
        assert torch.equal(pair[0][0], pair[1][0]) and torch.equal(pair[0][1], pair[1][1]), epi


@pytest.mark.parametrize("n,most", [(4096, 3.0), (4093, 2.2)])
@pytest.mark.parametrize("tile", [128, 256])
def test_gemm_bf16_epilogues_do_not_wait_for_every_element(n, most, tile):
    """A residual together with GELU or GELU', and fp32 with any of these, are vectors where the columns are a multiple of eight:
    at most three times the plain product's time (they move up to five times its bytes and take 1.2 to 2.1 times as long, one
    element at a time up to 6.3 times).  Ragged columns: what is read for several elements is waited for once (1.0 to 1.7 times
    the plain product's time, with a wait for each element up to 2.8)."""
    m, k = 4096, 512
    gen = torch.Generator(device=DEV).manual_seed(1)
    a, b, bias = _bf16(gen, m, k), _bf16(gen, n, k), _bf16(gen, n)
    us = {}
    for epi in EPILOGUES:
        flags, biased, residual, has_aux, _, _ = _epilogue(epi, *[torch.zeros(1, device=DEV)] * 4)
        dtype = torch.float32 if "f32" in epi else torch.bfloat16
        c, res, aux = (torch.zeros((m, n), device=DEV, dtype=t) for t in (dtype, dtype, torch.bfloat16))
        launch = lambda: S.sif_k_gemm_bf16(a, b, c, m, n, k, k, k, n, epilogue=flags, bias=bias if biased else None, res=res if residual else None,
                                           aux=aux if has_aux else None, tile=tile)
        times = []
        for _ in range(6):
            at = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            torch.cuda.synchronize()
            at[0].record()
            for _ in range(10):
                launch()
            at[1].record()
            torch.cuda.synchronize()
            times.append(at[0].elapsed_time(at[1]) * 100)
        us[epi] = min(times)
    assert all(t <= most * us["plain"] for t in us.values()), us


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("bsz,s,h", [(2, 2, 2), (1, 63, 1), (2, 65, 2), (1, 129, 3), (2, 192, 1), (1, 257, 2), (1, 449, 1)])
def test_attention_with_heads_of_128_at_the_edges_of_its_tiles(bsz, s, h, causal):
    """K and V fetched in turns (forward), in 64-key tiles (dq), q and do in 64-query steps (dk, dv): one tile, an odd and
    an even number of them, remainders of one row and of all but one.  Bounds: those of the fused attention's other tests, and in dq and dk what
    rowsum(do o) is off by for an o rounded to bf16 (2^-8 sum |do| |o|): with two keys a gradient is a small difference of
    such sums."""
    from oracle.decoder import attention_bwd, attention_fwd
    from oracle.numerics import Prec
    from gpu_util import assert_bf16_close
    rng, da = np.random.default_rng(s + 7 * causal), 128 * h
    Q, DO = (torch.from_numpy(rng.standard_normal((bsz, s, n), dtype=np.float32)).to(DEV).to(torch.bfloat16) for n in (3 * da, da))
    o, dqkv = torch.zeros((bsz, s, da), device=DEV, dtype=torch.bfloat16), torch.full((bsz, s, 3 * da), 5.0, device=DEV, dtype=torch.bfloat16)
    lse, delta = torch.zeros((bsz * h, s), device=DEV), torch.zeros((bsz * h, s), device=DEV)
    torch.cuda.synchronize()
    S.sif_k_attn_fwd(Q, o, bsz, s, h, 128, 3 * da, da, causal, lse=lse)
    S.sif_k_attn_bwd(Q, o, DO, lse, delta, dqkv, bsz, s, h, 128, 3 * da, da, 3 * da, causal)
    torch.cuda.synchronize()
    prec, qkv, do = Prec("bf16"), up(Q), up(DO)
    ref_o, prob = attention_fwd(qkv, h, 128, bool(causal), prec)
    ref = attention_bwd(do, qkv, prob, h, 128, prec)
    assert_bf16_close(up(o), ref_o, "o", elem_slack=4e-3)
    heads = lambda x: x.reshape(bsz, s, h, 128).transpose(0, 2, 1, 3)
    back = lambda x: x.transpose(0, 2, 1, 3).reshape(bsz, s, da)
    err = prob * (2.0 ** -8 / 128 ** 0.5 * (np.abs(heads(do)) * np.abs(heads(ref_o))).sum(-1)[..., None])
    aq, ak = np.abs(heads(qkv[..., :da])), np.abs(heads(qkv[..., da:2 * da]))
    for name, lo, extra in (("dq", 0, back(err @ ak)), ("dk", da, back(err.transpose(0, 1, 3, 2) @ aq)), ("dv", 2 * da, 0.0)):
        got, want = up(dqkv)[..., lo:lo + da], ref[..., lo:lo + da]
        assert np.all(np.abs(got - want) <= 2.0 ** -7 * np.abs(want) + 6e-3 * np.abs(want).max() + extra), name


@pytest.mark.parametrize("with_sum", [False, True])
@pytest.mark.parametrize("rows,d,shift", [(1, 2056, 0), (17, 2056, 1), (33, 4088, 0), (530, 4096, 0), (8200, 2568, 1)])
def test_layernorm_backward_of_rows_wider_than_2048(rows, d, shift, with_sum):
    """Groups of four rows in a block: one row, an odd number of rows per block, blocks without rows, vectors past the row's end, partial
    sums that are not 16-byte aligned.  Bounds: those of the other LayerNorm test; the column sums of n rows are fp32 sums,
    which err by at most (n + 4) 2^-24 of their terms' magnitudes, and are rounded to bf16 once (2^-8)."""
    from oracle import numerics as N
    from gpu_util import assert_bf16_close
    gen = torch.Generator(device=DEV).manual_seed(rows + d)
    X, DY, R, G = _bf16(gen, rows, d) * 2, _bf16(gen, rows, d), _bf16(gen, rows, d), _bf16(gen, d) + 1
    x, dy, res, g = up(X), up(DY), up(R), up(G)
    _, mu, rs = N.layernorm_fwd(x, g, np.zeros(d))
    dx, dg, db = torch.zeros_like(X), torch.zeros_like(G), torch.zeros_like(G)
    dsum = torch.zeros_like(G) if with_sum else None
    part = torch.full((3 * S.sif_colsum_parts(rows) * d + 4,), float("nan"), device=DEV)[shift:]
    mean, rstd = f32(mu[:, 0].astype(np.float32)), f32(rs[:, 0].astype(np.float32))
    torch.cuda.synchronize()
    S.sif_k_layernorm_bwd(DY, X, G, mean, rstd, R, dx, dg, db, part, rows, d, dsum=dsum)
    torch.cuda.synchronize()
    rdx, rdg, _ = N.layernorm_bwd(dy, x, g, mu, rs)
    assert_bf16_close(up(dx), res + rdx, "dx")
    assert_bf16_close(up(dg), rdg, "dg")
    for got, terms in ((db, dy),) + (((dsum, up(dx)),) if with_sum else ()):
        want = terms.sum(0)
        assert np.all(np.abs(up(got) - want) <= 2.0 ** -8 * np.abs(want) + (rows + 4) * 2.0 ** -24 * np.abs(terms).sum(0))


@pytest.mark.parametrize("rows,d", [(1, 2056), (3, 4096), (17, 2056), (33, 4088), (530, 4096), (8200, 2568), (16400, 2560)])
def test_layernorm_backward_of_wide_rows_sums_in_the_order_of_narrow_ones(rows, d):
    """The order of every sum is that of a wavefront per row: lane l of 64 adds the row's terms of columns 8 (l + 64 t) + i by
    ascending t and i and the lanes are joined by halves; a block's column sums are those of its rows 0, 4, 8, .., of 1, 5, 9,
    .. and so on, added in turn.  So longer chains of additions (another error against 64 bits) fail here, at blocks of one
    row, of remainders and of more rows than a block takes at a time.  fp32 steps are taken in 64 bits and rounded once, a
    product that feeds a sum only there, as the fused operations do; all bits must agree."""
    gen = torch.Generator(device=DEV).manual_seed(3 * rows + d)
    X, DY, R, G = _bf16(gen, rows, d) * 2, _bf16(gen, rows, d), _bf16(gen, rows, d), _bf16(gen, d) + 1
    mean = X.float().mean(1)
    rstd = 1 / (X.float().var(1, unbiased=False) + 1e-5).sqrt()
    dx, outs = torch.zeros_like(X), [torch.zeros_like(G) for _ in range(3)]
    parts = S.sif_colsum_parts(rows)
    part = torch.full((3, parts, d), float("nan"), device=DEV)
    torch.cuda.synchronize()
    S.sif_k_layernorm_bwd(DY, X, G, mean, rstd, R, dx, outs[0], outs[1], part, rows, d, dsum=outs[2])
    torch.cuda.synchronize()

    r32 = lambda v: v.float().double()
    dy, g, m, rs = DY.double(), G.double(), mean.double()[:, None], rstd.double()[:, None]
    xh, dxh = r32(r32(X.double() - m) * rs), r32(dy * g)
    chunks = (d + 511) // 512

    def row_mean(a, b):                          # of a b, in the wavefront's order
        lanes = torch.zeros(2, rows, chunks * 512, device=DEV, dtype=torch.float64)
        lanes[0, :, :d], lanes[1, :, :d] = a, b
        a, b = lanes.view(2, rows, chunks, 64, 8)
        s = torch.zeros(rows, 64, device=DEV, dtype=torch.float64)
        for t in range(chunks):
            for i in range(8):
                s = r32(s + a[:, t, :, i] * b[:, t, :, i])
        while s.shape[1] > 1:
            half = s.shape[1] // 2
            s = r32(s[:, :half] + s[:, half:])
        return r32(s / d)

    want = r32(rs * r32(r32(dxh - row_mean(dxh, torch.ones_like(dxh))) - xh * row_mean(dxh, xh)) + R.double()).to(torch.bfloat16)
    assert torch.equal(dx, want)

    per = (rows + parts - 1) // parts
    for which, (a, b) in enumerate(((dy, xh), (dy, torch.ones_like(dy)), (dx.double(), torch.ones_like(dy)))):
        want = torch.zeros(parts, d, device=DEV, dtype=torch.float64)
        for first in range(4):
            s = torch.zeros_like(want)
            for k in range(first, per, 4):
                at = torch.arange(parts, device=DEV) * per + k
                ok = at < rows
                s[ok] = r32(s[ok] + a[at[ok]] * b[at[ok]])
            want = r32(want + s)
        assert torch.equal(part[which], want.float()), which


@pytest.mark.parametrize("case", ["k_causal_1", "k_causal_2", "causal_skip"])
def test_causal_products_of_a_group_keep_to_their_128_tiles(case):
    """A causal product in a group reads no more of its left operand than the 128-row tile has (beyond it stands what was
    never written, here NaN) and writes no tile above the diagonal, also where the group's size asks for taller tiles: the
    bits of the product by itself on 128x128 tiles."""
    gen = torch.Generator(device=DEV).manual_seed(11)
    m = n = 2560
    k = 64 if case == "causal_skip" else m
    a, b = _bf16(gen, k, m), _bf16(gen, k, n)
    row, col = torch.arange(k, device=DEV)[:, None], torch.arange(m, device=DEV)[None]
    kw = {}
    if case == "k_causal_1":                     # A(m, k) is zero for k > m, and unwritten from the next 128 on
        a[row > col] = 0
        a[row >= (col // 128 + 1) * 128] = float("nan")
        kw = dict(k_causal=1)
    elif case == "k_causal_2":                   # zero for k < m, unwritten before the 128 that hold m
        a[row < col] = 0
        a[row < col // 128 * 128] = float("nan")
        kw = dict(k_causal=2)
    else:
        kw = dict(epilogue=S.SIF_EPI_CAUSAL_SKIP)
    long_a, long_b = _bf16(gen, 8192, 136), _bf16(gen, 8192, 264)      # a product beside it that asks for the tall tiles
    c, alone = torch.full((m, n), 7.0, device=DEV, dtype=torch.bfloat16), torch.full((m, n), 7.0, device=DEV, dtype=torch.bfloat16)
    other = torch.zeros((136, 264), device=DEV, dtype=torch.bfloat16)
    lay = dict(a_layout=S.SIF_A_ROW_M, b_layout=S.SIF_B_ROW_N)
    records = torch.zeros(S.sif_k_gemm_bf16_group_bytes(2) + 16, device=DEV, dtype=torch.uint8)
    torch.cuda.synchronize()
    S.sif_k_gemm_bf16_group([S.gemm_args(a, b, c, m, n, k, m, n, n, **lay, **kw), S.gemm_args(long_a, long_b, other, 136, 264, 8192, 136, 264, 264, **lay)], records)
    S.sif_k_gemm_bf16(a, b, alone, m, n, k, m, n, n, tile=128, **lay, **kw)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(alone.float()).all())
    assert torch.equal(c, alone)
    assert float((other.double() - long_a.double().t() @ long_b.double()).norm() / other.double().norm()) <= 2.0 ** -8
