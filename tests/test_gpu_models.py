"""GPU parity of whole models against the oracle, through the C ABI: the fp32 MLP training step and forward,
the bf16 decoder training step (stage by stage), the bf16 encoder forward."""
import numpy as np
import pytest
import torch

import synth_inputs as Y
from oracle import decoder as OD
from oracle import encoder as OE
from oracle import mlp as OM
from oracle.numerics import Prec

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2503_02550_amd as S
    from paper_2503_02550_amd import params as P
    from paper_2503_02550_amd.session import Session, decoder_shape, encoder_shape, mlp_shape
    from gpu_util import DEV, bf, f32, i32, up, q, rel_err, assert_bf16_close, assert_f32_close, lse_reference



def assert_update_close(p_got, p_ref, g_got, g_ref, lr, name):
    """fp32 master parameters after p <- p - lr g.  The update is fp32 arithmetic on a gradient held in bf16: the two
    sides' parameters may differ by lr times the difference of their gradients (bounded by the bf16 tolerance on the
    gradients, 2e-2 of the largest) on top of the fp32 tolerance 1e-4."""
    p_got, p_ref = np.asarray(p_got, np.float64), np.asarray(p_ref, np.float64)
    bound = 1e-4 * np.max(np.abs(p_ref)) + lr * 2e-2 * np.max(np.abs(g_ref))
    assert np.max(np.abs(p_got - p_ref)) <= bound, name
    # and the device's own update, from the gradient it holds, is exact to fp32 rounding
    step = (p_got - p_ref) + lr * (np.asarray(g_got, np.float64) - np.asarray(g_ref, np.float64))
    assert np.max(np.abs(step)) <= 1e-6 * np.max(np.abs(p_ref)) + 1e-9, name

def test_mlp_training_steps_and_forward_match_oracle():
    c = Y.TINY_MLP
    shape = mlp_shape(c["d_in"], c["d_hidden"], c["d_out"], c["train_batch"])
    p0 = Y.mlp_params(0, c["d_in"], c["d_hidden"], c["d_out"])
    p0["b1"] = p0["b1"] + 0.01
    ref = {k: v.astype(np.float64) for k, v in p0.items()}
    with Session() as s:
        s.register_training(shape, P.pack(shape, p0), par_mode=S.SIF_PAR_FIXED, lr=c["lr"], fixed_bubble_ns=200_000)
        loss = torch.zeros(1, device=DEV)
        for step in range(5):
            x, t = Y.mlp_batch(0, step, c["train_batch"], c["d_in"], c["d_out"])
            X, T = f32(x), f32(t)
            torch.cuda.synchronize()
            s.step(X, T, loss)
            s.sync()
            rl, ref, rg = OM.mlp_train_step(ref, x, t, c["lr"])
            assert abs(loss.item() - rl) <= 1e-4 * abs(rl), step
            got_g = P.unpack(shape, up(s.train_tensor("grads", dtype=torch.float32)))
            got_p = P.unpack(shape, up(s.train["master"]))
            for k in ref:
                assert_f32_close(got_g[k], rg[k], f"step {step} grad {k}")
                assert_f32_close(got_p[k], ref[k], f"step {step} param {k}", 1e-5)
    # inference forward, batch 8 and a smaller batch
    ishape = mlp_shape(c["d_in"], c["d_hidden"], c["d_out"], c["infer_batch"])
    with Session() as s:
        m = s.register_inference(ishape, P.pack(ishape, p0))
        for b in (c["infer_batch"], 3):
            x = Y.activations(5, b, c["d_in"])
            X, out = f32(x), torch.zeros((b, c["d_out"]), device=DEV)
            torch.cuda.synchronize()
            s.wait(s.submit_offline(m, X, out, b))
            y, _ = OM.mlp_forward({k: v.astype(np.float64) for k, v in p0.items()}, x)
            assert_f32_close(up(out), y, f"mlp forward batch {b}")


DEC_SMALL = dict(n_layers=2, d_model=64, n_heads=4, d_head=16, d_ffn=256, vocab=211, max_pos=40, batch=3, seq=40, causal=True)
DEC_TILES = dict(n_layers=2, d_model=256, n_heads=2, d_head=64, d_ffn=512, vocab=1000, max_pos=136, batch=2, seq=136, causal=True)
DEC_SPLIT = dict(n_layers=2, d_model=128, n_heads=2, d_head=64, d_ffn=256, vocab=600, max_pos=128, batch=2, seq=128, causal=True)
# a vocabulary long enough for the LM head's data gradient to be cut along K (ragged last slice: 8203 = 7 * 1088 + 587)
DEC_VOCAB = dict(n_layers=1, d_model=64, n_heads=1, d_head=64, d_ffn=128, vocab=8203, max_pos=72, batch=2, seq=72, causal=True)


@pytest.mark.parametrize("cfg", [DEC_SMALL, DEC_TILES, DEC_SPLIT, DEC_VOCAB],
                         ids=["small", "several-tiles-ragged", "split-weight-gradients", "vocabulary-cut-along-k"])
def test_decoder_training_step_matches_oracle_stage_by_stage(cfg):
    shape = decoder_shape(cfg)
    master = Y.decoder_params(1, cfg, perturb=True)
    ids, tg = Y.token_ids(2, cfg["batch"], cfg["seq"], cfg["vocab"]), Y.token_ids(3, cfg["batch"], cfg["seq"], cfg["vocab"])
    ids[0, 5] = ids[0, 1] = ids[1, 7]                                 # repeated tokens
    rl, rnew, rg, rc = OD.gpt_train_step(master, ids, tg, cfg, 0.01, "bf16")
    b, sq, d = cfg["batch"], cfg["seq"], cfg["d_model"]
    with Session() as s:
        s.register_training(shape, P.pack(shape, master), par_mode=S.SIF_PAR_NONE, lr=0.01)
        loss, I, T = torch.zeros(1, device=DEV), i32(ids), i32(tg)
        torch.cuda.synchronize()
        s.step(I, T, loss)
        s.sync()
        # forward activations, layer by layer
        for l in range(cfg["n_layers"]):
            for name in ("ln1", "qkv", "o", "x_mid", "ln2", "z", "a"):
                got = up(s.train_tensor(name, l)).reshape(rc["layers"][l][name].shape)
                assert_bf16_close(got, rc["layers"][l][name], f"L{l}.{name}", elem_slack=8e-3)
            if cfg["d_head"] in (64, 128):     # fused attention keeps log-sum-exp of the scores, not the probabilities
                # the saved log-sum-exp of the scores, against its definition on the qkv the device holds (checked above)
                lse = up(s.train_tensor("lse", l, dtype=torch.float32)).reshape(b * cfg["n_heads"], sq)
                qkv_dev = up(s.train_tensor("qkv", l)).reshape(b, sq, -1)
                assert rel_err(lse, lse_reference(qkv_dev, cfg["n_heads"], cfg["d_head"])) <= 1e-5
            else:
                sp = (sq + 7) // 8 * 8
                prob = up(s.train_tensor("prob", l)).reshape(b, cfg["n_heads"], sq, sp)[..., :sq]
                assert_bf16_close(prob, rc["layers"][l]["prob"], f"L{l}.prob", elem_slack=8e-3)
        assert abs(loss.item() - rl) <= 2e-2 * abs(rl)
        # gradients and updated parameters
        got_g = P.unpack(shape, up(s.train_tensor("grads")))
        got_p = P.unpack(shape, up(s.train["master"]))
        got_w = P.unpack(shape, up(s.train_tensor("work")))
        worst = 0.0
        for path, _ in P.layout(shape):
            g_ref = rg[path] if isinstance(path, str) else rg["layers"][path[1]][path[2]]
            g_got = got_g[path] if isinstance(path, str) else got_g["layers"][path[1]][path[2]]
            e = rel_err(g_got, g_ref)
            worst = max(worst, e)
            assert e <= 2e-2, (path, e)
            p_ref = rnew[path] if isinstance(path, str) else rnew["layers"][path[1]][path[2]]
            p_got = got_p[path] if isinstance(path, str) else got_p["layers"][path[1]][path[2]]
            assert_update_close(p_got, p_ref, g_got, g_ref, 0.01, path)
            w_got = got_w[path] if isinstance(path, str) else got_w["layers"][path[1]][path[2]]
            assert np.array_equal(w_got, q(p_got)), path                # working copy = bf16(master)
        print("worst gradient error", worst)


# 258 tile rows of 256 for the LM head's weight gradient: 256 of them are one whole round of one block per CU, the last
# two (464 rows, the second one ragged) are cut along the 768 tokens into six slices of 128
DEC_WTE_TAIL = dict(n_layers=1, d_model=64, n_heads=1, d_head=64, d_ffn=128, vocab=66000, max_pos=128, batch=6, seq=128, causal=True)


def test_lm_head_weight_gradient_with_its_last_tile_rows_cut_along_k_matches_oracle():
    cfg = DEC_WTE_TAIL
    shape = decoder_shape(cfg)
    master = Y.decoder_params(1, cfg, perturb=True)
    ids, tg = Y.token_ids(2, cfg["batch"], cfg["seq"], cfg["vocab"]), Y.token_ids(3, cfg["batch"], cfg["seq"], cfg["vocab"])
    tg[0, :8] = np.arange(65990, 65998)            # targets and inputs among the last rows as well
    ids[1, :8] = np.arange(65700, 65708)
    rl, rnew, rg, rc = OD.gpt_train_step(master, ids, tg, cfg, 0.01, "bf16")
    with Session() as s:
        s.register_training(shape, P.pack(shape, master), par_mode=S.SIF_PAR_NONE, lr=0.01)
        names, i = [], 0
        while S.sif_train_op_name(s.ctx, 0, i) is not None:
            names.append(S.sif_train_op_name(s.ctx, 0, i))
            i += 1
        assert "dwte_head_tail" in names and "dwte_head_sum" in names, "the plan did not cut the last tile rows"
        loss, I, T = torch.zeros(1, device=DEV), i32(ids), i32(tg)
        torch.cuda.synchronize()
        s.step(I, T, loss)
        s.sync()
        assert abs(loss.item() - rl) <= 2e-2 * abs(rl)
        got_g = P.unpack(shape, up(s.train_tensor("grads")))
        for lo, hi in ((0, 65536), (65536, 65792), (65792, 66000)):      # the whole round, the two cut tile rows
            e = rel_err(got_g["wte"][lo:hi], rg["wte"][lo:hi])
            assert e <= 2e-2, (lo, hi, e)
        for path, _ in P.layout(shape):
            g_ref = rg[path] if isinstance(path, str) else rg["layers"][path[1]][path[2]]
            g_got = got_g[path] if isinstance(path, str) else got_g["layers"][path[1]][path[2]]
            assert rel_err(g_got, g_ref) <= 2e-2, path


def test_decoder_stack_with_local_heads_matches_oracle():
    # tensor-shard shaped block: n_heads*d_head != d_model, no embedding, upstream gradient from the caller
    cfg = dict(n_layers=2, d_model=128, n_heads=2, d_head=32, d_ffn=192, vocab=0, max_pos=0, batch=2, seq=72, causal=True)
    shape = decoder_shape(cfg)
    master = Y.decoder_params(4, cfg, perturb=True)
    x, dy = Y.activations(5, 2, 72, 128), Y.activations(6, 2, 72, 128, scale=0.01)
    prec = Prec("bf16")
    w = OD.working_copy(master, prec)
    ry, rdx, rgr, _ = OD.stack_fwd_bwd(w["layers"], q(x), q(dy), cfg, prec)
    with Session() as s:
        s.register_training(shape, P.pack(shape, master), par_mode=S.SIF_PAR_TP, lr=0.0, bw_bytes_per_s=50_000_000_000)
        X, DY = bf(x), bf(dy)
        torch.cuda.synchronize()
        s.step(X, DY)
        s.sync()
        assert_bf16_close(up(s.train_tensor("x_out", 1)).reshape(ry.shape), ry, "stack output", elem_slack=8e-3)
        assert rel_err(up(s.train_tensor("dx_in")).reshape(rdx.shape), rdx) <= 2e-2
        got_g = P.unpack(shape, up(s.train_tensor("grads")))
        for l in range(2):
            for k in OD.LAYER_KEYS:
                assert rel_err(got_g["layers"][l][k], rgr[l][k]) <= 2e-2, (l, k)
        assert s.stats().bubble_ns > 0                               # 8 tensor-parallel bubbles were modelled


ENC_SMALL = dict(n_layers=2, d_model=64, n_heads=4, d_head=16, d_ffn=256, vocab=97, max_pos=64, batch=4, seq=37)
ENC_TILES = dict(n_layers=3, d_model=256, n_heads=4, d_head=64, d_ffn=1024, vocab=500, max_pos=200, batch=3, seq=200)


@pytest.mark.parametrize("cfg", [ENC_SMALL, ENC_TILES], ids=["small-ragged", "several-tiles"])
def test_encoder_forward_matches_oracle(cfg):
    shape = encoder_shape(cfg)
    master = Y.encoder_params(7, cfg, perturb=True)
    w = OE.working_copy(master, "bf16")
    with Session() as s:
        m = s.register_inference(shape, P.pack(shape, master))
        for b, sq in ((cfg["batch"], cfg["seq"]), (1, 5), (2, cfg["seq"] - 3)):
            ids = Y.token_ids(8 + b, b, sq, cfg["vocab"])
            I, out = i32(ids), torch.zeros((b, sq, cfg["d_model"]), device=DEV, dtype=torch.bfloat16)
            torch.cuda.synchronize()
            s.wait(s.submit_offline(m, I, out, b, sq))
            ref = OE.encoder_forward(w, ids, cfg, "bf16")
            assert_bf16_close(up(out), ref, f"encoder {b}x{sq}", elem_slack=1.5e-2)


def test_registration_and_submit_errors():
    cfg = ENC_SMALL
    shape = encoder_shape(cfg)
    master = P.pack(shape, Y.encoder_params(9, cfg))
    with Session() as s:
        m = s.register_inference(shape, master)
        out = torch.zeros((4, 37, 64), device=DEV, dtype=torch.bfloat16)
        ids = i32(Y.token_ids(1, 4, 37, cfg["vocab"]))
        with pytest.raises(S.SifError):
            s.submit_offline(m, ids, out, 5, 37)                       # batch above the registered maximum
        with pytest.raises(S.SifError):
            s.submit_offline(m, ids, out, 4, 38)                       # sequence above the registered maximum
        with pytest.raises(S.SifError):
            s.submit_offline(m + 1, ids, out, 4, 37)                   # unknown model
        with pytest.raises(S.SifError):
            s.submit_online(m, ids, out, 37)                           # registered as offline
        with pytest.raises(S.SifError):
            s.register_inference(shape, master, peak_bytes=1 << 60)    # Principle-I
        bad = encoder_shape(dict(cfg, d_model=60))
        with pytest.raises(S.SifError):
            s.register_inference(bad, master)


def test_pipeline_stage_1f1b_step_matches_oracle():
    """Pipeline-parallel stage share: micro-batches in 1F1B order, gradient accumulation, one update, the idle
    intervals of the schedule as bubbles."""
    from oracle import bubbles as OB
    cfg = dict(n_layers=2, d_model=128, n_heads=2, d_head=64, d_ffn=256, vocab=0, max_pos=0, batch=2, seq=64, causal=True)
    stages, micro, stage, tf, tb = 3, 4, 1, 300_000, 500_000
    shape = decoder_shape(cfg)
    master = Y.decoder_params(40, cfg, perturb=True)
    xs, dys = Y.activations(41, micro, 2, 64, 128), Y.activations(42, micro, 2, 64, 128, scale=0.01)
    rys, rdxs, rnew, rg = OD.stack_train_step_microbatched(master["layers"], q(xs), q(dys), cfg, 0.01, "bf16")
    with Session() as s:
        s.register_training(shape, P.pack(shape, master), par_mode=S.SIF_PAR_PP, lr=0.01, pp_stages=stages, pp_micro=micro,
                            pp_stage=stage, pp_tf_ns=tf, pp_tb_ns=tb)
        X, DY = bf(xs), bf(dys)
        torch.cuda.synchronize()
        s.step(X, DY)
        s.sync()
        assert_bf16_close(up(s.train_tensor("y_all")).reshape(rys.shape), rys, "stage outputs", elem_slack=8e-3)
        assert rel_err(up(s.train_tensor("dx_all")).reshape(rdxs.shape), rdxs) <= 2e-2
        got_g = P.unpack(shape, up(s.train_tensor("grads")))
        got_p = P.unpack(shape, up(s.train["master"]))
        for l in range(2):
            for k in OD.LAYER_KEYS:
                assert rel_err(got_g["layers"][l][k], rg[l][k]) <= 2e-2, (l, k)
                assert_update_close(got_p["layers"][l][k], rnew[l][k], got_g["layers"][l][k], rg[l][k], 0.01, (l, k))
        bubbles = [(t1 - t0) for kind, _, _, _, t0, t1 in S.sif_read_trace(s.ctx, 0) if kind == 3]
        want = [ns for _, ns in OB.pp_1f1b_bubbles(stage, stages, micro, tf, tb)]
        assert len(bubbles) == len(want) == 4
        # at least the modelled length; well below the device deadline (4x + 100 ms) that a lost host release would show
        assert all(b >= w for b, w in zip(bubbles, want)) and all(b <= w + 50_000_000 for b, w in zip(bubbles, want)), (bubbles, want)
    with pytest.raises(S.SifError):
        with Session() as s:
            s.register_training(shape, P.pack(shape, master), par_mode=S.SIF_PAR_PP, pp_stages=4, pp_micro=3, pp_stage=0)


def test_pipeline_stage_sizes_its_bubbles_from_measured_pass_times():
    """Registered without per-micro-batch times, a stage measures them during calibration; its idle intervals then
    add up to (stages - 1)(t_f + t_b), the textbook total of the 1F1B schedule, with t_f + t_b = compute time / micro-batches."""
    cfg = dict(n_layers=2, d_model=256, n_heads=4, d_head=64, d_ffn=1024, vocab=0, max_pos=0, batch=2, seq=128, causal=True)
    stages, micro, stage = 4, 6, 1
    shape = decoder_shape(cfg)
    master = Y.decoder_params(44, cfg)
    xs, dys = Y.activations(45, micro, 2, 128, 256), Y.activations(46, micro, 2, 128, 256, scale=0.01)
    with Session() as s:
        s.register_training(shape, P.pack(shape, master), par_mode=S.SIF_PAR_PP, lr=0.01, pp_stages=stages, pp_micro=micro, pp_stage=stage)
        X, DY = bf(xs), bf(dys)
        torch.cuda.synchronize()
        S.sif_calibrate(s.ctx, 2, X, DY)
        s.step(X, DY)
        s.sync()
        tr = [r for r in S.sif_read_trace(s.ctx, 0)]
        last_step = [i for i, r in enumerate(tr) if r[0] == 4][-2:]                 # the step's begin and end markers
        recs = tr[last_step[0] + 1:last_step[1]]
        bubbles = [(t1 - t0) for kind, _, _, _, t0, t1 in recs if kind == 3]
        span = recs[-1][5] - recs[0][4]
        compute = span - sum(bubbles)
        want_total = (stages - 1) * compute / micro
        assert len(bubbles) == len(OB_bubbles(stage, stages, micro))
        assert 0.7 * want_total <= sum(bubbles) <= 1.3 * want_total, (sum(bubbles), want_total)


def OB_bubbles(stage, stages, micro):
    from oracle import bubbles as OB
    return OB.pp_1f1b_bubbles(stage, stages, micro, 1000, 2000)


@pytest.mark.parametrize("more", [0, 8, 808])
@pytest.mark.parametrize("vocab,blocks_per_cu", [(97, 16), (1000, 4), (5000, 3), (13000, 2)])
def test_cross_entropy_of_a_step_hands_out_its_rows(vocab, blocks_per_cu, more):
    """In a training step the blocks of the cross entropy take two rows each and get the others, where there are any, from a
    counter that is re-armed from step to step: as many rows as that, a few more, and many more, for every number of vectors per
    thread.  Gradient and loss have the bits of the same kernel without a counter on the same logits."""
    tokens = 2 * blocks_per_cu * torch.cuda.get_device_properties(0).multi_processor_count + more
    c = dict(n_layers=1, d_model=64, n_heads=1, d_head=64, d_ffn=128, vocab=vocab, max_pos=tokens // 8, batch=8, seq=tokens // 8)
    shape = decoder_shape(c)
    ld = (vocab + 63) // 64 * 64 if vocab >= 8192 else (vocab + 7) // 8 * 8
    ids, tg = i32(Y.token_ids(3, 8, c["seq"], vocab)), i32(Y.token_ids(4, 8, c["seq"], vocab))
    loss, rows, mean = torch.zeros(1, device=DEV), torch.zeros(tokens, device=DEV), torch.zeros(1, device=DEV)
    with Session() as s:
        s.register_training(shape, P.pack(shape, Y.decoder_params(1, c)), lr=0.0)
        for step in range(3):
            loss.zero_()
            torch.cuda.synchronize()
            s.step(ids, tg, loss)
            s.sync()
            got = s.train_tensor("logits").clone()
            wte = s.train_tensor("work")[:vocab * 64]
            logits = torch.zeros(tokens * ld, device=DEV, dtype=torch.bfloat16)
            S.sif_k_gemm_bf16(s.train_tensor("lnf"), wte, logits, tokens, vocab, 64, 64, 64, ld)
            S.sif_k_xent_fwd_bwd(logits, tg, rows, tokens, vocab, ld)
            S.sif_k_reduce_sum(rows, mean, tokens, 1.0 / tokens)
            torch.cuda.synchronize()
            assert torch.equal(got.view(torch.int16), logits.view(torch.int16)), step
            assert loss.item() == mean.item(), step
