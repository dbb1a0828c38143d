"""CPU-side checks of the library: it loads without a GPU, exports every symbol the header declares, and its
pure host functions (Bubble Monitor zero-count, Algorithm 1, Kernel Barrier rules, principles, bubble model)
agree with the scheduler oracle bit for bit."""
import itertools
import os
import re

import numpy as np
import pytest

import paper_2503_02550_amd as S
import synth_inputs as Y
from oracle import bubbles as OB
from oracle import scheduler as OK

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "specinf.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(sif_[a-z0-9_]+)\s*\(", header))
    assert len(declared) >= 50
    for name in sorted(declared):
        assert hasattr(S.lib, name), f"{name} declared in specinf.h but not exported"
    assert S.sif_abi_version() == 1


def test_zero_count_matches_oracle():
    rng = np.random.default_rng(0)
    for _ in range(300):
        w = [int(v) for v in rng.integers(0, 3, rng.integers(0, 12))]
        assert S.sif_zero_count(w) == OK.zero_count(w)


def test_alg1_matches_oracle_exhaustively():
    for alpha, beta, gn, gd, m, ll, ul, t0 in ((2, 5, 2, 1, 2, 8, 64, 1), (1, 3, 2, 1, 1, 100, 400, 25), (0, 2, 3, 2, 3, 7, 50, 2), (2, 2, 5, 4, 1, 9, 9, 4)):
        p = S.sif_alg1_params(alpha, beta, gn, gd, m, 0, ll, ul, t0)
        for trace in itertools.product(range(7), repeat=5):
            pool_c = pool_o = 0
            for zc in trace:
                pool_c, grant_c, st_c = S.sif_alg1_step(p, zc, pool_c)
                pool_o, grant_o, st_o = OK.alg1_step(zc, pool_o, alpha, beta, gn, gd, m, ll, ul, t0)
                assert (pool_c, grant_c, st_c) == (pool_o, grant_o, st_o)


def test_alg1_golden_table():
    rows = [tuple(map(int, l.split())) for l in open(os.path.join(ROOT, "tests", "golden", "alg1_worked_example.txt")) if l[0] != "#"]
    p = S.sif_alg1_params(2, 5, 2, 1, 2, 0, 8, 64, 1)
    pool = 0
    for zc, want_pool, want_grant, want_status in rows:
        pool, grant, status = S.sif_alg1_step(p, zc, pool)
        assert (pool, grant, status) == (want_pool, want_grant, want_status)


def test_alg1_rejects_bad_parameters():
    with pytest.raises(S.SifError):
        S.sif_alg1_step(S.sif_alg1_params(1, 2, 2, 1, 0, 0, 1, 2, 1), 3, 0)      # m = 0
    with pytest.raises(S.SifError):
        S.sif_alg1_step(S.sif_alg1_params(1, 2, 2, 0, 1, 0, 1, 2, 1), 3, 0)      # gamma_den = 0


def test_barrier_rules_and_principles_match_oracle():
    rng = np.random.default_rng(1)
    for _ in range(500):
        costs = [int(v) for v in rng.integers(0, 9, rng.integers(0, 8))]
        bal = int(rng.integers(0, 30))
        assert S.sif_kb_release(costs, bal) == OK.kb_release(costs, bal)
    for status, qlen, rem, req in itertools.product((0, 1), (0, 2), (0, 5, 10), (0, 5, 11)):
        assert S.sif_online_pull_ok(status, qlen, rem, req) == OK.online_pull_ok(status, qlen, rem, req)
    assert S.sif_principle_1([30, 9], 40) == OK.principle_1([30, 9], 40) == True
    assert S.sif_principle_1([30, 10], 40) == OK.principle_1([30, 10], 40) == False
    assert S.sif_principle_1([2 ** 63, 2 ** 63], 2 ** 64 - 1) is False           # overflow is a violation
    assert S.sif_principle_2(5, 6) and not S.sif_principle_2(6, 6)


def test_monitor_scheduler_barrier_chain_over_traces_matches_oracle():
    """The objects the monitor and barrier threads keep (window, Algorithm 1 state, token account), driven over count
    traces without a GPU, against the oracle's run over the same traces: Z_c, pool, grant, status and the number of
    kernels forwarded in every period; and from the C side's own outputs, the cost forwarded per period stays within
    that period's grant."""
    rng = np.random.default_rng(3)
    for case in range(300):
        alpha = int(rng.integers(0, 3)); beta = alpha + int(rng.integers(0, 4))
        gn, gd = [(2, 1), (3, 2), (5, 4), (1, 1), (3, 1)][int(rng.integers(0, 5))]
        m = int(rng.integers(1, 4))
        ll = int(rng.integers(1, 60)); ul = ll + int(rng.integers(0, 200)); t0 = int(rng.integers(1, 30))
        window = int(rng.integers(1, 12))
        n = int(rng.integers(1, 120))
        # training phases (counts > 0) and bubbles (runs of zero counts) of random lengths
        counts = []
        while len(counts) < n:
            counts += [int(v) for v in rng.integers(1, 5, rng.integers(1, 6))]
            counts += [0] * int(rng.integers(0, 15))
        counts = counts[:n]
        costs = [int(v) for v in rng.integers(0, max(2, ul // m + 3), rng.integers(0, 200))]
        p = S.sif_alg1_params(alpha, beta, gn, gd, m, 0, ll, ul, t0)
        got = S.sif_sched_run_trace(p, window, counts, costs)
        want = OK.run_trace(counts, costs, window, alpha, beta, gn, gd, m, ll, ul, t0)
        assert got == want, (case, alpha, beta, gn, gd, m, ll, ul, t0, window)
        head = 0
        for zc, pool, grant, status, nrel in got:
            assert sum(costs[head:head + nrel]) <= grant
            assert head + nrel == len(costs) or costs[head + nrel] > grant - sum(costs[head:head + nrel])   # the head blocks only when it must
            assert (pool == 0) == (zc <= alpha) and grant == pool // m and (status == OK.IDLE) == (zc > beta)
            head += nrel
    with pytest.raises(S.SifError):
        S.sif_sched_run_trace(S.sif_alg1_params(1, 2, 2, 1, 1, 0, 1, 2, 1), 0, [0], [1])                # window = 0


def test_kernel_charge_is_its_predicted_time_capped_by_the_largest_grant():
    for us, ul, m, want in ((7, 800, 1, 7), (800, 800, 1, 800), (801, 800, 1, 800), (500, 800, 2, 400), (3, 2, 4, 1), (0, 10, 1, 0),
                            (2 ** 40, 2 ** 50, 1, 2 ** 32 - 1)):
        assert S.sif_kb_charge(us, ul, m) == want, (us, ul, m)
    # a charged kernel can always be forwarded by a full grant of the stable phase
    for ul, m in ((800, 1), (800, 3), (5, 7)):
        grant = ul // m
        assert S.sif_kb_release([S.sif_kb_charge(10 ** 6, ul, m)], max(grant, 1))[0] == 1


def test_gate_violation_checker_on_synthetic_records():
    """The check behind sif_stats.gate_violations: a kernel start against the bubble's own begin / end stamps."""
    begin, end = 1_000_000, 1_500_000
    assert not S.sif_gate_violation(begin, begin, end) and not S.sif_gate_violation(end, begin, end)      # the stamps themselves are inside
    assert not S.sif_gate_violation(1_200_000, begin, end)
    assert S.sif_gate_violation(begin - 1, begin, end) and S.sif_gate_violation(end + 1, begin, end)
    assert not S.sif_gate_violation(2_000_000, begin, 0) and S.sif_gate_violation(999_999, begin, 0)       # bubble not over yet: only its begin binds
    rng = np.random.default_rng(11)
    for _ in range(2000):
        b0 = int(rng.integers(1, 2 ** 60)); b1 = b0 + int(rng.integers(0, 10 ** 7)); t = b0 + int(rng.integers(-10 ** 7, 2 * 10 ** 7))
        assert S.sif_gate_violation(max(t, 0), b0, b1) == (not (b0 <= max(t, 0) <= b1))


def test_latency_histogram_buckets_and_percentiles():
    nb = S.sif_latency_buckets()
    lows = [S.sif_latency_bucket_lower_ns(b) for b in range(nb)]
    assert lows[0] == 0 and all(b > a for a, b in zip(lows, lows[1:]))
    for b in range(nb):
        assert S.sif_latency_bucket(lows[b]) == b
        if b + 1 < nb:
            assert S.sif_latency_bucket(lows[b + 1] - 1) == b
            assert lows[b + 1] - lows[b] <= max(1, lows[b] // 16)                  # at most 1/16 wider than its lower edge
    assert S.sif_latency_bucket(2 ** 64 - 1) == nb - 1
    rng = np.random.default_rng(12)
    for trial in range(20):
        lat = np.exp(rng.normal(15.5, 0.8, int(rng.integers(1, 4000)))).astype(np.int64)      # milliseconds, log-normal
        counts = [0] * nb
        for v in lat:
            counts[S.sif_latency_bucket(int(v))] += 1
        srt = np.sort(lat)
        for p in (0.5, 0.95, 0.99, 1.0):
            exact = int(srt[int(np.ceil(p * len(srt))) - 1])                       # nearest rank
            got = S.sif_latency_percentile(counts, p)
            assert S.sif_latency_bucket(got) == S.sif_latency_bucket(exact)
            assert abs(got - exact) <= exact / 32 + 1
    assert S.sif_latency_percentile([0] * nb, 0.5) == 0


def test_bubble_model_matches_oracle():
    from oracle.decoder import n_params
    n = n_params(Y.DP_DECODER)
    assert S.sif_collective_ns(2 * n, 50_000_000_000) == OB.dp_bubbles(n, 2, 50_000_000_000)[0][1] == 4_977_592
    c = Y.TP_DECODER
    assert S.sif_collective_ns(c["batch"] * c["seq"] * c["d_model"] * 2, c["bw_bytes_per_s"]) == OB.tp_bubbles(1, c["batch"] * c["seq"], c["d_model"], 2, c["bw_bytes_per_s"])[0][1]
    assert S.sif_collective_ns(2 ** 62, 10 ** 12) == (2 ** 62 * 10 ** 9) // 10 ** 12                # the product passes 2^64: 128-bit intermediate
    kinds = {0: "F", 1: "B"}
    for p, m, tf, tb in ((4, 8, 100, 200), (3, 3, 5, 5), (2, 6, 11, 30), (5, 9, 3, 8)):
        for s in range(p):
            got = S.sif_pp_1f1b_bubbles(s, p, m, tf, tb)
            want = OB.pp_1f1b_bubbles(s, p, m, tf, tb)
            conv = [((("before", (kinds[k], i)) if k < 2 else ("end", None)), ns) for k, i, ns in got]
            assert conv == want
    with pytest.raises(S.SifError):
        S.sif_pp_1f1b_bubbles(4, 4, 8, 1, 1)
    with pytest.raises(S.SifError):
        S.sif_pp_1f1b_bubbles(0, 4, 3, 1, 1)


def test_bucketed_gradient_exchange_matches_oracle():
    rng = np.random.default_rng(5)
    for _ in range(200):
        n = int(rng.integers(0, 9))
        sizes = [int(v) for v in rng.integers(1, 60, n)]
        cap = int(rng.integers(1, 90))
        nb, of = S.sif_dp_gradient_buckets(sizes, cap)
        want = OB.dp_gradient_buckets(sizes, cap)
        assert nb == len(want)
        assert of == [b for b, grp in enumerate(want) for _ in grp]
        ready = sorted(int(v) for v in rng.integers(0, 10 ** 7, n))
        dur = [int(v) for v in rng.integers(0, 10 ** 6, n)]
        end = (ready[-1] if n else 0) + int(rng.integers(0, 10 ** 5))
        assert S.sif_dp_overlapped_wait(ready, dur, end) == OB.dp_overlapped_wait(ready, dur, end)
    with pytest.raises(S.SifError):
        S.sif_dp_gradient_buckets([1, 2], 0)


def test_feedback_rules_match_oracle():
    from oracle import scheduler as OKS
    rng = np.random.default_rng(9)
    for _ in range(3000):
        share = int(rng.integers(0, 1_000_001))
        ref = int(rng.integers(1, 2 ** 40))
        step = int(ref * (1 + rng.uniform(-0.1, 0.1))) if rng.random() < 0.8 else int(rng.integers(1, 2 ** 40))
        eps, add, cap = int(rng.integers(0, 200_000)), int(rng.integers(0, 300_000)), int(rng.integers(0, 1_000_001))
        assert S.sif_feedback_share(share, step, ref, eps, add, cap) == OKS.feedback_share(share, step, ref, eps, add, cap)
        bal, period, burst = int(rng.integers(0, 10 ** 9)), int(rng.integers(1, 10 ** 7)), int(rng.integers(0, 10 ** 9))
        assert S.sif_concurrent_account(bal, share, period, burst) == OKS.concurrent_account(bal, share, period, burst)
    # the threshold itself is "not lengthened", one nanosecond more is
    assert S.sif_feedback_share(400_000, 1_020_000, 1_000_000, 20_000, 0, 1_000_000) == 400_000
    assert S.sif_feedback_share(400_000, 1_020_001, 1_000_000, 20_000, 0, 1_000_000) == 200_000
    # products beyond 64 bits
    assert S.sif_feedback_share(10, 2 ** 63, 2 ** 63 - 1, 0, 5, 100) == OKS.feedback_share(10, 2 ** 63, 2 ** 63 - 1, 0, 5, 100) == 5


def test_param_layout_counts():
    from paper_2503_02550_amd import params as P
    from paper_2503_02550_amd.session import decoder_shape, encoder_shape, mlp_shape
    from oracle.decoder import n_params
    assert S.sif_model_n_params(decoder_shape(Y.DP_DECODER)) == n_params(Y.DP_DECODER) == 124_439_808
    assert S.sif_model_n_params(decoder_shape(Y.TP_DECODER)) == n_params(Y.TP_DECODER)
    assert S.sif_model_n_params(mlp_shape(256, 256, 256, 32)) == 2 * 256 * 256 + 512
    for shape in (decoder_shape(Y.DP_DECODER), encoder_shape(Y.FILL_ENCODER)):
        assert sum(int(np.prod(s)) for _, s in P.layout(shape)) == S.sif_model_n_params(shape)


def test_default_config_and_sizes():
    cfg = S.sif_default_config()
    assert cfg.period_us == 5 and cfg.alg1.alpha <= cfg.alg1.beta and cfg.alg1.ll <= cfg.alg1.ul
    assert S.sif_ctx_workspace_bytes() > 2 * 65536 * 32


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU; asked for more it must say so and exit with an error before touching a device."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in (r.stdout + r.stderr)


@pytest.mark.parametrize("d,f,tokens", [(64, 256, 1024), (128, 512, 2048), (256, 1024, 4096), (384, 1536, 512), (128, 512, 16384)])
def test_group_of_a_small_layer_is_not_put_on_tall_tiles(d, f, tokens):
    """The weight gradients of a small layer are few tiles and one long K: on tiles twice as tall they keep half as many
    CUs busy with the same chain of K steps."""
    from tile_choice import group
    shapes = [(d, f), (f, d), (d, d), (3 * d, d), (1, f), (1, 3 * d)]
    lay = dict(a_layout=S.SIF_A_ROW_M, b_layout=S.SIF_B_ROW_N)
    tiles, name = group([S.gemm_args(1 << 20, 1 << 20, 1 << 20, m, n, tokens, (m + 7) // 8 * 8, n, n, **lay) for m, n in shapes])
    up = lambda v, by: (v + by - 1) // by
    assert name == "128x128 one" and tiles == sum(up(up(m, 128) * up(n, 128), 8) * 8 for m, n in shapes)


@pytest.mark.parametrize("m,n,ring,fetching", [(32, 768, "32x64", "32x32"), (77, 3072, "32x64", "32x64"), (1000, 768, "64x64", "64x64"), (1024, 1024, "64x64", "64x64")])
def test_products_of_one_k_step_run_on_the_ring(m, n, ring, fetching):
    """Wavefronts that only fetch have nothing to keep in flight for a single K step, and their larger blocks start later."""
    from tile_choice import kernel
    args = lambda k: S.gemm_args(1 << 20, 1 << 20, 1 << 20, m, n, k, 128, 128, n)
    assert [kernel(args(k)) for k in (8, 64)] == [ring] * 2
    assert [kernel(args(k)) for k in (72, 128)] == ["fetching " + fetching] * 2


@pytest.mark.parametrize("tokens", [4096, 8192, 8200])
def test_group_counts_the_tiles_of_the_fullest_xcd(tokens):
    """85 + 85 + 20 + 60 tiles of 128x128 are fewer than the chip has CUs, but every product begins at the first XCD, which gets 11
    + 11 + 3 + 8 of them for its 32 CUs: no single round.  The one-row products stay in the launch, which is one on taller tiles."""
    from tile_choice import group, part
    lay = dict(a_layout=S.SIF_A_ROW_M, b_layout=S.SIF_B_ROW_N)
    d, da, f = 520, 512, 2056
    list_ = [S.gemm_args(1 << 20, 1 << 20, 1 << 20, m, n, tokens, (m + 7) // 8 * 8, n, n, **lay) for m, n in ((d, f), (f, d), (d, da), (3 * da, d), (1, f), (1, 3 * da))]
    assert group(list_[:4])[1] != "128x128 one"
    assert part(list_, 4) == 6 and group(list_)[1] == "256x128"


@pytest.mark.parametrize("d,da,f,tokens,apart", [(2048, 2048, 8192, 4096, True), (1984, 1984, 7936, 2048, True), (1920, 1920, 7680, 1024, True), (2048, 2048, 8192, 256, False),
                                                 (1984, 1984, 7936, 512, False), (816, 1408, 5520, 8192, False), (776, 1280, 5360, 4096, False), (488, 1408, 4288, 2048, False)])
def test_one_row_products_leave_a_group_only_for_more_than_the_models_error(d, da, f, tokens, apart):
    """Layers where the one-row products as launches of their own were measured to be faster, and ones where the model sees a
    small gain and they were measured to be slower."""
    from tile_choice import part
    lay = dict(a_layout=S.SIF_A_ROW_M, b_layout=S.SIF_B_ROW_N)
    list_ = [S.gemm_args(1 << 20, 1 << 20, 1 << 20, m, n, tokens, (m + 7) // 8 * 8, n, n, **lay) for m, n in ((d, f), (f, d), (d, da), (3 * da, d), (1, f), (1, 3 * da))]
    assert part(list_, 4) == (4 if apart else 6)
