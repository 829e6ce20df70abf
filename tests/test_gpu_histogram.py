"""GPU checks of the histogram stage by itself (Eq. 6-9, App. C.3, Prop. 1) - the threshold parity
tests alone would not see a wrong bin, window move or closed-form root, because the safeguarded
refinement repairs a bad start - and metamorphic checks of the whole path that need no oracle."""
import numpy as np
import pytest
import torch

import workloads
from tests import list_replay, parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ea():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_15180_amd as ea
    ea.lib()
    return ea


def grid_histogram_root(x, alpha, nb):
    """Float64 root of f_h (Eq. 9) for one row of pre-scaled scores x = (alpha-1) s, with the bins the
    GPU uses: width h = 1/nb on an absolute grid (bin a holds nb x in [a, a+1)), of which the nb + 1
    bins up to the one holding the maximum are kept.  Returns (tau_h, max x)."""
    h, r = 1.0 / nb, 1.0 / (alpha - 1.0)
    m = x.max()
    top = int(np.floor(nb * m))
    a = np.floor(nb * x).astype(np.int64)
    keep = a >= top - nb
    edges, counts = np.unique(a[keep], return_counts=True)
    e = edges.astype(np.float64) * h

    def f(tau):
        y = np.maximum(e - tau, 0.0)
        return float((counts * y ** r).sum() - 1.0)

    lo, hi = e.max() - 1.0 - 2 * h, e.max()        # f(lo) >= 0: the top bin alone weighs (1 + 2h)^r there; f(hi) = -1
    for _ in range(80):
        mid = 0.5 * (lo + hi)
        if f(mid) >= 0:
            lo = mid
        else:
            hi = mid
    return 0.5 * (lo + hi), m


CASES = [("bf16", 64, 1.5, "gauss", 2.0, True), ("bf16", 128, 1.5, "gauss", 1.0, True), ("bf16", 128, 2.0, "gauss", 3.0, False),
         ("bf16", 64, 1.25, "gauss", 2.0, True), ("f32", 64, 1.5, "gauss", 1.0, False), ("bf16", 64, 1.5, "ramp", 0.25, True),
         ("bf16", 64, 1.5, "ramp", 2.5, False), ("bf16", 64, 1.5, "flat", 0.3, True), ("f32", 64, 2.0, "flat", 0.3, True)]


@pytest.mark.parametrize("dtype,d,alpha,kind,scale,causal", CASES)
def test_histogram_root_brackets_the_threshold(ea, dtype, d, alpha, kind, scale, causal):
    # Prop. 1 on what the kernels' histogram stage produced: tau_0 <= tau* <= upper, upper - tau_0 <= 1/B
    # (+ rounding slack), and tau_0 equal to the float64 root of the same histogram.  Flat inputs
    # overflow the candidate lists of the long rows, which the sweep-based kernel then redoes.
    from oracle import entmax_oracle as eo
    B, H, N = 1, 2, (2048 if kind == "flat" else 640)
    print(f"histogram case {dtype} d={d} alpha={alpha} {kind} {scale} causal={causal}", flush=True)
    if kind == "ramp":
        q, k, v, _ = workloads.ramp_qkv(B, H, N, d, dtype, scale, seed=41)
    else:
        q, k, v, _ = workloads.gaussian_qkv(B, H, N, d, dtype, scale, seed=43)
    ws = torch.empty(ea.entmax_attn_workspace_bytes(B, H, N, d, dtype, causal, False), dtype=torch.uint8, device="cuda")
    O, tau, mask, iters = ea.entmax_attn_fwd(q.cuda(), k.cuda(), v.cuda(), alpha, causal, want_iters=True, workspace=ws)
    tau0, upper = ea.entmax_attn_fwd_histogram_bounds(ws, B, H, N, d, dtype)
    torch.cuda.synchronize()
    if kind == "flat" and alpha == 1.5:
        assert ea.read_stats(ws)["list_overflow_blocks"] > 0
    nb = ea.entmax_attn_histogram_bins()
    ref = eo.attn_fwd(parity.to_np64(q), parity.to_np64(k), parity.to_np64(v), alpha, causal, want_margin=False)
    t0, up, tg = (parity.to_np64(t) for t in (tau0, upper, tau))
    ts = ref["tau"]
    eps = 3e-5 * (1.0 + np.abs(ts))            # fp32 scores and sums against float64
    assert (t0 <= ts + eps).all(), f"tau_0 above the true threshold by {(t0 - ts).max():.3e}"
    assert (ts <= up + eps).all(), f"true threshold above the bracket by {(ts - up).max():.3e}"
    assert (up - t0 <= 1.0 / nb + 1e-4).all(), f"bracket wider than 1/B: {(up - t0).max():.3e}"
    assert (tg >= t0 - eps).all() and (tg <= up + eps).all()
    # the root itself, against float64 on the same bins
    Qn, Kn = parity.to_np64(q), parity.to_np64(k)
    want = np.empty_like(ts)
    for h_ in range(H):
        X = (alpha - 1.0) * (Qn[0, h_] @ Kn[0, h_].T) / np.sqrt(d)
        for r_ in range(N):
            x = X[r_, : r_ + 1] if causal else X[r_]
            th, m = grid_histogram_root(x, alpha, nb)
            want[0, h_, r_] = max(th, m - 1.0)
    diff = np.abs(t0 - want)
    close = (diff <= 1e-4 * (1.0 + np.abs(want))).mean()
    print(f"  tau_0 within 1e-4 of the float64 root of the same bins on {100 * close:.2f} % of the rows; max {diff.max():.3e};"
          f" tau* - tau_0 mean {np.mean(ts - t0):.4f}; mean iters {iters.float().mean().item():.2f}", flush=True)
    # a score that fp32 puts on the other side of a bin edge moves one count by one bin
    assert close >= 0.995 and diff.max() <= 1.0 / nb + 1e-4


def test_shifting_every_key_by_one_vector(ea):
    # K <- K + 1 c^T adds q_r . c / sqrt(d) to every score of row r: P, O and every gradient stay,
    # tau_r moves by (alpha - 1) q_r . c / sqrt(d)   (fp32 path; shift invariance of Eq. 3)
    B, H, N, d, alpha = 1, 2, 512, 64, 1.5
    for causal in (False, True):
        q, k, v, do = workloads.gaussian_qkv(B, H, N, d, "f32", 1.0, seed=51)
        g = torch.Generator().manual_seed(52)
        c = 0.5 * torch.randn(d, generator=g)
        Q, K, V, dO = (t.cuda() for t in (q, k, v, do))
        K2 = (k + c).cuda()
        O, tau, mask = ea.entmax_attn_fwd(Q, K, V, alpha, causal)
        O2, tau2, mask2 = ea.entmax_attn_fwd(Q, K2, V, alpha, causal)
        g1 = ea.entmax_attn_bwd(Q, K, V, O, dO, tau, alpha, causal, block_mask=mask)
        g2 = ea.entmax_attn_bwd(Q, K2, V, O2, dO, tau2, alpha, causal, block_mask=mask2)
        torch.cuda.synchronize()
        shift = (alpha - 1.0) * (q.double() @ c.double()) / d ** 0.5
        assert (tau2.double().cpu() - tau.double().cpu() - shift).abs().max().item() <= 2e-5
        assert (O2 - O).abs().max().item() <= 2e-5
        assert (mask2 != mask).sum().item() <= 2          # (a tile whose largest probability is about 1e-6 may flip)
        for name, a, b in zip(("dQ", "dK", "dV"), g1, g2):
            err = ((a - b).abs() / (1 + a.abs())).max().item()
            assert err <= 5e-5, f"{name} moved by {err:.3e} (causal={causal})"


def test_permuting_key_tiles(ea):
    # not causal: whole 64-key tiles of K and V in another order leave O, tau and dQ as they are and
    # move the rows of dK, dV and the bits of the mask the same way
    B, H, N, d, alpha = 1, 2, 768, 64, 1.5
    T = N // 64
    q, k, v, do = workloads.gaussian_qkv(B, H, N, d, "f32", 1.5, seed=61)
    perm = torch.randperm(T, generator=torch.Generator().manual_seed(62))
    idx = (perm[:, None] * 64 + torch.arange(64)[None, :]).reshape(-1)        # new position p holds old key idx[p]
    Q, K, V, dO = (t.cuda() for t in (q, k, v, do))
    K2, V2 = k[:, :, idx].contiguous().cuda(), v[:, :, idx].contiguous().cuda()
    O, tau, mask = ea.entmax_attn_fwd(Q, K, V, alpha, False)
    O2, tau2, mask2 = ea.entmax_attn_fwd(Q, K2, V2, alpha, False)
    dQ, dK, dV = ea.entmax_attn_bwd(Q, K, V, O, dO, tau, alpha, False, block_mask=mask)
    dQ2, dK2, dV2 = ea.entmax_attn_bwd(Q, K2, V2, O2, dO, tau2, alpha, False, block_mask=mask2)
    torch.cuda.synchronize()
    assert (tau2 - tau).abs().max().item() <= 1e-5 and (O2 - O).abs().max().item() <= 2e-5
    assert ((dQ2 - dQ).abs() / (1 + dQ.abs())).max().item() <= 5e-5
    idx_c = idx.cuda()
    assert ((dK2 - dK[:, :, idx_c]).abs() / (1 + dK2.abs())).max().item() <= 5e-5
    assert ((dV2 - dV[:, :, idx_c]).abs() / (1 + dV2.abs())).max().item() <= 5e-5
    bits, bits2 = parity.unpack_mask(mask, T), parity.unpack_mask(mask2, T)
    assert (bits2 != bits[..., perm.numpy()]).sum() <= 2


@pytest.mark.parametrize("dtype,d,alpha,sigma,causal,N", [("bf16", 128, 1.5, 2.0, True, 1024), ("bf16", 64, 2.0, 2.0, False, 640),
                                                       ("f32", 64, 1.25, 1.0, True, 320), ("bf16", 64, 3.0, 2.0, True, 640),
                                                       ("bf16", 64, 1.5, 0.3, True, 2048), ("bf16", 128, 1.5, 4.0, True, 1024)])
def test_right_edge_binning_gives_a_sparser_approximation(ea, dtype, d, alpha, sigma, causal, N):
    # The approximate forward (Sec. 3.2, binning strategies): thresholds are the right-edge histogram
    # roots, unrefined.  Asserted: what defines the mode - tau* <= tau < tau* + h + slack against the
    # oracle's tau*, one evaluation per row, rows of P summing to at most 1, and O = P(tau) V for
    # the tau returned (float64, from the same inputs).  Its distance from the exact result is
    # printed, not asserted: the mode is not meant to reach it.  sigma = 0.3 overflows the candidate
    # lists (the sweep-based kernel), sigma = 4 takes the gather path.
    from oracle import entmax_oracle as eo
    B, H = 1, 2
    print(f"right-edge case N={N} d={d} {dtype} alpha={alpha} sigma={sigma} causal={causal}", flush=True)
    q, k, v, _ = workloads.gaussian_qkv(B, H, N, d, dtype, sigma, seed=77)
    Q, K, V = (t.cuda() for t in (q, k, v))
    ea.entmax_attn_right_edge_enable(True)
    try:
        O, tau, mask, iters = ea.entmax_attn_fwd(Q, K, V, alpha, causal, want_iters=True)
        torch.cuda.synchronize()
    finally:
        ea.entmax_attn_right_edge_enable(False)
    O2, tau2, mask2 = ea.entmax_attn_fwd(Q, K, V, alpha, causal)          # and the switch is off again
    torch.cuda.synchronize()
    ref = eo.attn_fwd(*(parity.to_np64(t) for t in (q, k, v)), alpha, causal, tile=64)
    parity.check_forward(q, k, v, alpha, causal, O2, tau2, mask2, ref=ref, label="exact mode after the approximate one")
    h = 1.0 / ea.entmax_attn_histogram_bins()
    t, ts = parity.to_np64(tau), ref["tau"]
    slack = 2e-6 * (1 + np.abs(ts))
    assert (t >= ts - slack).all() and (t <= ts + h + 2 * slack).all(), ((t - ts).min(), (t - ts).max())
    assert (iters.cpu().numpy() == 1).all()
    Qn, Kn, Vn = (parity.to_np64(x) for x in (q, k, v))
    r = 1.0 / (alpha - 1.0)
    worst_o, sums = 0.0, []
    for hh in range(H):
        X = (alpha - 1.0) * Qn[0, hh] @ Kn[0, hh].T / np.sqrt(d)
        if causal:
            X = np.where(np.tril(np.ones((N, N), bool)), X, -np.inf)
        P = np.maximum(X - t[0, hh][:, None], 0.0) ** r
        sums.append(P.sum(-1))
        worst_o = max(worst_o, np.abs(P @ Vn[0, hh] - parity.to_np64(O)[0, hh]).max())
    sums = np.concatenate(sums)
    assert sums.max() <= 1 + 1e-3
    assert worst_o <= parity.TOL[q.dtype]["O"], worst_o
    # block mask: every tile it marks is marked in the exact result (support inside the true one)
    T = N // 64
    got, exact = parity.unpack_mask(mask, T), parity.unpack_mask(mask2, T)
    assert not (got & ~exact).any()
    print("  right edge:", dict(tau_above=float((t - ts).mean()), row_sum_mean=float(sums.mean()), row_sum_min=float(sums.min()),
                               dO_vs_exact=float(np.abs(parity.to_np64(O) - ref["O"]).max()),
                               tiles=int(got.sum()), tiles_exact=int(exact.sum())), flush=True)


@pytest.mark.parametrize("dtype,d,alpha,scale,causal", [("bf16", 64, 1.1, 2.0, True), ("bf16", 128, 1.4, 1.0, False), ("bf16", 64, 1.6, 1.0, True),
                                                        ("bf16", 128, 1.75, 3.0, True), ("f32", 64, 1.75, 1.0, False), ("bf16", 64, 2.5, 2.0, True)])
def test_histogram_root_from_each_closed_form_bound(ea, dtype, d, alpha, scale, causal):
    # the scan's closed-form bound by 1/(alpha-1): power means from 2 on, the square below, the plain sum below 1
    # - the refined bound while the sweep runs, and where the Newton solve of the full histogram starts
    test_histogram_root_brackets_the_threshold(ea, dtype, d, alpha, "gauss", scale, causal)


@pytest.mark.parametrize("dtype,d,alpha,scale,causal", [("bf16", 64, 1.5, 0.45, False), ("bf16", 64, 1.5, 0.6, False), ("bf16", 128, 1.5, 0.6, True),
                                                        ("bf16", 128, 1.25, 0.8, False), ("bf16", 64, 2.0, 0.3, False), ("f32", 64, 1.5, 0.6, False)])
def test_histogram_of_long_lists(ea, dtype, d, alpha, scale, causal):
    # supports of one to several hundred keys: lists that are counted as they grow, pruned at a refresh of the bound, or full
    test_histogram_root_brackets_the_threshold(ea, dtype, d, alpha, "gauss", scale, causal)


@pytest.mark.parametrize("dtype,d,alpha,scale", [("bf16", 64, 1.01, 3.0), ("bf16", 128, 1.03, 3.0)])
def test_histogram_root_for_alpha_near_one(ea, dtype, d, alpha, scale):
    # where the closed-form bound lies many bins below the root (see tests/host/histogram_main.cpp)
    test_histogram_root_brackets_the_threshold(ea, dtype, d, alpha, "gauss", scale, True)


@pytest.mark.parametrize("dtype,d,alpha,causal", [("bf16", 64, 1.5, True), ("bf16", 128, 1.5, False), ("bf16", 64, 2.0, False),
                                                  ("bf16", 128, 1.25, False), ("f32", 64, 1.5, True)])
def test_histogram_of_rising_maxima(ea, dtype, d, alpha, causal):
    # keys grow along the sequence, so the maximum of nearly every row rises with every tile and the window of
    # bins keeps moving, with the bins kept spare above it taken up in between; queries grow from 32-row block to block,
    # so that some waves count their lists' entries from the first tile, some once a list has grown, some only at the end
    from oracle import entmax_oracle as eo
    B, H, N = 1, 1, 1472
    q, k, v, _ = workloads.gaussian_qkv(B, H, N, d, dtype, 1.0, seed=53)
    block = torch.arange(N) // 32
    q = (q.float() * torch.linspace(0.5, 3.5, 8)[block % 8][None, None, :, None]).to(q.dtype)
    k = (k.float() * torch.linspace(0.6, 1.4, N)[None, None, :, None]).to(k.dtype)
    ws = torch.empty(ea.entmax_attn_workspace_bytes(B, H, N, d, dtype, causal, False), dtype=torch.uint8, device="cuda")
    O, tau, mask = ea.entmax_attn_fwd(q.cuda(), k.cuda(), v.cuda(), alpha, causal, workspace=ws)
    tau0, upper = ea.entmax_attn_fwd_histogram_bounds(ws, B, H, N, d, dtype)
    torch.cuda.synchronize()
    Qn, Kn = parity.to_np64(q), parity.to_np64(k)
    ref = eo.attn_fwd(Qn, Kn, parity.to_np64(v), alpha, causal, tile=64)
    parity.check_forward(q, k, v, alpha, causal, O, tau, mask, ref=ref, label=f"rising maxima {dtype} {d} {alpha}")
    t0, up, ts = parity.to_np64(tau0), parity.to_np64(upper), ref["tau"]
    eps, nb = 3e-5 * (1.0 + np.abs(ts)), ea.entmax_attn_histogram_bins()
    assert (t0 <= ts + eps).all() and (ts <= up + eps).all() and (up - t0 <= 1.0 / nb + 1e-4).all()
    X = (alpha - 1.0) * (Qn[0, 0] @ Kn[0, 0].T) / np.sqrt(d)
    want = np.empty(N)
    for r_ in range(N):
        th, m = grid_histogram_root(X[r_, : r_ + 1] if causal else X[r_], alpha, nb)
        want[r_] = max(th, m - 1.0)
    diff = np.abs(t0[0, 0] - want)
    # a score that fp32 puts on the other side of a bin edge moves one count by one bin
    assert (diff <= 1e-4 * (1.0 + np.abs(want))).mean() >= 0.995 and diff.max() <= 1.0 / nb + 1e-4


def rising_root_scores():
    """Scores (alpha = 1.5) of one row whose threshold rises through a single histogram bin in 232 steps: 24 keys in the top bin put the
    root 12.86 bins below it, and each step's key, two bins above the root, raises it by a few hundredths of a bin.  All other
    keys lie just above the root of their step: each is listed, and dropped by the next prune.  Steps are as long
    as the two lists of the row have room for (n kept entries per list, 64 or so more in each pair of tiles)."""
    nb = 63.0
    key = np.arange(64)
    halves = [key[(key >> 3) & 1 == s] for s in (0, 1)]

    def root(n):                                     # 24 (0 - tau)^2 + n (-11/63 - tau)^2 = 1
        a, b, c = 24.0 + n, 2 * n * 11 / nb, n * (11 / nb) ** 2 - 1.0
        return (-b - np.sqrt(b * b - 4 * a * c)) / (2 * a)

    top = np.full(64, -3.0)
    top[np.concatenate([s[:12] for s in halves])] = 0.5 / nb
    tiles, kept = [top, np.full(64, -3.0)], 12
    for n in range(232):
        pairs = 3 if kept + 192 <= 256 else 2
        step = np.full((2 * pairs, 64), root(n) + 1e-5)
        step[-1, halves[n & 1][5]] = -10.5 / nb
        tiles.extend(step)
        kept = 12 + (n + 2) // 2
    return np.concatenate(tiles)


def test_counters_of_pruned_lists_do_not_overflow(ea):
    # A prune drops entries that stay counted, so a row's counters can take in far more than its lists ever hold at once.  Rows
    # 0 - 31 would put 72000 keys into one bin if their lists were pruned at every chance; their 16-bit counters lie beside those of
    # rows 32 - 63, whose two keys of support a carry would hide: the carry lands five bins below their maximum.
    alpha, nb, d = 1.5, ea.entmax_attn_histogram_bins(), 64
    x = rising_root_scores()
    N = x.size
    print(f"counters of pruned lists, N={N}", flush=True)
    freely = list_replay.replay_wave(np.broadcast_to(x, (32, N)), alpha, nb, MAX_PRUNES=1 << 30)
    assert freely["max_count"] > 65536 and not freely["overflow"], freely
    assert list_replay.replay_wave(np.broadcast_to(x, (32, N)), alpha, nb)["max_count"] < 65536
    other = np.full(N, -3.0)
    other[20], other[N - 10] = (51 + 5.5) / nb, (51 + 5.5) / nb - 0.9
    # the scores as sums of three bf16 parts each, which the queries' ones pick: x = (alpha - 1) <q, k> / 8 with q = 16
    k, q = torch.zeros(N, d), torch.zeros(N, d)
    for first, scores in ((0, x), (3, other)):
        left = torch.from_numpy(scores).clone()
        for i in range(3):
            k[:, first + i] = left.to(torch.bfloat16).float()
            left -= k[:, first + i].double()
    k[7, 6] = 4.0
    q[:32, 0:3], q[32:64, 3:6], q[64:, 6] = 16.0, 16.0, 16.0
    v = torch.randn(N, d, generator=torch.Generator().manual_seed(3))
    q, k, v = (t.to(torch.bfloat16)[None, None] for t in (q, k, v))
    ws = torch.empty(ea.entmax_attn_workspace_bytes(1, 1, N, d, "bf16", False, False), dtype=torch.uint8, device="cuda")
    O, tau, _ = ea.entmax_attn_fwd(q.cuda(), k.cuda(), v.cuda(), alpha, False, workspace=ws)
    tau0, upper = ea.entmax_attn_fwd_histogram_bounds(ws, 1, 1, N, d, "bf16")
    torch.cuda.synchronize()
    X = parity.to_np64(k)[0, 0, :, :6] @ np.repeat(np.eye(2), 3, 0)
    for rows, scores in ((slice(0, 32), X[:, 0]), (slice(32, 64), X[:, 1])):
        lo, hi = scores.max() - 1.0, scores.max()
        for _ in range(60):
            mid = 0.5 * (lo + hi)
            lo, hi = (mid, hi) if (np.maximum(scores - mid, 0.0) ** 2).sum() >= 1.0 else (lo, mid)
        P = np.maximum(scores - lo, 0.0) ** 2
        t0, up, t, o = (parity.to_np64(a)[0, 0, rows] for a in (tau0, upper, tau, O))
        print("  tau*", lo, "tau_0", t0.min(), t0.max(), "upper", up.min(), up.max(), flush=True)
        assert (t0 <= lo + 3e-5).all() and (lo <= up + 3e-5).all() and (up - t0 <= 1.0 / nb + 1e-4).all()
        assert np.abs(t - lo).max() <= parity.TOL[torch.bfloat16]["tau"] and np.abs(o - P @ parity.to_np64(v)[0, 0]).max() <= parity.TOL[torch.bfloat16]["O"]


@pytest.mark.parametrize("dtype,d,alpha,scale", [("bf16", 64, 1.5, 0.3), ("bf16", 128, 1.25, 0.6), ("f32", 64, 1.5, 0.3)])
def test_walks_whose_lists_overflowed_end_early(ea, dtype, d, alpha, scale):
    # Flat attention without a mask: every row has more keys of support than its lists hold.  A wave whose list overflowed has nothing more
    # to list: it works on about the same number of tiles at 1024 and at 2048 tokens, on 10 of 16 and of 32.  (The fallback kernel works
    # on every tile the same number of times, so per tile of the scores the counter falls by the list kernel's share.)
    B, H, seen = 1, 2, {}
    for N in (1024, 2048):
        print(f"overflowed lists {dtype} d={d} alpha={alpha} N={N}", flush=True)
        q, k, v, _ = workloads.gaussian_qkv(B, H, N, d, dtype, scale, seed=47)
        ws = torch.empty(ea.entmax_attn_workspace_bytes(B, H, N, d, dtype, False, False), dtype=torch.uint8, device="cuda")
        O, tau, mask = ea.entmax_attn_fwd(q.cuda(), k.cuda(), v.cuda(), alpha, False, workspace=ws)
        torch.cuda.synchronize()
        st = ea.read_stats(ws)
        seen[N] = st["tau_subtiles"] / (B * H * (N / 32) * (N / 64))
        print("  tiles", seen[N], "overflow", st["list_overflow_blocks"], flush=True)
        assert st["list_overflow_blocks"] == B * H * N // 64
        parity.check_forward(q, k, v, alpha, False, O, tau, mask, label=f"overflowed lists N={N}")
    assert seen[1024] - seen[2048] > 0.25


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64)])
def test_lists_that_are_pruned_or_nearly_full(ea, dtype, d):
    # 64-row blocks of eight kinds: four spreads of the scores, and a first tile like the others, so that list entries are counted as they
    # are listed, or one with two keys near the maximum and the rest far below, so that the lists are counted at a refresh.  Which
    # branches the lists go through is asked of the replay: pruned (some to an odd length, where the count resumes in the middle of
    # a load), walked on where the next tiles may fill them, and full, in both modes.
    from oracle import entmax_oracle as eo
    B, H, N, alpha = 1, 1, 2048, 1.5
    print(f"pruned and nearly full lists {dtype} d={d}", flush=True)
    q, k, v, _ = workloads.gaussian_qkv(B, H, N, d, "f32", 1.0, seed=61)
    block = torch.arange(N) // 64
    q *= torch.tensor([0.1, 0.2, 0.3, 0.35])[block % 4][None, None, :, None]
    q[..., 0] = torch.where(block // 4 % 2 == 0, 16.0, 0.0)
    k[..., 0], k[:, :, :64, 0] = 0.0, -4.0
    k[:, :, 5, 0] = k[:, :, 13, 0] = 0.0
    q, k, v = (t.to(torch.bfloat16 if dtype == "bf16" else torch.float32) for t in (q, k, v))
    ws = torch.empty(ea.entmax_attn_workspace_bytes(B, H, N, d, dtype, False, False), dtype=torch.uint8, device="cuda")
    O, tau, mask = ea.entmax_attn_fwd(q.cuda(), k.cuda(), v.cuda(), alpha, False, workspace=ws)
    tau0, upper = ea.entmax_attn_fwd_histogram_bounds(ws, B, H, N, d, dtype)
    torch.cuda.synchronize()
    nb = ea.entmax_attn_histogram_bins()
    Qn, Kn = parity.to_np64(q), parity.to_np64(k)
    X = (alpha - 1.0) * (Qn[0, 0] @ Kn[0, 0].T) / np.sqrt(d)
    waves = [list_replay.replay_wave(X[w:w + 32], alpha, nb) for w in range(0, N, 32)]
    longest = [max(a["longest"], b["longest"]) for a, b in zip(waves[::2], waves[1::2])]
    cap = list_replay.constants()["LIST_CAP"]
    redone = [n > cap - 8 for n in longest]          # (or nearly: fp32 scores may decide otherwise on an entry or two)
    assert sum(n > cap + 8 for n in longest) <= ea.read_stats(ws)["list_overflow_blocks"] <= sum(redone)
    for counting in (False, True):
        mine = [w for i, w in enumerate(waves) if w["counting"] == counting and not redone[i // 2]]
        print("  counting", counting, [{n: int(w[n]) for n in ("refreshes", "prunes", "pruned", "tight_tiles", "longest")} for w in mine[:6]], flush=True)
        assert any(w["prunes_leaving_odd_lists"] for w in mine) and any(w["prunes"] > 1 for w in mine) and any(w["tight_tiles"] for w in mine)
        assert any(w["counting"] == counting and w["longest"] > cap + 8 for w in waves)
    ref = eo.attn_fwd(Qn, Kn, parity.to_np64(v), alpha, False, tile=64)
    parity.check_forward(q, k, v, alpha, False, O, tau, mask, ref=ref, label=f"pruned and nearly full lists {dtype} {d}")
    t0, up, ts = parity.to_np64(tau0), parity.to_np64(upper), ref["tau"]
    eps = 3e-5 * (1.0 + np.abs(ts))
    assert (t0 <= ts + eps).all() and (ts <= up + eps).all() and (up - t0 <= 1.0 / nb + 1e-4).all()
    want = np.array([max(th, m - 1.0) for th, m in (grid_histogram_root(row, alpha, nb) for row in X)])
    # (a score that fp32 puts on the other side of a bin edge moves one count by one bin: among n counts the root moves by 1 / (n nb))
    diff = np.abs(t0[0, 0] - want)
    assert (diff <= 1e-4 * (1.0 + np.abs(want))).mean() >= 0.5 and diff.max() <= 0.25 / nb, (diff.max(), (diff > 1e-4).mean())
