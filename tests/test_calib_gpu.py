"""GPU parity of the activation calibration objective (Sec. 4.3, Eq. 9)
through the C ABI: the fp64 target X~ W^ against the oracle's, and the
objective of every candidate against the oracle's, within a bound derived
from the fused linear's fp32 contract; the candidate the GPU ranks first is
the oracle's best within that bound; results are reproducible and do not
depend on the batch a candidate is evaluated in."""
import numpy as np
import pytest
import torch

from gpu_util import f32_to_dev, i32_to_dev, u8_to_dev, u16_to_dev
from tile_sizes import ERR_EIGHT, ERR_FOUR
from oracle import sq_oracle as O
from paper_2609_39056_amd import binding as B
from paper_2609_39056_amd import synth

pytestmark = pytest.mark.gpu

F32 = np.float32


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def weight(L, G):
    pw = O.pack_weights(L.w, L.d, G)
    W = B.Weight(qw=u8_to_dev(pw["qw"]), w_scale=u16_to_dev(pw["w_scale"].T, torch.float16), w_group=G,
                 bias=u16_to_dev(L.bias_bits, torch.bfloat16))
    return pw, W


def abs_reference(L, pw, G, use_dinv=True):
    """sum_k |x~_ik| |w^_jk| in fp64: the scale of the fp64 sums' rounding."""
    xt = O.bf16_bits_to_f32(L.x_bits)
    if use_dinv:
        xt = (xt * L.dinv[None, :]).astype(F32)
    wq = pw["codes"].astype(np.float64) * np.repeat(O.f16_bits_to_f32(pw["w_scale"]).astype(np.float64), G, axis=1)
    return np.abs(xt.astype(np.float64)) @ np.abs(wq).T


def gpu_reference(L, W, use_dinv=True):
    M, N = L.x_bits.shape[0], W.N
    ref = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda")
    B.sq_calib_reference(u16_to_dev(L.x_bits, torch.bfloat16), f32_to_dev(L.dinv) if use_dinv else None, W, ref)
    return ref


def candidates(L, n_extra, seed):
    """The layer's step tables plus perturbed ones: gains per stream and clips."""
    rng = np.random.default_rng(seed)
    g = [L.gamma[t] for t in range(L.gamma.shape[0])]
    c = [L.clip[t] for t in range(L.clip.shape[0])]
    for _ in range(n_extra):
        g.append((L.gamma[0] * rng.lognormal(0.0, 0.4, L.gamma.shape[1])).astype(F32))
        c.append(F32(L.clip[0] * rng.lognormal(0.0, 0.5)))
    return np.stack(g).astype(F32), np.array(c, dtype=F32)


def gpu_objective(L, W, bits, gammas, clips, omega, ref, S=None):
    M, K, N = L.x_bits.shape[0], W.K, W.N
    S = L.gamma.shape[1] if S is None else S
    ws = torch.empty(B.sq_calib_workspace_bytes(M, K, N, bits, S), dtype=torch.uint8, device="cuda")
    obj = torch.full((len(clips),), float("nan"), dtype=torch.float64, device="cuda")
    B.sq_calib_objective(u16_to_dev(L.x_bits, torch.bfloat16), i32_to_dev(L.tok2stream), S, f32_to_dev(L.dinv),
                         bits, W, ref, f32_to_dev(gammas), f32_to_dev(clips),
                         torch.as_tensor(np.asarray(omega, dtype=np.float64), device="cuda"), obj, ws)
    torch.cuda.synchronize()
    return obj.cpu().numpy()


def objective_bound(L, pw, G, bits, gammas, clips, omega, ref, ref_abs, S):
    """Per candidate, how far the GPU objective may sit from the oracle's.
    The GPU's output is y64 + d with |d| <= 1e-5 A (the fused linear's fp32
    bound, A = sum of |terms|) plus fp32 rounding of y, and its target is
    ref + r with |r| <= K 2^-52 sum|x~||w^|; with t = |d| + |r|, each squared
    error moves by at most 2 |e| t + t^2, weighted as in the objective."""
    K = L.x_bits.shape[1]
    t2s = L.tok2stream
    out = []
    for g, c in zip(gammas, clips):
        res = O.linear(L.x_bits, t2s, g[None, :], 0, pw["codes"], pw["w_scale"], G, dinv=L.dinv,
                       clip=np.array([c], dtype=F32), bias_bits=None, range_mode=O.RANGE_STATIC, act_bits=bits)
        e = np.abs(res["y64"] - ref)
        t = 1e-5 * res["A"] + 2.0**-23 * np.abs(res["y64"]) + K * 2.0**-52 * ref_abs
        row = (2 * e * t + t * t).sum(axis=1)
        b = 0.0
        for s in range(S):
            n = int((t2s == s).sum())
            if n:
                b += float(omega[s]) / n * float(row[t2s == s].sum())
        out.append(b)
    return np.array(out)


def check_objectives(got, want, bound):
    err = np.abs(got - want)
    assert np.all(np.isfinite(got))
    assert np.all(err <= bound + 1e-12 * np.abs(want)), f"err {err} bound {bound} want {want}"
    # the candidate ranked first on the GPU is the oracle's best within the bound
    best = int(np.argmin(got))
    assert want[best] <= want.min() + bound[best] + bound[int(np.argmin(want))] + 1e-12 * want.min()


@pytest.mark.parametrize("use_dinv", [True, False])
@pytest.mark.parametrize("G", [128, 256])
@pytest.mark.parametrize("M,N", [(200, 192), (1, 64), (129, 128)])
def test_calib_reference(M, N, G, use_dinv):
    """X~ W^ in fp64 against the oracle: ragged rows (200 = 128 + 72), a
    half tile of columns (192), a single row; one weight step per 128-channel
    group or per output channel."""
    K = 256
    L = synth.make_layer(K=K, N=N, stream_counts=(max(M - 2, 1), 1, 1) if M > 2 else (M, 0, 0), seed=[40, M, N])
    pw, W = weight(L, G)
    got = gpu_reference(L, W, use_dinv).cpu().numpy()
    want = O.calib_reference(L.x_bits, pw["codes"], pw["w_scale"], G, L.dinv if use_dinv else None)
    ref_abs = abs_reference(L, pw, G, use_dinv)
    assert np.all(np.abs(got - want) <= K * 2.0**-52 * ref_abs)


@pytest.mark.parametrize("G", [128, 256])
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M", [1, 37, 200])
def test_calib_objective(M, bits, G):
    """Seven candidates on a three-stream layer (permuted rows), uniform and
    uneven stream weights: 37 tokens (weight-streaming GEMM) and 200 (tiled;
    4-bit codes on the fp8 matrix cores)."""
    K, N = 256, 192
    L = synth.make_layer(K=K, N=N, stream_counts=(M - M // 4 - M // 8, M // 8, M // 4), T=3, seed=[41, M, bits],
                         permute=True)
    pw, W = weight(L, G)
    ref_dev = gpu_reference(L, W)
    ref = O.calib_reference(L.x_bits, pw["codes"], pw["w_scale"], G, L.dinv)
    ref_abs = abs_reference(L, pw, G)
    gammas, clips = candidates(L, 4, seed=[42, M])
    for omega in (np.full(3, 1 / 3), np.array([0.5, 0.2, 0.3])):
        got = gpu_objective(L, W, bits, gammas, clips, omega, ref_dev)
        want = O.calib_objective(L.x_bits, L.tok2stream, 3, pw["codes"], pw["w_scale"], G, gammas, clips, omega,
                                 dinv=L.dinv, act_bits=bits, ref=ref)
        bound = objective_bound(L, pw, G, bits, gammas, clips, omega, ref, ref_abs, 3)
        check_objectives(got, want, bound)


def test_calib_empty_stream_and_reuse():
    """A stream with no token adds nothing (four streams, the second empty,
    with weight 0.4); the same candidates evaluated again, one at a time and in
    another order give bit-identical objectives."""
    K, N, bits, G = 256, 128, 8, 128
    L = synth.make_layer(K=K, N=N, stream_counts=(60, 0, 25, 15), T=2, seed=43, permute=True)
    assert L.gamma.shape[1] == 4 and not np.any(L.tok2stream == 1)
    pw, W = weight(L, G)
    ref_dev = gpu_reference(L, W)
    ref = O.calib_reference(L.x_bits, pw["codes"], pw["w_scale"], G, L.dinv)
    gammas, clips = candidates(L, 3, seed=44)
    omega = np.array([0.3, 0.4, 0.2, 0.1])
    got = gpu_objective(L, W, bits, gammas, clips, omega, ref_dev)
    want = O.calib_objective(L.x_bits, L.tok2stream, 4, pw["codes"], pw["w_scale"], G, gammas, clips, omega,
                             dinv=L.dinv, act_bits=bits, ref=ref)
    bound = objective_bound(L, pw, G, bits, gammas, clips, omega, ref, abs_reference(L, pw, G), 4)
    check_objectives(got, want, bound)
    again = gpu_objective(L, W, bits, gammas, clips, omega, ref_dev)
    assert np.array_equal(got.view(np.uint64), again.view(np.uint64))
    order = np.arange(len(clips))[::-1].copy()
    rev = gpu_objective(L, W, bits, gammas[order], clips[order], omega, ref_dev)
    assert np.array_equal(rev.view(np.uint64), got[order].view(np.uint64))
    one = gpu_objective(L, W, bits, gammas[2:3], clips[2:3], omega, ref_dev)
    assert one.view(np.uint64)[0] == got.view(np.uint64)[2]


@pytest.mark.parametrize("bits", [8, 4])
def test_calib_objective_larger(bits):
    """512 calibration tokens of a K = 2048, N = 512 linear (16 K-blocks,
    four tiles of rows), three candidates."""
    K, N, G = 2048, 512, 128
    L = synth.make_layer(K=K, N=N, stream_counts=(384, 48, 80), T=3, seed=[45, bits], permute=True)
    pw, W = weight(L, G)
    ref_dev = gpu_reference(L, W)
    ref = O.calib_reference(L.x_bits, pw["codes"], pw["w_scale"], G, L.dinv)
    gammas, clips = L.gamma.copy(), L.clip.copy()
    omega = np.full(3, 1 / 3)
    got = gpu_objective(L, W, bits, gammas, clips, omega, ref_dev)
    want = O.calib_objective(L.x_bits, L.tok2stream, 3, pw["codes"], pw["w_scale"], G, gammas, clips, omega,
                             dinv=L.dinv, act_bits=bits, ref=ref)
    bound = objective_bound(L, pw, G, bits, gammas, clips, omega, ref, abs_reference(L, pw, G), 3)
    check_objectives(got, want, bound)


# ---------------------------------------------------------------- constrained search
def gpu_search(L, W, bits, omega, ref, bounds, clip_init, log_step, rounds, S=None):
    M, K, N = L.x_bits.shape[0], W.K, W.N
    S = L.gamma.shape[1] if S is None else S
    ws = torch.empty(B.sq_calib_search_workspace_bytes(M, K, N, bits, S), dtype=torch.uint8, device="cuda")
    g = torch.full((S,), float("nan"), dtype=torch.float32, device="cuda")
    c = torch.full((1,), float("nan"), dtype=torch.float32, device="cuda")
    obj = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda")
    p = B.sq_calib_search_params(*[float(b) for b in bounds], float(clip_init), float(log_step), rounds)
    B.sq_calib_search(u16_to_dev(L.x_bits, torch.bfloat16), i32_to_dev(L.tok2stream), S, f32_to_dev(L.dinv), bits,
                      W, ref, torch.as_tensor(np.asarray(omega, dtype=np.float64), device="cuda"), p, g, c, obj, ws)
    torch.cuda.synchronize()
    return g.cpu().numpy(), F32(c.cpu().numpy()[0]), float(obj.cpu().numpy()[0])


def check_constraints(gam, c, counts, bounds):
    g_min, g_max, c_min, c_max = (F32(b) for b in bounds)
    assert np.all(gam >= g_min) and np.all(gam <= g_max) and c_min <= c <= c_max
    lg = np.log(gam.astype(np.float64))
    # each fp32 gain carries a rounding of 2^-24 relative: |log| moves by <= 2^-24
    assert abs((counts * lg).sum()) <= counts.sum() * (2.0**-23 + 1e-12)


@pytest.mark.parametrize("bits,M,counts", [(8, 200, (140, 20, 40)), (4, 200, (140, 20, 40)),
                                           (8, 37, (25, 4, 8)), (4, 96, (60, 0, 20, 16))])
def test_calib_search_matches_oracle(bits, M, counts):
    """The GPU search against the oracle's compass search on the same layer:
    when every decision of the oracle's run (which candidate is smallest,
    whether it beats the incumbent) is separated by more than the objective's
    error bound, the GPU takes the same path and returns the same fp32 point;
    in every case the result meets the constraints, its objective is the
    GPU's sq_calib_objective of that point, and the oracle's objective of it
    is no worse than the start's.  Includes a stream without tokens."""
    K, N, G = 256, 128, 128
    L = synth.make_layer(K=K, N=N, stream_counts=counts, T=2, seed=[50, bits, M], permute=True)
    S = L.gamma.shape[1]
    n = np.bincount(L.tok2stream, minlength=S)
    pw, W = weight(L, G)
    ref_dev = gpu_reference(L, W)
    ref = O.calib_reference(L.x_bits, pw["codes"], pw["w_scale"], G, L.dinv)
    ref_abs = abs_reference(L, pw, G)
    omega = np.full(S, 1.0 / S)
    bounds = (0.5, 2.0, float(L.clip[0]) / 8, float(L.clip[0]) * 2)
    bounds = tuple(float(F32(b)) for b in bounds)
    rounds = 6

    def f(Gm, Cm):
        return O.calib_objective(L.x_bits, L.tok2stream, S, pw["codes"], pw["w_scale"], G, Gm, Cm, omega,
                                 dinv=L.dinv, act_bits=bits, ref=ref)

    g_or, c_or, L_or, h_or, trace = O.calib_search(f, n, bounds, L.clip[0], 0.5, rounds)
    g_gpu, c_gpu, L_gpu = gpu_search(L, W, bits, omega, ref_dev, bounds, L.clip[0], 0.5, rounds)
    check_constraints(g_gpu, c_gpu, n, bounds)
    # the returned objective is the evaluator's for the returned point
    again = gpu_objective(L, W, bits, g_gpu[None, :], np.array([c_gpu]), omega, ref_dev)
    assert again.view(np.uint64)[0] == np.float64(L_gpu).view(np.uint64)
    start = f(np.ones((1, S), F32), np.array([np.clip(F32(L.clip[0]), F32(bounds[2]), F32(bounds[3]))]))[0]
    got_or = f(g_gpu[None, :], np.array([c_gpu]))[0]
    b_pt = objective_bound(L, pw, G, bits, g_gpu[None, :], np.array([c_gpu]), omega, ref, ref_abs, S)[0]
    assert got_or <= start + b_pt
    assert abs(L_gpu - got_or) <= b_pt + 1e-12 * got_or

    # separated decisions: replay the oracle's rounds with the bound of every candidate
    c0 = np.clip(F32(L.clip[0]), F32(bounds[2]), F32(bounds[3]))
    u, vc, h = np.zeros(S), float(np.log(np.float64(c0))), 0.5
    inc_b = objective_bound(L, pw, G, bits, np.ones((1, S), F32), np.array([c0]), omega, ref, ref_abs, S)[0]
    separated = True
    inc_g, inc_c = np.ones(S, F32), c0
    for L_inc, obj in trace:
        Gm, Cm, U, V = O.compass_candidates(u, vc, h, n, bounds)
        bd = objective_bound(L, pw, G, bits, Gm, Cm, omega, ref, ref_abs, S)
        j = int(np.argmin(obj))
        # points that differ only in the gains of streams without tokens give
        # bit-identical outputs, hence equal objectives, on both sides
        live = n > 0
        for k in range(len(obj)):
            same = np.array_equal(Gm[k][live], Gm[j][live]) and Cm[k] == Cm[j]
            if k != j and not same and obj[k] - obj[j] <= bd[k] + bd[j]:
                separated = False
        same_as_inc = np.array_equal(Gm[j][live], inc_g[live]) and Cm[j] == inc_c
        if not same_as_inc and abs(obj[j] - L_inc) <= bd[j] + inc_b:
            separated = False
        if obj[j] < L_inc:
            u, vc, inc_b, inc_g, inc_c = U[j], float(V[j]), bd[j], Gm[j], Cm[j]
        else:
            h = 0.5 * h
    if separated:
        assert np.array_equal(g_gpu, g_or) and c_gpu == c_or, (g_gpu, g_or, c_gpu, c_or)
        assert abs(L_gpu - L_or) <= inc_b + 1e-12 * L_or
    print(f"separated={separated} L_gpu={L_gpu} L_or={L_or} start={start}")


def test_calib_search_start_and_single_stream():
    """rounds = 0 evaluates the start (gamma = 1, c = clip_init clamped); with
    one stream the constraint pins gamma to 1 and only c moves."""
    K, N, G, bits = 256, 64, 128, 8
    L = synth.make_layer(K=K, N=N, stream_counts=(48, 16, 8), T=1, seed=51, permute=True)
    pw, W = weight(L, G)
    ref_dev = gpu_reference(L, W)
    bounds = (0.5, 2.0, 0.25, 4.0)
    g, c, obj = gpu_search(L, W, bits, np.full(3, 1 / 3), ref_dev, bounds, 100.0, 0.5, 0)
    assert np.all(g == 1.0) and c == F32(4.0)
    want = gpu_objective(L, W, bits, np.ones((1, 3), F32), np.array([4.0], F32), np.full(3, 1 / 3), ref_dev)[0]
    assert np.float64(obj).view(np.uint64) == want.view(np.uint64)
    L1 = synth.make_layer(K=K, N=N, stream_counts=(64,), T=1, seed=52)
    pw1, W1 = weight(L1, G)
    ref1 = gpu_reference(L1, W1)
    g1, c1, o1 = gpu_search(L1, W1, bits, np.ones(1), ref1, (0.5, 2.0, float(L1.clip[0]) / 4, float(L1.clip[0]) * 2),
                            L1.clip[0], 0.5, 5)
    assert g1[0] == F32(1.0)
    start = gpu_objective(L1, W1, bits, np.ones((1, 1), F32),
                          np.array([np.clip(L1.clip[0], F32(L1.clip[0] / 4), F32(L1.clip[0] * 2))]), np.ones(1), ref1)
    assert o1 <= start[0]


@pytest.mark.parametrize("bits", [8, 4])
def test_calib_objective_max_rows(bits):
    """M = 2^24 calibration tokens (the C ABI's maximum; row offsets of the
    fp64 target pass 2^31 bytes): a 256-token block tiled 65536 times, so
    every stream's error sum and token count grow by the same factor and the
    objective must equal the block's.  Compared with the oracle on the block
    (within its bound) and with the GPU's own objective of the block."""
    K, N, G, R = 128, 64, 128, 1 << 16
    L = synth.make_layer(K=K, N=N, stream_counts=(192, 24, 40), T=2, seed=60, permute=True)
    pw, W = weight(L, G)
    gammas, clips = candidates(L, 1, seed=61)
    omega = np.array([0.5, 0.3, 0.2])
    ref_small = gpu_reference(L, W)
    small = gpu_objective(L, W, bits, gammas, clips, omega, ref_small)
    ref = O.calib_reference(L.x_bits, pw["codes"], pw["w_scale"], G, L.dinv)
    want = O.calib_objective(L.x_bits, L.tok2stream, 3, pw["codes"], pw["w_scale"], G, gammas, clips, omega,
                             dinv=L.dinv, act_bits=bits, ref=ref)
    bound = objective_bound(L, pw, G, bits, gammas, clips, omega, ref, abs_reference(L, pw, G), 3)
    check_objectives(small, want, bound)
    del ref_small
    x = u16_to_dev(L.x_bits, torch.bfloat16).repeat(R, 1)
    t2s = i32_to_dev(L.tok2stream).repeat(R)
    M = x.shape[0]
    assert M == 1 << 24
    ref_big = torch.empty((M, N), dtype=torch.float64, device="cuda")
    dinv = f32_to_dev(L.dinv)
    B.sq_calib_reference(x, dinv, W, ref_big)
    ws = torch.empty(B.sq_calib_workspace_bytes(M, K, N, bits, 3), dtype=torch.uint8, device="cuda")
    obj = torch.full((len(clips),), float("nan"), dtype=torch.float64, device="cuda")
    B.sq_calib_objective(x, t2s, 3, dinv, bits, W, ref_big, f32_to_dev(gammas), f32_to_dev(clips),
                         torch.as_tensor(omega, device="cuda"), obj, ws)
    torch.cuda.synchronize()
    big = obj.cpu().numpy()
    # identical rows give identical per-row errors; only the order of the fp64 sums differs
    assert np.allclose(big, small, rtol=1e-9, atol=0), (big, small)
    # the last tiled copy of the target equals the block's
    tail = ref_big[M - L.x_bits.shape[0]:].cpu().numpy()
    assert np.all(np.abs(tail - ref) <= K * 2.0**-52 * abs_reference(L, pw, G))


# ---------------------------------------------------------------- shared channel scaling, Eq. (7)
@pytest.mark.parametrize("M,N", [(200, 192), (4500, 64)])
def test_smooth_scales(M, N):
    """d and 1/d of the family, bit-exact against the oracle for five
    exponents, on a layer with x20 outlier channels (the clamp binds at alpha
    = 1) and an all-zero channel (d = 1); 4500 rows span 71 row blocks of the
    amax kernel."""
    K = 256
    L = synth.make_layer(K=K, N=N, stream_counts=(M - 30, 10, 20), T=1, seed=[70, M])
    xb = L.x_bits.copy()
    xb[:, 3] = 0
    x = u16_to_dev(xb, torch.bfloat16)
    w = f32_to_dev(L.w)
    d = torch.empty(K, dtype=torch.float32, device="cuda")
    dinv = torch.empty_like(d)
    for alpha in (0.0, 0.25, 0.5, 0.75, 1.0):
        B.sq_smooth_scales(x, w, alpha, d, dinv)
        torch.cuda.synchronize()
        want_d, want_dinv = O.smooth_scales(xb, L.w, alpha)
        got_d, got_dinv = d.cpu().numpy(), dinv.cpu().numpy()
        assert np.array_equal(got_d.view(np.uint32), want_d.view(np.uint32)), alpha
        assert np.array_equal(got_dinv.view(np.uint32), want_dinv.view(np.uint32)), alpha
        assert got_d[3] == 1.0
    assert want_d.max() == 64.0  # alpha = 1: the clamp binds on the outlier channels


@pytest.mark.parametrize("M,N", [(200, 192), (1, 64)])
def test_calib_fp_reference(M, N):
    """X W^T in fp64 against the oracle's full-precision product."""
    K = 384
    L = synth.make_layer(K=K, N=N, stream_counts=(M, 0, 0), T=1, seed=[71, M])
    ref = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda")
    B.sq_calib_fp_reference(u16_to_dev(L.x_bits, torch.bfloat16), f32_to_dev(L.w), ref)
    want = O.full_precision_linear(L.x_bits, L.w)
    scale = np.abs(O.bf16_bits_to_f32(L.x_bits).astype(np.float64)) @ np.abs(L.w.astype(np.float64)).T
    assert np.all(np.abs(ref.cpu().numpy() - want) <= K * 2.0**-52 * scale)


def scaling_bound(L, G, bits, region, R, weights, alphas, ref, ref_abs):
    """As objective_bound, for Eq. (7)'s candidates (DYNAMIC ranges, unit
    gains, the fp64 full-precision target)."""
    K = L.x_bits.shape[1]
    out = []
    for alpha in alphas:
        d, dinv = O.smooth_scales(L.x_bits, L.w, alpha)
        pw = O.pack_weights(L.w, d, G)
        res = O.linear(L.x_bits, region, np.ones((1, R), F32), 0, pw["codes"], pw["w_scale"], G, dinv=dinv,
                       bias_bits=None, act_bits=bits)
        e = np.abs(res["y64"] - ref)
        t = 1e-5 * res["A"] + 2.0**-23 * np.abs(res["y64"]) + K * 2.0**-52 * ref_abs
        row = (2 * e * t + t * t).sum(axis=1)
        b = 0.0
        for r in range(R):
            n = int((region == r).sum())
            if n:
                b += float(weights[r]) / n * float(row[region == r].sum())
        out.append(b)
    return np.array(out)


@pytest.mark.parametrize("G", [128, 256])
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M", [1, 37, 200])
def test_calib_scaling_objective(M, bits, G):
    """Eq. (7) for five exponents against the oracle within the derived bound,
    with six regions (three streams x two step halves, uneven weights); the
    GPU's best exponent is the oracle's within that bound."""
    K, N = 256, 128
    L = synth.make_layer(K=K, N=N, stream_counts=(M - M // 4 - M // 8, M // 8, M // 4), T=1, seed=[72, M, bits],
                         permute=True)
    R = 6
    region = (L.tok2stream + 3 * (np.arange(M) % 2)).astype(np.int32)
    weights = np.array([0.3, 0.1, 0.1, 0.3, 0.1, 0.1])
    alphas = [0.0, 0.25, 0.5, 0.75, 1.0]
    x, w = u16_to_dev(L.x_bits, torch.bfloat16), f32_to_dev(L.w)
    ref_dev = torch.empty((M, N), dtype=torch.float64, device="cuda")
    B.sq_calib_fp_reference(x, w, ref_dev)
    ws = torch.empty(B.sq_calib_scaling_workspace_bytes(M, K, N, G, bits, R), dtype=torch.uint8, device="cuda")
    obj = torch.full((len(alphas),), float("nan"), dtype=torch.float64, device="cuda")
    B.sq_calib_scaling_objective(x, i32_to_dev(region), R, torch.as_tensor(weights, device="cuda"), w, G, bits,
                                 ref_dev, alphas, obj, ws)
    torch.cuda.synchronize()
    got = obj.cpu().numpy()
    ref = O.full_precision_linear(L.x_bits, L.w)
    want = O.scaling_objective(L.x_bits, region, R, weights, L.w, G, alphas, act_bits=bits, ref=ref)
    ref_abs = np.abs(O.bf16_bits_to_f32(L.x_bits).astype(np.float64)) @ np.abs(L.w.astype(np.float64)).T
    bound = scaling_bound(L, G, bits, region, R, weights, alphas, ref, ref_abs)
    check_objectives(got, want, bound)


@pytest.mark.parametrize("bits,G", [(8, 2048), (4, 128)])
def test_calib_objective_benchmark_shape(bits, G):
    """The benchmark's calibration configuration: the 2B up projection
    (2048 -> 8192) over 4192 tokens, in the launch configuration the
    benchmark times (the tiled GEMM with its split tail; one weight step per
    output channel for A8).  The 4192 rows are a 262-token block repeated 16
    times, so the objective must equal the oracle's objective of the block
    (within its bound); the search over the full batch is checked for its
    constraints and its returned objective."""
    K, N, R = 2048, 8192, 16
    L = synth.make_layer(K=K, N=N, stream_counts=(256, 2, 4), T=2, seed=80, permute=True)
    pw, W = weight(L, G)
    gammas, clips = candidates(L, 1, seed=81)
    omega = np.full(3, 1 / 3)
    ref = O.calib_reference(L.x_bits, pw["codes"], pw["w_scale"], G, L.dinv)
    want = O.calib_objective(L.x_bits, L.tok2stream, 3, pw["codes"], pw["w_scale"], G, gammas, clips, omega,
                             dinv=L.dinv, act_bits=bits, ref=ref)
    bound = objective_bound(L, pw, G, bits, gammas, clips, omega, ref, abs_reference(L, pw, G), 3)
    x = u16_to_dev(L.x_bits, torch.bfloat16).repeat(R, 1)
    t2s = i32_to_dev(L.tok2stream).repeat(R)
    M = x.shape[0]
    assert M == 4192
    dinv = f32_to_dev(L.dinv)
    ref_big = torch.empty((M, N), dtype=torch.float64, device="cuda")
    B.sq_calib_reference(x, dinv, W, ref_big)
    ws = torch.empty(B.sq_calib_search_workspace_bytes(M, K, N, bits, 3), dtype=torch.uint8, device="cuda")
    obj = torch.full((len(clips),), float("nan"), dtype=torch.float64, device="cuda")
    om = torch.as_tensor(omega, device="cuda")
    B.sq_calib_objective(x, t2s, 3, dinv, bits, W, ref_big, f32_to_dev(gammas), f32_to_dev(clips), om, obj, ws)
    torch.cuda.synchronize()
    check_objectives(obj.cpu().numpy(), want, bound)
    g = torch.empty(3, dtype=torch.float32, device="cuda")
    c = torch.empty(1, dtype=torch.float32, device="cuda")
    o = torch.empty(1, dtype=torch.float64, device="cuda")
    bnds = (0.25, 4.0, float(F32(L.clip[0] / 8)), float(F32(L.clip[0] * 4)))
    p = B.sq_calib_search_params(*bnds, float(L.clip[0]), 0.5, 4)
    B.sq_calib_search(x, t2s, 3, dinv, bits, W, ref_big, om, p, g, c, o, ws)
    torch.cuda.synchronize()
    gam_np, c_np = g.cpu().numpy(), F32(c.cpu().numpy()[0])
    n = np.bincount(L.tok2stream, minlength=3) * R
    check_constraints(gam_np, c_np, n, bnds)
    again = gpu_objective_dev(x, t2s, dinv, W, bits, ref_big, gam_np[None, :], np.array([c_np]), omega, ws)
    assert again.view(np.uint64)[0] == np.float64(o.cpu().numpy()[0]).view(np.uint64)


def gpu_objective_dev(x, t2s, dinv, W, bits, ref, gammas, clips, omega, ws):
    obj = torch.full((len(clips),), float("nan"), dtype=torch.float64, device="cuda")
    B.sq_calib_objective(x, t2s, len(omega), dinv, bits, W, ref, f32_to_dev(gammas), f32_to_dev(clips),
                         torch.as_tensor(np.asarray(omega, np.float64), device="cuda"), obj, ws)
    torch.cuda.synchronize()
    return obj.cpu().numpy()


def test_calib_search_max_streams():
    """The search at its stream limit (64 streams, a third of them without
    tokens; 130 candidates a round): every constraint holds, streams without
    tokens keep gamma = 1 (a step on them never improves the objective), the
    returned objective is the evaluator's for the returned point, and it is no
    worse than the start."""
    K, N, G, bits, S = 256, 64, 128, 8, 64
    rng = np.random.default_rng(90)
    counts = [int(v) if i % 3 else 0 for i, v in enumerate(rng.integers(1, 9, S))]
    L = synth.make_layer(K=K, N=N, stream_counts=tuple(counts), T=1, seed=91, permute=True)
    assert L.gamma.shape[1] == S
    n = np.bincount(L.tok2stream, minlength=S)
    pw, W = weight(L, G)
    ref_dev = gpu_reference(L, W)
    omega = np.full(S, 1.0 / S)
    bounds = (0.5, 2.0, float(F32(L.clip[0] / 4)), float(F32(L.clip[0] * 2)))
    g, c, obj = gpu_search(L, W, bits, omega, ref_dev, bounds, L.clip[0], 0.5, 3)
    check_constraints(g, c, n, bounds)
    assert np.all(g[n == 0] == 1.0)
    again = gpu_objective(L, W, bits, g[None, :], np.array([c]), omega, ref_dev)
    assert again.view(np.uint64)[0] == np.float64(obj).view(np.uint64)
    c0 = np.clip(F32(L.clip[0]), F32(bounds[2]), F32(bounds[3]))
    start = gpu_objective(L, W, bits, np.ones((1, S), F32), np.array([c0]), omega, ref_dev)[0]
    assert obj <= start


@pytest.mark.parametrize("bits,G,M,K,N", [(8, G, *s) for G in (128, 0) for s in ERR_EIGHT] +
                         [(4, 128, *s) for s in ERR_FOUR])
def test_calib_epilogue_equals_two_pass(M, K, N, bits, G):
    """The objective from the GEMM's epilogue (more than 128 tokens) against
    the same sum taken in two passes: the fused linear's fp32 output (STATIC,
    one-step table, no bias) minus the target, squared and weighted in fp64.
    Every tile shape whole and split along K, as far as sizes reach it
    (tile_sizes.py, held by test_tile_choice.py), a half tile of columns, a last
    row of tiles with one row.  Both sum the same M N non-negative terms, so they
    differ by at most the summation error (M N + 4) 2^-53."""
    L = synth.make_layer(K=K, N=N, stream_counts=(M - M // 4 - 8, 8, M // 4), T=2, seed=[46, M, N], permute=True)
    pw, W = weight(L, G or K)
    ref = gpu_reference(L, W)
    omega = np.array([0.5, 0.2, 0.3])
    got = gpu_objective(L, W, bits, L.gamma, L.clip, omega, ref)
    x, t2s = u16_to_dev(L.x_bits, torch.bfloat16), i32_to_dev(L.tok2stream)
    n = np.bincount(L.tok2stream, minlength=3)
    row_w = torch.as_tensor((omega / n)[L.tok2stream], device="cuda")
    Wn = B.Weight(qw=W.qw, w_scale=W.w_scale, w_group=W.w_group)
    for c in range(len(L.clip)):
        act = B.ActParams(tok2stream=t2s, gamma=f32_to_dev(L.gamma), step=c, act_bits=bits,
                          range_mode=B.SQ_RANGE_STATIC, clip=f32_to_dev(L.clip), dinv=f32_to_dev(L.dinv))
        y = torch.empty((M, N), dtype=torch.float32, device="cuda")
        fn = B.sq_linear_w4a8 if bits == 8 else B.sq_linear_w4a4
        fn(x, act, Wn, y, B.SQ_OUT_F32, B.alloc_workspace(B.SQ_VARIANT_FUSED, M, K, N, bits))
        want = float(((y.double() - ref).square().sum(dim=1) * row_w).sum())
        assert abs(got[c] - want) <= (M * N + 4) * 2.0**-53 * want


@pytest.mark.parametrize("bits,G", [(8, 128), (8, 0), (4, 128)])
@pytest.mark.parametrize("M,K,N", [(129, 256, 64), (200, 1024, 192), (1537, 1536, 8128), (1001, 2048, 8320)])
def test_calib_epilogue_overflowing_last_row(M, K, N, bits, G):
    """The last row's fp32 outputs overflow (its stream's gain is 1e-36 and its
    codes are all q_max): the objective is the two passes' infinity, whatever
    the last row of tiles holds past row M - 1, and an objective without that
    row's stream stays finite."""
    W = B.prepare_weight(torch.full((N, K), 7.0, device="cuda"), None, G or K)
    x = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda")
    x[-1] = 1e37
    t2s = torch.zeros(M, dtype=torch.int32, device="cuda")
    t2s[-1] = 1
    ref = torch.zeros((M, N), dtype=torch.float64, device="cuda")
    gamma, clip = torch.tensor([[1.0, 1e-36], [1.0, 1.0]], device="cuda"), torch.ones(2, device="cuda")
    omega = torch.full((2,), 0.5, dtype=torch.float64, device="cuda")
    obj = torch.empty(2, dtype=torch.float64, device="cuda")
    ws = torch.empty(B.sq_calib_workspace_bytes(M, K, N, bits, 2), dtype=torch.uint8, device="cuda")
    B.sq_calib_objective(x, t2s, 2, None, bits, W, ref, gamma, clip, omega, obj, ws)
    y = torch.empty((M, N), dtype=torch.float32, device="cuda")
    for c in range(2):
        act = B.ActParams(tok2stream=t2s, gamma=gamma, step=c, act_bits=bits, range_mode=B.SQ_RANGE_STATIC, clip=clip)
        fn = B.sq_linear_w4a8 if bits == 8 else B.sq_linear_w4a4
        fn(x, act, W, y, B.SQ_OUT_F32, B.alloc_workspace(B.SQ_VARIANT_FUSED, M, K, N, bits))
        assert not bool(y.isnan().any()) and bool(y[-1].isinf().all()) == (c == 0)
    assert obj[0].item() == float("inf") and obj[1].isfinite().item()


@pytest.mark.parametrize("M,N", [(1, 64), (63, 64), (64, 128), (65, 576), (600, 64)])
def test_calib_target_tiles(M, N):
    """Both fp64 targets at the edges of the kernel's 64 x 64 tiles and of its
    groups of eight row tiles, within K 2^-52 of the sum of |terms|."""
    K = 384
    L = synth.make_layer(K=K, N=N, stream_counts=(M, 0, 0), T=1, seed=[47, M, N])
    pw, W = weight(L, 128)
    got = gpu_reference(L, W).cpu().numpy()
    want = O.calib_reference(L.x_bits, pw["codes"], pw["w_scale"], 128, L.dinv)
    assert np.all(np.abs(got - want) <= K * 2.0**-52 * abs_reference(L, pw, 128))
    x, w = O.bf16_bits_to_f32(L.x_bits).astype(np.float64), L.w.astype(np.float64)
    y = torch.full((M, N), float("nan"), dtype=torch.float64, device="cuda")
    B.sq_calib_fp_reference(u16_to_dev(L.x_bits, torch.bfloat16), f32_to_dev(L.w), y)
    assert np.all(np.abs(y.cpu().numpy() - x @ w.T) <= K * 2.0**-52 * (np.abs(x) @ np.abs(w).T))
