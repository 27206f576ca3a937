// Calibration.  Activation calibration (Sec. 4.3, Eq. 9): the reconstruction
// error of one linear under a candidate (gain per stream, shared threshold),
// weighted per stream by omega_s / n_s, and a constrained search over
// candidates.  Shared scaling (Sec. 4.2, Eq. 7): the same error against the
// full-precision product for a family of channel scalings D.
//
//   - calib_reference_kernel<false>: the target X~ W^ in fp64, X~ = fp32(x) *
//     dinv (the quantizer's first step) and W^ = code * Delta_W.  Every
//     product is exact in fp64 (24 x 15 significant bits), so the kernel
//     differs from any other fp64 evaluation only in the order of its K sums.
//     On the fp64 matrix cores.  Computed once per linear.
//     calib_reference_kernel<true>: the same with fp32 W (the target X W of
//     Eq. 7; products of 8 x 24 significant bits, exact).
//   - channel_amax_kernel, smooth_scale_kernel: the per-channel maxima of |X|
//     and |W| and the family d = amax|X|^alpha / amax|W|^(1 - alpha) of Eq. 7.
//   - calib_count_kernel: n_s, the tokens of every stream (LDS histogram per
//     workgroup, one global add per non-empty bin).
//   - on the tiled GEMMs (more than 128 tokens) the error comes from the GEMM's
//     epilogue (kEpiErr), which leaves partial sums weighted by
//     calib_row_weight_kernel's omega_s(i) / n_s(i); else
//   - calib_row_error_kernel: e_i = omega_s(i) / n_s(i) * sum_j (y_ij - ref_ij)^2
//     for the candidate's fp32 output y, one wave per row, fixed order.
//   - calib_sum_kernel: the sum of either in one workgroup, fixed order.
// The candidate's output itself comes from the fused linear (no bias; STATIC
// with the candidate's one-step table for Eq. 9, DYNAMIC with unit gains for
// Eq. 7), so the objective measures the arithmetic that runs.
#include "sq_internal.h"

namespace sq {
namespace {

constexpr int kRefTile = 64;            // output rows and columns per workgroup
constexpr int kRefKc = 32;              // K per LDS stage
constexpr int kRefStride = kRefKc + 4;  // floats per LDS row: 16 rows' 16-byte reads fill all 64 banks
constexpr int kRefGroupM = 8;           // row tiles that share a column tile's weights in L2

typedef double v4d __attribute__((ext_vector_type(4)));

// 8 consecutive channels of one row of X (times D^-1) and of one column of W,
// as loaded; the widening to fp32 happens when they are put into LDS.
template <bool FPW>
struct RefChunk {
  uint4 x;
  float4 d0, d1;  // D^-1
  float4 w0, w1;  // FPW
  uint32_t p;     // packed codes and their step otherwise
  uint32_t step;
};

// The fp64 target on v_mfma_f64_16x16x4_f64.  Bound by the fp64 rate, which
// is the same for the matrix cores and the VALU (78.6 TFLOP/s); the matrix
// cores leave the VALU and the LDS to the staging.  The VALU kernel before it
// (128 x 128 tiles, 8 x 8 outputs per thread) spent 16 LDS reads of 8 bytes
// per 64 fmas and reached 45 TFLOP/s (3.16 ms) at 4192 x 2048 -> 8192; this
// one reaches 61 (2.31 ms), the matrix cores busy 78 % of the time at the
// 2.18 GHz the board's power allows (a library product of that shape: 64).  Measured and not faster: two LDS slots
// with one barrier per stage, a raised priority of the MFMA phase, fp64 in
// LDS (half the conversions, twice the LDS traffic).
//
// A workgroup computes 64 x 64 outputs, a wave 32 x 32 as 2 x 2 MFMA tiles:
// small tiles, since nothing but the matrix cores is short here (a stage is
// 4 KB of X and 1 KB of codes per 2048 matrix-core cycles) and they spread
// over the CUs evenly (four workgroups fit on one; 1048 x 2048 outputs are
// 544 tiles, with 128 x 128 only 144).  x~ is an fp32 value and code * Delta_W
// (4 x 11 significant bits) is one exactly, so LDS holds fp32 and the
// fragments are widened to fp64 in registers.  Lane (row or column lane & 15,
// g = lane >> 4) feeds the MFMA step s of a 16-channel block with channel
// 4 g + s: one 16-byte read per operand serves four steps.  An accumulator
// lane holds column lane & 15 and rows 4 j + (lane >> 4).
template <bool FPW>
__global__ __launch_bounds__(256, 4) void calib_reference_kernel(const uint16_t* __restrict__ x,
                                                                 const float* __restrict__ dinv,
                                                                 const uint8_t* __restrict__ qw,
                                                                 const uint16_t* __restrict__ w_scale,
                                                                 const float* __restrict__ wf,
                                                                 double* __restrict__ y, int32_t M, int32_t N,
                                                                 int32_t K, int32_t w_group, int32_t tiles_m,
                                                                 int32_t tiles_n) {
  const size_t wg = flat_wg();
  if (wg >= static_cast<size_t>(tiles_m) * tiles_n) return;
  // supertiles of kRefGroupM row tiles, column tile by column tile
  const size_t per_group = static_cast<size_t>(kRefGroupM) * tiles_n;
  const int32_t first_m = static_cast<int32_t>(wg / per_group) * kRefGroupM;
  const int32_t gm = min(tiles_m - first_m, kRefGroupM);
  const int32_t in_group = static_cast<int32_t>(wg % per_group);
  const int64_t m0 = static_cast<int64_t>(first_m + in_group % gm) * kRefTile;
  const int32_t n0 = in_group / gm * kRefTile;
  __shared__ __align__(16) float xs[kRefTile * kRefStride];
  __shared__ __align__(16) float ws[kRefTile * kRefStride];

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  // staging: thread t fills row (column) t / 4 of the tile, channels 8 (t % 4) .. + 7 of the stage;
  // rows past M repeat the last one (N % 64 == 0: every column is in)
  const int sr = t >> 2, sc = (t & 3) * 8;
  const uint16_t* xrow = x + min(m0 + sr, static_cast<int64_t>(M) - 1) * K + sc;
  const int32_t wn = n0 + sr;
  const uint8_t* wrow = FPW ? nullptr : qw + (static_cast<size_t>(wn) * K + sc) / 2;
  const float* wfrow = FPW ? wf + static_cast<size_t>(wn) * K + sc : nullptr;

  auto load = [&](int32_t k0) {
    RefChunk<FPW> c;
    c.x = *reinterpret_cast<const uint4*>(xrow + k0);
    if (!FPW && dinv != nullptr) {
      c.d0 = *reinterpret_cast<const float4*>(dinv + k0 + sc);
      c.d1 = *reinterpret_cast<const float4*>(dinv + k0 + sc + 4);
    }
    if constexpr (FPW) {
      c.w0 = *reinterpret_cast<const float4*>(wfrow + k0);
      c.w1 = *reinterpret_cast<const float4*>(wfrow + k0 + 4);
    } else {
      c.p = *reinterpret_cast<const uint32_t*>(wrow + k0 / 2);
      c.step = w_scale[static_cast<size_t>((k0 + sc) / w_group) * N + wn];
    }
    return c;
  };
  auto store = [&](const RefChunk<FPW>& c) {
    const uint32_t xw[4] = {c.x.x, c.x.y, c.x.z, c.x.w};
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = bf16_to_f32((xw[j >> 1] >> (16 * (j & 1))) & 0xFFFFu);
    if (!FPW && dinv != nullptr) {
      const float d[8] = {c.d0.x, c.d0.y, c.d0.z, c.d0.w, c.d1.x, c.d1.y, c.d1.z, c.d1.w};
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] *= d[j];
    }
    float4* xd = reinterpret_cast<float4*>(xs + sr * kRefStride + sc);
    xd[0] = make_float4(v[0], v[1], v[2], v[3]);
    xd[1] = make_float4(v[4], v[5], v[6], v[7]);
    float4* wd = reinterpret_cast<float4*>(ws + sr * kRefStride + sc);
    if constexpr (FPW) {
      wd[0] = c.w0;
      wd[1] = c.w1;
    } else {
      // byte b of the dword holds code sc + b (low nibble) and sc + b + 4 (high nibble)
      const float step = f16_to_f32(c.step);
      float w[8];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        w[b] = static_cast<float>(static_cast<int32_t>(c.p << (28 - 8 * b)) >> 28) * step;
        w[b + 4] = static_cast<float>(static_cast<int32_t>(c.p << (24 - 8 * b)) >> 28) * step;
      }
      wd[0] = make_float4(w[0], w[1], w[2], w[3]);
      wd[1] = make_float4(w[4], w[5], w[6], w[7]);
    }
  };

  const int wm = (wave >> 1) * 32, wc = (wave & 1) * 32;
  const int l16 = lane & 15, g = lane >> 4;
  v4d acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (v4d)(0.0);

  RefChunk<FPW> c = load(0);
  for (int32_t k0 = 0; k0 < K; k0 += kRefKc) {
    __syncthreads();  // the previous stage's reads are done
    store(c);
    __syncthreads();
    if (k0 + kRefKc < K) c = load(k0 + kRefKc);  // in flight under this stage's MFMAs
#pragma unroll
    for (int kb = 0; kb < kRefKc; kb += 16) {
      float4 a[2], b[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[i] = *reinterpret_cast<const float4*>(xs + (wm + 16 * i + l16) * kRefStride + kb + 4 * g);
        b[i] = *reinterpret_cast<const float4*>(ws + (wc + 16 * i + l16) * kRefStride + kb + 4 * g);
      }
      const float av[2][4] = {{a[0].x, a[0].y, a[0].z, a[0].w}, {a[1].x, a[1].y, a[1].z, a[1].w}};
      const float bv[2][4] = {{b[0].x, b[0].y, b[0].z, b[0].w}, {b[1].x, b[1].y, b[1].z, b[1].w}};
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(av[i][s]),
                                                             static_cast<double>(bv[j][s]), acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t m = m0 + wm + 16 * i + 4 * r + g;
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < 2; ++j) y[m * N + n0 + wc + 16 * j + l16] = acc[i][j][r];
    }
}

__global__ __launch_bounds__(256) void calib_zero_kernel(int32_t* __restrict__ counts, int32_t S) {
  for (int32_t s = blockIdx.x * 256 + threadIdx.x; s < S; s += gridDim.x * 256) counts[s] = 0;
}

__global__ __launch_bounds__(256) void calib_count_kernel(const int32_t* __restrict__ tok2stream, int32_t M,
                                                          int32_t S, int32_t* __restrict__ counts) {
  __shared__ int32_t bins[kCalibMaxStreams];
  for (int32_t s = threadIdx.x; s < S; s += 256) bins[s] = 0;
  __syncthreads();
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < M;
       i += static_cast<int64_t>(gridDim.x) * 256) {
    const int32_t s = tok2stream[i];
    if (static_cast<uint32_t>(s) < static_cast<uint32_t>(S)) atomicAdd(&bins[s], 1);
  }
  __syncthreads();
  for (int32_t s = threadIdx.x; s < S; s += 256)
    if (bins[s] != 0) atomicAdd(&counts[s], bins[s]);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// One wave per row; four rows per workgroup.
__global__ __launch_bounds__(256) void calib_row_error_kernel(const float* __restrict__ yq,
                                                              const double* __restrict__ ref,
                                                              const int32_t* __restrict__ tok2stream,
                                                              const int32_t* __restrict__ counts,
                                                              const double* __restrict__ omega, int32_t M,
                                                              int32_t N, int32_t S, double* __restrict__ err) {
  const int64_t i = static_cast<int64_t>(flat_wg()) * 4 + (threadIdx.x >> 6);
  if (i >= M) return;
  const int lane = threadIdx.x & 63;
  const float4* yr = reinterpret_cast<const float4*>(yq + i * N);
  const double2* rr = reinterpret_cast<const double2*>(ref + i * N);
  double acc = 0.0;
#pragma unroll 4
  for (int32_t j = lane; j < N / 4; j += 64) {
    const float4 a = yr[j];
    const double2 b0 = rr[2 * j], b1 = rr[2 * j + 1];
    const double e0 = static_cast<double>(a.x) - b0.x, e1 = static_cast<double>(a.y) - b0.y;
    const double e2 = static_cast<double>(a.z) - b1.x, e3 = static_cast<double>(a.w) - b1.y;
    acc = fma(e0, e0, acc);
    acc = fma(e1, e1, acc);
    acc = fma(e2, e2, acc);
    acc = fma(e3, e3, acc);
  }
  acc = wave_sum(acc);
  if (lane == 0) {
    const int32_t s = tok2stream[i];
    double w = 0.0;
    if (static_cast<uint32_t>(s) < static_cast<uint32_t>(S)) w = omega[s] / static_cast<double>(counts[s]);
    err[i] = w * acc;
  }
}

// One workgroup, fixed order; eight loads in flight per thread.
constexpr int kSumThreads = 1024;
__global__ __launch_bounds__(kSumThreads) void calib_sum_kernel(const double* __restrict__ part, int64_t n,
                                                                double* __restrict__ out) {
  __shared__ double wsum[kSumThreads / 64];
  double acc = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 8 * kSumThreads) {
    double v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = i + j * kSumThreads < n ? part[i + j * kSumThreads] : 0.0;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc += v[j];
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x < 64) {
    acc = wave_sum(threadIdx.x < kSumThreads / 64 ? wsum[threadIdx.x] : 0.0);
    if (threadIdx.x == 0) *out = acc;
  }
}

__global__ __launch_bounds__(256) void calib_row_weight_kernel(const int32_t* __restrict__ tok2stream,
                                                               const int32_t* __restrict__ counts,
                                                               const double* __restrict__ omega, int32_t M, int32_t S,
                                                               double* __restrict__ weight) {
  const int32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i >= M) return;
  const int32_t s = tok2stream[i];
  weight[i] = static_cast<uint32_t>(s) < static_cast<uint32_t>(S) ? omega[s] / static_cast<double>(counts[s]) : 0.0;
}

// ---------------------------------------------------------------- shared channel scaling (Eq. 7)
// Per-channel absolute maxima by atomic max on the bits of |v| (non-negative
// floats order like their bit patterns; the result does not depend on the
// order), then d_k = amax|X_k|^alpha / amax|W_k|^(1 - alpha) in fp64, clamped
// to [2^-6, 2^6], and dinv = 1 / d in fp32.
__global__ __launch_bounds__(256) void calib_fill_kernel(float* __restrict__ p, int32_t n, float v) {
  for (int32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) p[i] = v;
}

__global__ __launch_bounds__(256) void calib_zero_u32_kernel(uint32_t* __restrict__ p, int32_t n) {
  for (int32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) p[i] = 0u;
}

// A workgroup covers 32 x CH channels (CH = 8 bf16 or 4 fp32: one 16-byte
// load per row) and a range of rows (grid.y); its eight row lanes take every
// eighth row, meet in LDS, and one atomic max per channel leaves the
// workgroup.
constexpr int kAmaxLanes = 32;
template <bool BF16>
__global__ __launch_bounds__(256) void channel_amax_kernel(const void* __restrict__ src, int64_t rows, int32_t K,
                                                           int64_t rows_per_block, uint32_t* __restrict__ amax) {
  constexpr int CH = BF16 ? 8 : 4;
  constexpr int WCH = kAmaxLanes * CH;  // channels per workgroup
  __shared__ uint32_t red[8][WCH];
  const int cl = threadIdx.x % kAmaxLanes, rl = threadIdx.x / kAmaxLanes;
  const int32_t k0 = blockIdx.x * WCH + cl * CH;
  const int64_t r0 = static_cast<int64_t>(blockIdx.y) * rows_per_block;
  const int64_t r1 = min(rows, r0 + rows_per_block);
  const size_t row_bytes = static_cast<size_t>(K) * (BF16 ? 2 : 4);
  uint32_t m[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) m[c] = 0u;
  if (k0 < K) {
    const uint8_t* base = static_cast<const uint8_t*>(src) + static_cast<size_t>(k0) * (BF16 ? 2 : 4);
#pragma unroll 4
    for (int64_t r = r0 + rl; r < r1; r += 8) {
      const uint4 v = *reinterpret_cast<const uint4*>(base + static_cast<size_t>(r) * row_bytes);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const uint32_t b = BF16 ? ((w[c >> 1] >> (16 * (c & 1))) & 0x7FFFu) << 16 : w[c] & 0x7FFFFFFFu;
        m[c] = max(m[c], b);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < CH; ++c) red[rl][cl * CH + c] = m[c];
  __syncthreads();
  if (threadIdx.x < WCH) {
    uint32_t v = red[0][threadIdx.x];
#pragma unroll
    for (int i = 1; i < 8; ++i) v = max(v, red[i][threadIdx.x]);
    const int32_t k = blockIdx.x * WCH + threadIdx.x;
    if (k < K && v != 0u) atomicMax(&amax[k], v);
  }
}

__global__ __launch_bounds__(256) void smooth_scale_kernel(const uint32_t* __restrict__ ax_bits,
                                                           const uint32_t* __restrict__ aw_bits, int32_t K,
                                                           float alpha, float* __restrict__ d,
                                                           float* __restrict__ dinv) {
  const int32_t k = blockIdx.x * 256 + threadIdx.x;
  if (k >= K) return;
  const double ax = static_cast<double>(__uint_as_float(ax_bits[k]));
  const double aw = static_cast<double>(__uint_as_float(aw_bits[k]));
  const double a = static_cast<double>(alpha);
  double v = 1.0;
  if (ax > 0.0 && aw > 0.0) v = pow(ax, a) / pow(aw, 1.0 - a);
  const float dk = static_cast<float>(fmin(fmax(v, 0.015625), 64.0));
  d[k] = dk;
  dinv[k] = 1.0f / dk;
}

// ---------------------------------------------------------------- constrained search
// Compass search over (log gamma_1 .. log gamma_S, log c).  State in device
// memory: st = {unused, h, log c}, u = the incumbent's log gains, and the
// caller's gamma / clip / objective outputs hold the incumbent's evaluated
// values.  Candidate j of a round moves coordinate j/2 (the gains, then the
// threshold) by +h (j even) or -h (j odd).

__device__ __forceinline__ double clampd(double v, double lo, double hi) { return fmin(fmax(v, lo), hi); }
__device__ __forceinline__ float clampf_(float v, float lo, float hi) { return fminf(fmaxf(v, lo), hi); }

__global__ __launch_bounds__(64) void calib_search_init_kernel(SearchBounds b, int32_t S, double* st, double* u,
                                                               float* gamma, float* clip) {
  for (int32_t s = threadIdx.x; s < S; s += 64) {
    u[s] = 0.0;
    gamma[s] = 1.0f;
  }
  if (threadIdx.x == 0) {
    const float c = clampf_(b.clip_init, b.clip_min, b.clip_max);
    clip[0] = c;
    st[0] = 0.0;
    st[1] = static_cast<double>(b.log_step);
    st[2] = log(static_cast<double>(c));
  }
}

// One thread per candidate (C = 2 (S + 1) <= 256).  A gain step is projected
// onto lo <= u_s <= hi, sum_s n_s u_s = 0 (nearest point in the token-
// weighted norm: u_s = clamp(w_s - lam) for streams with tokens, lam by 64
// bisection halvings in fp64); a threshold step is clamped to the log bounds.
__global__ __launch_bounds__(256) void calib_propose_kernel(SearchBounds b, int32_t S, const int32_t* counts,
                                                            const double* st, const double* u, double* cand_u,
                                                            double* cand_v, float* cand_gamma, float* cand_clip) {
  const int32_t C = 2 * (S + 1);
  const int32_t j = threadIdx.x;
  if (j >= C) return;
  const int32_t d = j >> 1;
  const double step = (j & 1) ? -st[1] : st[1];
  const double lo = log(static_cast<double>(b.gamma_min)), hi = log(static_cast<double>(b.gamma_max));
  double* uj = cand_u + static_cast<size_t>(j) * S;
  double vc = st[2];
  if (d < S) {
    bool any = false;
    double wmin = 0.0, wmax = 0.0;
    for (int32_t s = 0; s < S; ++s) {
      const double w = u[s] + (s == d ? step : 0.0);
      if (counts[s] > 0) {
        wmin = any ? fmin(wmin, w) : w;
        wmax = any ? fmax(wmax, w) : w;
        any = true;
      }
    }
    double lam = 0.0;
    if (any) {
      double a = wmin - hi, c = wmax - lo;
      for (int it = 0; it < 64; ++it) {
        const double mid = 0.5 * (a + c);
        double f = 0.0;
        for (int32_t s = 0; s < S; ++s) {
          if (counts[s] <= 0) continue;
          const double w = u[s] + (s == d ? step : 0.0);
          f += static_cast<double>(counts[s]) * clampd(w - mid, lo, hi);
        }
        if (f > 0.0)
          a = mid;
        else
          c = mid;
      }
      lam = 0.5 * (a + c);
    }
    for (int32_t s = 0; s < S; ++s) {
      const double w = u[s] + (s == d ? step : 0.0);
      uj[s] = counts[s] > 0 ? clampd(w - lam, lo, hi) : clampd(w, lo, hi);
    }
  } else {
    for (int32_t s = 0; s < S; ++s) uj[s] = u[s];
    vc = clampd(vc + step, log(static_cast<double>(b.clip_min)), log(static_cast<double>(b.clip_max)));
  }
  for (int32_t s = 0; s < S; ++s)
    cand_gamma[static_cast<size_t>(j) * S + s] =
        clampf_(static_cast<float>(exp(uj[s])), b.gamma_min, b.gamma_max);
  cand_v[j] = vc;
  cand_clip[j] = clampf_(static_cast<float>(exp(vc)), b.clip_min, b.clip_max);
}

// The first candidate with the smallest objective replaces the incumbent if
// strictly better; otherwise the step halves.
__global__ __launch_bounds__(64) void calib_select_kernel(int32_t S, const double* cand_obj, const double* cand_u,
                                                          const double* cand_v, const float* cand_gamma,
                                                          const float* cand_clip, double* st, double* u,
                                                          float* gamma, float* clip, double* objective) {
  const int32_t C = 2 * (S + 1);
  int32_t best = 0;
  for (int32_t j = 1; j < C; ++j)
    if (cand_obj[j] < cand_obj[best]) best = j;
  const bool better = cand_obj[best] < objective[0];
  __syncthreads();  // every thread has read objective[0] before it changes
  if (better) {
    for (int32_t s = threadIdx.x; s < S; s += 64) {
      u[s] = cand_u[static_cast<size_t>(best) * S + s];
      gamma[s] = cand_gamma[static_cast<size_t>(best) * S + s];
    }
    if (threadIdx.x == 0) {
      st[2] = cand_v[best];
      clip[0] = cand_clip[best];
      objective[0] = cand_obj[best];
    }
  } else if (threadIdx.x == 0) {
    st[1] = 0.5 * st[1];
  }
}

}  // namespace

hipError_t launch_calib_search_init(const SearchBounds& b, int32_t S, double* st, double* u, float* gamma,
                                    float* clip, hipStream_t s) {
  hipLaunchKernelGGL(calib_search_init_kernel, dim3(1), dim3(64), 0, s, b, S, st, u, gamma, clip);
  return hipGetLastError();
}

hipError_t launch_calib_propose(const SearchBounds& b, int32_t S, const int32_t* counts, const double* st,
                                const double* u, double* cand_u, double* cand_v, float* cand_gamma,
                                float* cand_clip, hipStream_t s) {
  hipLaunchKernelGGL(calib_propose_kernel, dim3(1), dim3(256), 0, s, b, S, counts, st, u, cand_u, cand_v,
                     cand_gamma, cand_clip);
  return hipGetLastError();
}

hipError_t launch_calib_select(int32_t S, const double* cand_obj, const double* cand_u, const double* cand_v,
                               const float* cand_gamma, const float* cand_clip, double* st, double* u,
                               float* gamma, float* clip, double* objective, hipStream_t s) {
  hipLaunchKernelGGL(calib_select_kernel, dim3(1), dim3(64), 0, s, S, cand_obj, cand_u, cand_v, cand_gamma,
                     cand_clip, st, u, gamma, clip, objective);
  return hipGetLastError();
}

hipError_t launch_calib_reference(const CalibRefArgs& a, hipStream_t s) {
  const int32_t tiles_m = (a.M + kRefTile - 1) / kRefTile, tiles_n = a.N / kRefTile;
  const dim3 grid = wg_grid(static_cast<size_t>(tiles_m) * tiles_n);
  if (a.wf != nullptr)
    hipLaunchKernelGGL(calib_reference_kernel<true>, grid, dim3(256), 0, s, a.x, nullptr, nullptr, nullptr, a.wf, a.y,
                       a.M, a.N, a.K, 0, tiles_m, tiles_n);
  else
    hipLaunchKernelGGL(calib_reference_kernel<false>, grid, dim3(256), 0, s, a.x, a.dinv, a.qw, a.w_scale, nullptr,
                       a.y, a.M, a.N, a.K, a.w_group, tiles_m, tiles_n);
  return hipGetLastError();
}

namespace {
void launch_amax(bool bf16, const void* src, int64_t rows, int32_t K, uint32_t* amax, hipStream_t s) {
  const int64_t rpb = 256;  // rows per workgroup: one atomic per channel per 256 rows
  const int64_t yb = (rows + rpb - 1) / rpb;
  const int64_t ybc = yb < 65535 ? yb : 65535;
  const int64_t per = (rows + ybc - 1) / ybc;
  const int wch = kAmaxLanes * (bf16 ? 8 : 4);
  const dim3 grid((K + wch - 1) / wch, static_cast<unsigned>(ybc));
  if (bf16)
    hipLaunchKernelGGL(channel_amax_kernel<true>, grid, dim3(256), 0, s, src, rows, K, per, amax);
  else
    hipLaunchKernelGGL(channel_amax_kernel<false>, grid, dim3(256), 0, s, src, rows, K, per, amax);
}
}  // namespace

hipError_t launch_channel_amax(const uint16_t* x, int32_t M, const float* w, int32_t N, int32_t K,
                               uint32_t* ax_bits, uint32_t* aw_bits, hipStream_t s) {
  hipLaunchKernelGGL(calib_zero_u32_kernel, dim3((K + 255) / 256), dim3(256), 0, s, ax_bits, K);
  hipLaunchKernelGGL(calib_zero_u32_kernel, dim3((K + 255) / 256), dim3(256), 0, s, aw_bits, K);
  launch_amax(true, x, M, K, ax_bits, s);
  launch_amax(false, w, N, K, aw_bits, s);
  return hipGetLastError();
}

hipError_t launch_smooth_scales(const uint32_t* ax_bits, const uint32_t* aw_bits, int32_t K, float alpha, float* d,
                                float* dinv, hipStream_t s) {
  hipLaunchKernelGGL(smooth_scale_kernel, dim3((K + 255) / 256), dim3(256), 0, s, ax_bits, aw_bits, K, alpha, d,
                     dinv);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, int32_t n, float v, hipStream_t s) {
  hipLaunchKernelGGL(calib_fill_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_calib_counts(const int32_t* tok2stream, int32_t M, int32_t S, int32_t* counts, hipStream_t s) {
  hipLaunchKernelGGL(calib_zero_kernel, dim3((S + 255) / 256), dim3(256), 0, s, counts, S);
  const int64_t want = (static_cast<int64_t>(M) + 4095) / 4096;  // about 16 rows per thread
  const int grid = static_cast<int>(want < 1024 ? want : 1024);
  hipLaunchKernelGGL(calib_count_kernel, dim3(grid), dim3(256), 0, s, tok2stream, M, S, counts);
  return hipGetLastError();
}

hipError_t launch_calib_error(const float* yq, const double* ref, const int32_t* tok2stream,
                              const int32_t* counts, const double* omega, int32_t M, int32_t N, int32_t S,
                              double* err, double* out, hipStream_t s) {
  const size_t wgs = (static_cast<size_t>(M) + 3) / 4;
  hipLaunchKernelGGL(calib_row_error_kernel, wg_grid(wgs), dim3(256), 0, s, yq, ref, tok2stream, counts, omega,
                     M, N, S, err);
  return launch_calib_sum(err, static_cast<size_t>(M), out, s);
}

hipError_t launch_calib_sum(const double* part, size_t n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(calib_sum_kernel, dim3(1), dim3(kSumThreads), 0, s, part, static_cast<int64_t>(n), out);
  return hipGetLastError();
}

hipError_t launch_calib_row_weight(const int32_t* tok2stream, const int32_t* counts, const double* omega, int32_t M,
                                   int32_t S, double* weight, hipStream_t s) {
  hipLaunchKernelGGL(calib_row_weight_kernel, dim3((M + 255) / 256), dim3(256), 0, s, tok2stream, counts, omega, M, S,
                     weight);
  return hipGetLastError();
}

}  // namespace sq
