// Draft-side rejection predictor (Sec. 3.3, Sec. 4.1, App. B): the summary statistics of a draft
// model's next-token distribution (confidence, entropy, top-2 margin, dispersion of the
// logits) and the small MLP that maps them to the probability that the drafted token is
// accepted.  Declared in include/wisp.h.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/wisp.h"
#include "kernels.h"

namespace wisp {
wisp_status report_error(wisp_status st, const char *msg);
}

namespace {

// The statistics are formed in base 2: y = logits * log2(e) / T, so exp(z - m) = 2^(y - m')
// is one hardware exp2.  A row is cut into chunks of kChunk entries, one workgroup per
// (row, chunk); each thread sums its entries in fp32, each wave its lanes in fp32,
// the workgroup merges its waves in fp64, and a second kernel merges the chunks of a row in
// fixed order.  The partial state of a set of entries:
//   m  max y,  s = sum 2^(y - m),  c = sum (y - m) 2^(y - m)  (centred on m: no cancellation
//   against large logits),  v1 >= v2 the two largest y (as a multiset: a repeated maximum
//   gives v2 = v1),  d1 = sum (y - y_0),  d2 = sum (y - y_0)^2 with y_0 the row's first entry.
// Moving the centre from m to m' >= m: s' = r s, c' = r (c + (m - m') s) with r = 2^(m - m').
constexpr int kChunk = 8192;
constexpr float kLog2e = 1.4426950408889634f;

template <typename F>
struct St {
  F m, s, c, v1, v2, d1, d2;
};
using Part = St<double>;

// Reductions over a wave on the VALU: lanes l ^ 1, l ^ 2 by quad permutes, the other quad and
// the other half of a 16-lane row by mirrors (every lane of a quad, then of an octet, already
// holds the same value), rows by lane swaps.  The same pairs as a butterfly in steps 1, 2, 4,
// 8, 16, 32, every lane ending with the same bits.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  const int i = __float_as_int(v);
  return __int_as_float(__builtin_amdgcn_update_dpp(i, i, CTRL, 0xF, 0xF, false));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;

__device__ __forceinline__ float wave_sum(float v) {
  v += dpp<kXor1>(v);
  v += dpp<kXor2>(v);
  v += dpp<kHalfMirror>(v);
  v += dpp<kMirror>(v);
  return wisp::xor32_sum(wisp::xor16_sum(v));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp<kXor1>(v));
  v = fmaxf(v, dpp<kXor2>(v));
  v = fmaxf(v, dpp<kHalfMirror>(v));
  v = fmaxf(v, dpp<kMirror>(v));
  return wisp::xor32_max(wisp::xor16_max(v));
}
// the two largest of the wave's pairs (v1 >= v2), as a multiset
__device__ __forceinline__ void top2(float &v1, float &v2, float o1, float o2) {
  v2 = fmaxf(fminf(v1, o1), fmaxf(v2, o2));
  v1 = fmaxf(v1, o1);
}
__device__ __forceinline__ void wave_top2(float &v1, float &v2) {
  top2(v1, v2, dpp<kXor1>(v1), dpp<kXor1>(v2));
  top2(v1, v2, dpp<kXor2>(v1), dpp<kXor2>(v2));
  top2(v1, v2, dpp<kHalfMirror>(v1), dpp<kHalfMirror>(v2));
  top2(v1, v2, dpp<kMirror>(v1), dpp<kMirror>(v2));
  top2(v1, v2, __shfl_xor(v1, 16), __shfl_xor(v2, 16));
  top2(v1, v2, __shfl_xor(v1, 32), __shfl_xor(v2, 32));
}

template <typename F>
__device__ __forceinline__ St<F> merge(const St<F> &a, const St<F> &b) {
  St<F> r;
  r.m = a.m > b.m ? a.m : b.m;
  // an empty side (s = 0, m = -inf) contributes nothing: (m - r.m) * s would be -inf * 0
  const F ea = a.s > F(0) ? (F)exp2((double)(a.m - r.m)) : F(0);
  const F eb = b.s > F(0) ? (F)exp2((double)(b.m - r.m)) : F(0);
  r.s = a.s * ea + b.s * eb;
  r.c = (a.s > F(0) ? ea * (a.c + (a.m - r.m) * a.s) : F(0)) + (b.s > F(0) ? eb * (b.c + (b.m - r.m) * b.s) : F(0));
  r.v1 = a.v1 > b.v1 ? a.v1 : b.v1;
  const F lo = a.v1 > b.v1 ? b.v1 : a.v1, hi2 = a.v2 > b.v2 ? a.v2 : b.v2;
  r.v2 = lo > hi2 ? lo : hi2;
  r.d1 = a.d1 + b.d1;
  r.d2 = a.d2 + b.d2;
  return r;
}

template <typename F>
__device__ __forceinline__ St<F> shfl(const St<F> &a, int o) {
  return St<F>{__shfl_xor(a.m, o), __shfl_xor(a.s, o), __shfl_xor(a.c, o), __shfl_xor(a.v1, o),
               __shfl_xor(a.v2, o), __shfl_xor(a.d1, o), __shfl_xor(a.d2, o)};
}

__device__ __forceinline__ Part widen(const St<float> &a) {
  return Part{a.m, a.s, a.c, a.v1, a.v2, a.d1, a.d2};
}

// grid (chunks, rows), 256 threads; thread t holds entries 4 (t + 256 k) .. + 3 of its chunk
// (16-byte loads) when the row allows them, else entries t + 256 k.  HBM-bound as long as the
// VALU keeps up: with the entries in registers the thread's maximum comes first, so every
// entry costs one exp2 and eight other instructions and no branch (the second largest is the
// median of the running pair and the entry); the wave then agrees on one maximum, each lane
// rescales once, and the sums cross the lanes on the VALU.  256 rows of 128256: a running
// maximum with rescaling and 6 merge steps through LDS took 30 us, this 28, and 23.7 (5.5
// TB/s) with non-temporal loads.
template <bool VEC>
__global__ __launch_bounds__(256) void stats_chunk_kernel(const float *__restrict__ logits, int V, int64_t ld,
                                                          float sc, Part *__restrict__ parts) {
  constexpr int PER = kChunk / 256;
  const int c = blockIdx.x, nch = gridDim.x;
  const int64_t row = blockIdx.y;
  const float *x = logits + row * ld;
  const float y0 = x[0] * sc;
  const int base = c * kChunk, n = min(V - base, kChunk);
  float y[PER];
  bool full;   // every entry of this thread exists
  if constexpr (VEC) {
    const float4 *x4 = reinterpret_cast<const float4 *>(x + base);
    float4 buf[PER / 4];
#pragma unroll
    for (int k = 0; k < PER / 4; ++k) {        // all loads of the thread in flight at once
      const int e = (k * 256 + threadIdx.x) * 4;
      buf[k] = float4{0.f, 0.f, 0.f, 0.f};
      if (e + 4 <= n) {
        buf[k] = __builtin_bit_cast(float4, wisp::ld16_stream(x4 + k * 256 + threadIdx.x));
      } else if (e < n) {
        buf[k].x = x[base + e];
        if (e + 1 < n) buf[k].y = x[base + e + 1];
        if (e + 2 < n) buf[k].z = x[base + e + 2];
      }
    }
#pragma unroll
    for (int k = 0; k < PER / 4; ++k) {
      y[4 * k] = buf[k].x * sc;
      y[4 * k + 1] = buf[k].y * sc;
      y[4 * k + 2] = buf[k].z * sc;
      y[4 * k + 3] = buf[k].w * sc;
    }
    full = ((PER / 4 - 1) * 256 + (int)threadIdx.x) * 4 + 4 <= n;
  } else {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int e = k * 256 + threadIdx.x;
      y[k] = e < n ? x[base + e] * sc : 0.f;
    }
    full = (PER - 1) * 256 + (int)threadIdx.x < n;
  }
  auto exists = [&](int k) {
    return full || (VEC ? ((k >> 2) * 256 + (int)threadIdx.x) * 4 + (k & 3) : k * 256 + (int)threadIdx.x) < n;
  };
  float v1 = -INFINITY, v2 = -INFINITY, d1 = 0.f, d2 = 0.f;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (!exists(k)) y[k] = -INFINITY;
    const float d = exists(k) ? y[k] - y0 : 0.f;
    d1 += d;
    d2 = fmaf(d, d, d2);
    v2 = __builtin_amdgcn_fmed3f(v1, v2, y[k]);
    v1 = fmaxf(v1, y[k]);
  }
  const float m = v1;
  float s = 0.f, cs = 0.f;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const float u = y[k] - m;
    const float e = __builtin_amdgcn_exp2f(u);
    if (exists(k)) {   // an entry past the end has u = -inf: 0 x inf stays out of the sum
      s += e;
      cs = fmaf(u, e, cs);
    }
  }
  // the wave's common maximum, one rescaling per lane (a lane without entries adds nothing)
  const float mw = wave_max(m);
  const float up = m - mw;
  const float r = s > 0.f ? __builtin_amdgcn_exp2f(up) : 0.f;
  cs = s > 0.f ? r * fmaf(up, s, cs) : 0.f;
  s *= r;
  St<float> a{mw, wave_sum(s), wave_sum(cs), v1, v2, wave_sum(d1), wave_sum(d2)};
  wave_top2(a.v1, a.v2);
  __shared__ Part sh[4];
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = widen(a);
  __syncthreads();
  if (threadIdx.x == 0) parts[row * nch + c] = merge(merge(sh[0], sh[1]), merge(sh[2], sh[3]));
}

// one wave per row: lane l merges chunks l, l + 64, ... in order, then the wave merges (fp64)
__global__ __launch_bounds__(64) void stats_final_kernel(const Part *__restrict__ parts, int nch, int V,
                                                         float4 *__restrict__ stats) {
  const int64_t row = blockIdx.x;
  const int lane = threadIdx.x;
  Part p{-INFINITY, 0.0, 0.0, -INFINITY, -INFINITY, 0.0, 0.0};
  for (int c = lane; c < nch; c += 64) p = merge(p, parts[row * nch + c]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) p = merge(p, shfl(p, o));
  if (lane == 0) {
    const double ln2 = 0.6931471805599453;
    const double p1 = 1.0 / p.s;                       // 2^(v1 - m) = 1
    const double p2 = exp2(p.v2 - p.m) / p.s;          // 0 when V = 1
    const double H = log(p.s) - ln2 * (p.c / p.s);     // -sum p ln p
    const double mean = p.d1 / V;
    const double var = fmax(p.d2 / V - mean * mean, 0.0);
    stats[row] = make_float4((float)p1, (float)H, (float)(p1 - p2), (float)(sqrt(var) * ln2));
  }
}

constexpr int kH1 = 512, kH2 = 128, kH3 = 64;

struct MlpArgs {
  int n_in;
  const float *mean, *inv_std, *w1, *b1, *w2, *b2, *w3, *b3, *w4;
  float b4;
};

// Sums of N values per lane over the wave, N a power of two: at each step the lanes of a pair
// keep half of the values and exchange the other half, so lane l ends with the sum of value
// index l >> (6 - log2 N) after N - 1 + 6 - log2 N exchanges instead of 6 N.  The pairs are
// those of a butterfly in steps 32, 16, .., 1.
template <int N>
__device__ __forceinline__ float wave_sums(const float (&v)[N], int lane, int step = 32) {
  if constexpr (N == 1) {
    float s = v[0];
    for (int o = step; o > 0; o >>= 1) s += __shfl_xor(s, o);
    return s;
  } else {
    const bool hi = lane & step;
    float w[N / 2];
#pragma unroll
    for (int k = 0; k < N / 2; ++k)
      w[k] = (hi ? v[N / 2 + k] : v[k]) + __shfl_xor(hi ? v[k] : v[N / 2 + k], step);
    return wave_sums<N / 2>(w, lane, step >> 1);
  }
}

// One workgroup of 16 waves per R feature rows.  Layers 2 and 3: each wave owns 8 (4) outputs;
// for one output the 64 lanes read a contiguous stretch of its weight row.  Latency-bound (0.3
// MB of cached weights): every weight a thread needs is in flight before the first layer, so
// the layers themselves only wait for each other (4 waves that loaded 4 rows at a time and
// reduced each output by 6 shuffles took 16.6 us for 32 rows and 24.5 for 1024, this 7.9 and
// 9.7).  Several rows per workgroup
// once they outnumber the CUs: the weights then come from L2 once for all of them.
template <int R>
__global__ __launch_bounds__(1024) void reject_mlp_kernel(MlpArgs p, const float *__restrict__ feat, int rows,
                                                          float *__restrict__ prob) {
  __shared__ float x[R][8], h1[R][kH1], h2[R][kH2], h3[R][kH3];
  const int row0 = blockIdx.x * R, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float4 w2[8][2];
  const int o2 = wave * 8, o3 = wave * 4;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float4 *w = reinterpret_cast<const float4 *>(p.w2 + (int64_t)(o2 + j) * kH1 + lane * 8);
    w2[j][0] = w[0];
    w2[j][1] = w[1];
  }
  float2 w3[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) w3[j] = *reinterpret_cast<const float2 *>(p.w3 + (int64_t)(o3 + j) * kH2 + lane * 2);
  const float b2 = p.b2[o2 + (lane >> 3)], b3 = p.b3[o3 + (lane >> 4)], w4 = p.w4[lane];
  float w1[8], b1 = 0.f;
  if (tid < kH1) {
    b1 = p.b1[tid];
#pragma unroll
    for (int k = 0; k < 8; ++k) w1[k] = k < p.n_in ? p.w1[tid * p.n_in + k] : 0.f;
  }
  if (tid < R * p.n_in) {
    const int r = tid / p.n_in, k = tid % p.n_in;
    x[r][k] = (feat[(int64_t)min(row0 + r, rows - 1) * p.n_in + k] - p.mean[k]) * p.inv_std[k];
  }
  __syncthreads();
  if (tid < kH1) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float acc = b1;
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (k < p.n_in) acc = fmaf(w1[k], x[r][k], acc);
      h1[r][tid] = fmaxf(acc, 0.f);
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {                                // 512 inputs: 8 per lane, 8 outputs per wave
    const float4 ha = *reinterpret_cast<const float4 *>(&h1[r][lane * 8]);
    const float4 hb = *reinterpret_cast<const float4 *>(&h1[r][lane * 8 + 4]);
    const float hx[8] = {ha.x, ha.y, ha.z, ha.w, hb.x, hb.y, hb.z, hb.w};
    float s[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float w8[8] = {w2[j][0].x, w2[j][0].y, w2[j][0].z, w2[j][0].w,
                           w2[j][1].x, w2[j][1].y, w2[j][1].z, w2[j][1].w};
      s[j] = 0.f;
#pragma unroll
      for (int k = 0; k < 8; ++k) s[j] = fmaf(w8[k], hx[k], s[j]);
    }
    const float v = wave_sums<8>(s, lane);
    if ((lane & 7) == 0) h2[r][o2 + (lane >> 3)] = fmaxf(v + b2, 0.f);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) {                                // 128 inputs: 2 per lane, 4 outputs per wave
    const float ha = h2[r][lane * 2], hb = h2[r][lane * 2 + 1];
    float s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = fmaf(w3[j].y, hb, w3[j].x * ha);
    const float v = wave_sums<4>(s, lane);
    if ((lane & 15) == 0) h3[r][o3 + (lane >> 4)] = fmaxf(v + b3, 0.f);
  }
  __syncthreads();
  if (wave < R && row0 + wave < rows) {
    const float s[1] = {w4 * h3[wave][lane]};
    const float v = wave_sums<1>(s, lane);
    if (lane == 0) prob[row0 + wave] = 1.f / (1.f + expf(-(v + p.b4)));
  }
}

}  // namespace

using wisp::report_error;

extern "C" size_t wisp_draft_stats_workspace_size(int32_t rows, int32_t vocab) {
  if (rows < 0 || vocab < 1) return 0;
  return (size_t)rows * (size_t)((vocab + kChunk - 1) / kChunk) * sizeof(Part);
}

extern "C" wisp_status wisp_draft_stats(const float *logits, int32_t rows, int32_t vocab, int64_t ld,
                                        float temperature, float *stats, void *workspace, size_t workspace_bytes,
                                        void *stream) {
  if (rows < 0 || vocab < 1 || ld < vocab || !(temperature > 0.f))
    return report_error(WISP_E_INVALID, "wisp_draft_stats: rows < 0, vocab < 1, ld < vocab or temperature <= 0");
  if (rows == 0) return WISP_OK;
  if (rows > 65535) return report_error(WISP_E_UNSUPPORTED, "wisp_draft_stats: more than 65535 rows in one call");
  if (!logits || !stats || !workspace) return report_error(WISP_E_INVALID, "wisp_draft_stats: NULL pointer");
  if (((uintptr_t)stats & 15) != 0 || ((uintptr_t)workspace & 15) != 0)
    return report_error(WISP_E_INVALID, "wisp_draft_stats: stats or workspace not 16-byte aligned");
  if (workspace_bytes < wisp_draft_stats_workspace_size(rows, vocab))
    return report_error(WISP_E_WORKSPACE, "wisp_draft_stats: workspace too small");
  const int nch = (vocab + kChunk - 1) / kChunk;
  const bool vec = ((uintptr_t)logits & 15) == 0 && ld % 4 == 0;
  Part *parts = reinterpret_cast<Part *>(workspace);
  const hipStream_t s = (hipStream_t)stream;
  wisp::launch(vec ? stats_chunk_kernel<true> : stats_chunk_kernel<false>, dim3(nch, rows), dim3(256), 0, s, logits,
               (int)vocab, (int64_t)ld, kLog2e / temperature, parts);
  wisp::launch(stats_final_kernel, dim3(rows), dim3(64), 0, s, (const Part *)parts, nch, (int)vocab,
               reinterpret_cast<float4 *>(stats));
  if (hipGetLastError() != hipSuccess) return report_error(WISP_E_HIP, "wisp_draft_stats: launch failed");
  return WISP_OK;
}

extern "C" wisp_status wisp_reject_predict(const wisp_reject_mlp *mlp, const float *features, int32_t rows,
                                           float *p_accept, void *stream) {
  if (!mlp || rows < 0) return report_error(WISP_E_INVALID, "wisp_reject_predict: NULL mlp or rows < 0");
  if (mlp->n_in < 1 || mlp->n_in > 8) return report_error(WISP_E_INVALID, "wisp_reject_predict: n_in outside 1..8");
  if (rows == 0) return WISP_OK;
  if (!features || !p_accept || !mlp->mean || !mlp->inv_std || !mlp->w1 || !mlp->b1 || !mlp->w2 || !mlp->b2 ||
      !mlp->w3 || !mlp->b3 || !mlp->w4)
    return report_error(WISP_E_INVALID, "wisp_reject_predict: NULL pointer");
  if (((uintptr_t)mlp->w2 & 15) != 0 || ((uintptr_t)mlp->w3 & 7) != 0)
    return report_error(WISP_E_INVALID, "wisp_reject_predict: w2 not 16-byte or w3 not 8-byte aligned");
  MlpArgs a{mlp->n_in, mlp->mean, mlp->inv_std, mlp->w1, mlp->b1, mlp->w2, mlp->b2, mlp->w3, mlp->b3, mlp->w4, mlp->b4};
  // rows per workgroup: one while every row can have a CU of its own
  const int per = rows <= 256 ? 1 : rows <= 512 ? 2 : 4;
  wisp::launch(per == 1 ? reject_mlp_kernel<1> : per == 2 ? reject_mlp_kernel<2> : reject_mlp_kernel<4>,
               dim3((rows + per - 1) / per), dim3(1024), 0, (hipStream_t)stream, a, features, (int)rows, p_accept);
  if (hipGetLastError() != hipSuccess) return report_error(WISP_E_HIP, "wisp_reject_predict: launch failed");
  return WISP_OK;
}
