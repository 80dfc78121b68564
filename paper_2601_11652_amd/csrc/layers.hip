// Per-row kernels of the verification step: embedding + RMSNorm, the fixed-order sum of
// split-K partials fused with residual add + RMSNorm, RoPE + in-place KV append
// (Sec. 4.5: the new rows' K/V are written into their pages at ctx_len .. ctx_len+gamma),
// and SwiGLU.  Activations that feed a bf16 GEMM are written straight into the packed
// 32x16-fragment layout the GEMM streams; fp32 models keep row-major activations.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace wisp {

// The row of workgroup b: 8 consecutive rows, whose 16-byte pieces share a 128-byte line of the
// packed activations (and slots of a V page), go to one XCD, as workgroups are dealt to the 8
// in turn.  Launched over whole blocks of 64 rows (row_blocks); from 64 rows on, as fewer rows
// are spread over all XCDs instead.  (1291 rows x 4096, 2 splits: 25 -> 19 us; dealt one by one,
// every line is written back in up to 8 parts.)
__device__ __forceinline__ int row_of_block(int b, int n) {
  return n < 64 ? b : (b & ~63) + (b & 7) * 8 + ((b >> 3) & 7);
}
static int row_blocks(int n) { return n < 64 ? n : (n + 63) / 64 * 64; }

// store 8 consecutive activation columns c..c+7 of row r
template <typename T>
__device__ __forceinline__ void store8(T *out, bool packed, int64_t r, int64_t c, int64_t K,
                                      const float *v);
template <>
__device__ __forceinline__ void store8<float>(float *out, bool, int64_t r, int64_t c, int64_t K,
                                             const float *v) {
#pragma unroll
  for (int e = 0; e < 8; ++e) out[r * K + c + e] = v[e];
}
template <>
__device__ __forceinline__ void store8<uint16_t>(uint16_t *out, bool packed, int64_t r, int64_t c,
                                                int64_t K, const float *v) {
  uint4 w;
  w.x = pack2bf(v[0], v[1]);
  w.y = pack2bf(v[2], v[3]);
  w.z = pack2bf(v[4], v[5]);
  w.w = pack2bf(v[6], v[7]);
  const int64_t o = packed ? packed_off(r, c, K) : r * K + c;
  *reinterpret_cast<uint4 *>(out + o) = w;
}

// Sum of the K-split partials of 8 consecutive fp32 columns, in fixed split order; S: the
// splits, or a bound on them above 4.  The loads of up to 8 splits are issued before the
// first add, past the last split once more the last (a branch per split would wait for one
// load after another; 16 splits at once would spill).
constexpr int kMaxSplits = 16;
template <int S>
__device__ __forceinline__ void sum_splits8(const float *__restrict__ p, int64_t stride, int splits, float (&a)[8]) {
  constexpr bool EXACT = S <= 4;
  constexpr int R = S > 8 ? 8 : S;
#pragma unroll
  for (int z0 = 0; z0 < S; z0 += R) {
    float4 v[R][2];
#pragma unroll
    for (int z = 0; z < R; ++z)
#pragma unroll
      for (int x = 0; x < 2; ++x)
        v[z][x] = *reinterpret_cast<const float4 *>(p + (EXACT ? z : min(z0 + z, splits - 1)) * stride + x * 4);
#pragma unroll
    for (int z = 0; z < R; ++z) {
      const float w[8] = {v[z][0].x, v[z][0].y, v[z][0].z, v[z][0].w, v[z][1].x, v[z][1].y, v[z][1].z, v[z][1].w};
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = z0 + z == 0 ? w[e] : EXACT || z0 + z < splits ? a[e] + w[e] : a[e];
    }
    if (S > R) asm volatile("" ::: "memory");
  }
}
// calls go(std::integral_constant<int, S>) for the instance that covers `splits`
template <typename F>
static void with_splits(int splits, F &&go) {
  if (splits <= 1) go(std::integral_constant<int, 1>{});
  else if (splits == 2) go(std::integral_constant<int, 2>{});
  else if (splits == 3) go(std::integral_constant<int, 3>{});
  else if (splits == 4) go(std::integral_constant<int, 4>{});
  else if (splits <= 8) go(std::integral_constant<int, 8>{});
  else go(std::integral_constant<int, kMaxSplits>{});
}

// 8 consecutive elements as floats; v16: the address is a multiple of 16 bytes
__device__ __forceinline__ void load8(const float *p, bool v16, float (&v)[8]) {
  if (v16) {
    const float4 a = *reinterpret_cast<const float4 *>(p), b = *reinterpret_cast<const float4 *>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = p[e];
  }
}
__device__ __forceinline__ void load8(const uint16_t *p, bool v16, float (&v)[8]) {
  if (v16) {
    const uint4 w = ld16(p);
    const uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[2 * e] = __uint_as_float(x[e] << 16);
      v[2 * e + 1] = __uint_as_float(x[e] & 0xFFFF0000u);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = bf2f(p[e]);
  }
}
static bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// ---------------------------------------------------------------------------------------
__global__ void rope_table_kernel(const int32_t *__restrict__ row_pos, float *__restrict__ cs, int M,
                                  int hd, float base) {
  const int h2 = hd / 2;
  const int n = M * h2;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
    const int r = t / h2, i = t % h2;
    const double inv = pow((double)base, -2.0 * i / hd);
    const double ang = (double)row_pos[r] * inv;
    cs[2 * t] = (float)cos(ang);
    cs[2 * t + 1] = (float)sin(ang);
  }
}

void rope_table(const StepDesc &d, float *cs, int M, int hd, float base, hipStream_t s) {
  const int n = M * hd / 2;
  launch(rope_table_kernel, (n + 255) / 256, 256, 0, s, d.row_pos, cs, M, hd, base);
}

// ---------------------------------------------------------------------------------------
// The two row kernels below hold a row in one workgroup, 8 columns per thread (dm <= 8192).
// With few rows they are bound by the chain of loads, so everything a thread reads is asked
// for at once, the norm's gain too; with many by HBM.
// ---------------------------------------------------------------------------------------
// Fixed-order sum over the threads of a block of up to 1024 (waves reduce by shuffles,
// then wave sums are added in wave order).
__device__ __forceinline__ float block_sum(float v, float *sh) {
  v = xor16_sum(xor32_sum(v));
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  float t = 0.f;
  for (int i = 0; i < nw; ++i) t += sh[i];
  return t;
}

// y = x / rms * g of the row whose columns c .. c + 7 this thread holds
template <typename T>
__device__ __forceinline__ void norm_store(float (&v)[8], const float (&g)[8], bool on, T *__restrict__ xn, bool packed,
                                           int64_t r, int c, int dm, float eps, float *sh) {
  float ss = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
  ss = block_sum(ss, sh);
  if (!on) return;
  const float inv = 1.0f / sqrtf(ss / (float)dm + eps);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = v[e] * inv * g[e];
  store8<T>(xn, packed, r, c, dm, v);
}

template <typename T>
__global__ __launch_bounds__(1024) void embed_norm_kernel(StepDesc d, const T *__restrict__ embed,
                                                          const T *__restrict__ gain,
                                                          const int32_t *__restrict__ tokens,
                                                          float *__restrict__ h, T *__restrict__ xn,
                                                          bool packed, bool e16, bool g16, int M, int dm, int V,
                                                          float eps) {
  __shared__ float sh[16];
  const int r = row_of_block(blockIdx.x, M);
  if (r >= M) return;
  const int c = threadIdx.x * 8;
  const bool on = c < dm;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, g[8];
  if (on) load8(gain + c, g16, g);
  int tok = tokens[r];
  if (tok < 0 || tok >= V) {
    if (threadIdx.x == 0) flag_error(d.err, kErrToken);
    tok = 0;
  }
  if (on) {
    load8(embed + (int64_t)tok * dm + c, e16, v);
    float *hr = h + (int64_t)r * dm + c;
    *reinterpret_cast<float4 *>(hr) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4 *>(hr + 4) = make_float4(v[4], v[5], v[6], v[7]);
  }
  norm_store<T>(v, g, on, xn, packed, r, c, dm, eps, sh);
}

static int row_threads(int dm) { return ((dm / 8 + 63) / 64) * 64; }

template <typename T>
void embed_norm(const StepDesc &d, const T *embed, const T *gain, const int32_t *tokens, float *h,
                T *xn, bool packed, int M, int dm, int V, float eps, hipStream_t s) {
  launch(embed_norm_kernel<T>, row_blocks(M), row_threads(dm), 0, s, d, embed, gain, tokens, h, xn, packed,
         aligned16(embed), aligned16(gain), M, dm, V, eps);
}

// Every split partial, the residual and the gain are loaded in one round, the new residual
// stays in registers for the norm.  (6 rows of 4096, one load after another: 7.4 us; now 5.1 with
// 8 splits, 6.8 with 16.  171 rows, 8 splits: 9.4 -> 7.9.  4102 rows, 1 split: 57 -> 44, 5.3 TB/s.)
template <typename T, int S>
__global__ __launch_bounds__(1024) void resid_norm_kernel(const float *__restrict__ part, int splits,
                                                          float *__restrict__ h,
                                                          const T *__restrict__ gain,
                                                          T *__restrict__ xn, bool packed, bool g16, int M,
                                                          int n_out, int dm, float eps,
                                                          const int32_t *__restrict__ rows) {
  __shared__ float sh[16];
  const int ro = row_of_block(blockIdx.x, n_out);   // output row
  if (ro >= n_out) return;
  const int r = rows ? rows[ro] : ro;               // source row
  const int c = threadIdx.x * 8;
  const bool on = c < dm;
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, g[8];
  if (on) {
    float *hr = h + (int64_t)r * dm + c;
    const float4 h0 = *reinterpret_cast<const float4 *>(hr);
    const float4 h1 = *reinterpret_cast<const float4 *>(hr + 4);
    load8(gain + c, g16, g);
    sum_splits8<S>(part + (int64_t)r * dm + c, (int64_t)M * dm, splits, v);
    v[0] += h0.x; v[1] += h0.y; v[2] += h0.z; v[3] += h0.w;
    v[4] += h1.x; v[5] += h1.y; v[6] += h1.z; v[7] += h1.w;
    *reinterpret_cast<float4 *>(hr) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4 *>(hr + 4) = make_float4(v[4], v[5], v[6], v[7]);
  }
  norm_store<T>(v, g, on, xn, packed, ro, c, dm, eps, sh);
}

template <typename T>
void resid_norm(const float *part, int splits, float *h, const T *gain, T *xn, bool packed, int M,
                int dm, float eps, hipStream_t s, const int32_t *rows, int n_out) {
  const int n = rows ? n_out : M;
  if (n <= 0) return;
  with_splits(splits, [&](auto S) {
    launch(resid_norm_kernel<T, decltype(S)::value>, row_blocks(n), row_threads(dm), 0, s, part, splits, h, gain, xn,
           packed, aligned16(gain), M, n, dm, eps, rows);
  });
}

__global__ void gather_ints_kernel(const int32_t *__restrict__ src, const int32_t *__restrict__ idx, int n,
                                   int32_t *__restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[idx[i]];
}

void gather_ints(const int32_t *src, const int32_t *idx, int n, int32_t *dst, hipStream_t s) {
  if (n > 0) launch(gather_ints_kernel, (n + 255) / 256, 256, 0, s, src, idx, n, dst);
}

// ---------------------------------------------------------------------------------------
// qkv partials -> RoPE (rotate-half) -> q buffer, k/v appended into the pages in place
// ---------------------------------------------------------------------------------------
// Grid (row, group of 8 heads); each thread owns 8 consecutive dims of one head.  The
// rotate-half partner (dims i and i + hd/2) belongs to the thread hd/16 places further
// round the same head; partners are exchanged through LDS, which pairs the right threads
// for every head_dim (a head need not sit inside one wave, nor at a power-of-two lane
// offset).  q and K are written as 16-byte stores (8 consecutive dims are contiguous in
// the K page layout), V element by element.
constexpr int kRopeHeadsPerBlock = 8;

template <typename T>
__device__ __forceinline__ void store8_contig(T *p, const float *v);
template <>
__device__ __forceinline__ void store8_contig<float>(float *p, const float *v) {
  *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
  *reinterpret_cast<float4 *>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
template <>
__device__ __forceinline__ void store8_contig<uint16_t>(uint16_t *p, const float *v) {
  *reinterpret_cast<uint4 *>(p) = make_uint4(pack2bf(v[0], v[1]), pack2bf(v[2], v[3]),
                                             pack2bf(v[4], v[5]), pack2bf(v[6], v[7]));
}

template <typename T, int S>
__global__ __launch_bounds__(256) void qkv_rope_append_kernel(StepDesc d, const float *__restrict__ part,
                                                              int splits, const float *__restrict__ cs,
                                                              T *__restrict__ q, T *__restrict__ k_pool,
                                                              T *__restrict__ v_pool, int M, int nq,
                                                              int nkv, int hd) {
  const int r = row_of_block(blockIdx.x, M);
  if (r >= M) return;
  const int tph = hd / 8;                          // threads per head
  const int head = blockIdx.y * kRopeHeadsPerBlock + threadIdx.x / tph;
  const int nh = nq + 2 * nkv;
  const int i0 = (threadIdx.x % tph) * 8;          // first dim of this thread
  const int h2 = hd / 2;
  const int N = nh * hd;
  __shared__ float xch[kRopeHeadsPerBlock * 256];   // 8 values per thread, hd <= 256
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // everything that does not depend on the exchange is asked for before it
  const int req = d.row_req[r], pos = d.row_pos[r];
  const bool lo = i0 < h2;
  float cn[8], sn[8];
  if (head < nq + nkv) {   // RoPE on q and k heads
    const float4 *csr = reinterpret_cast<const float4 *>(cs + (int64_t)r * hd + 2 * (lo ? i0 : i0 - h2));   // [h2][2]
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float4 x = csr[e];
      cn[2 * e] = x.x;
      sn[2 * e] = x.y;
      cn[2 * e + 1] = x.z;
      sn[2 * e + 1] = x.w;
    }
  }
  int blk = 0;
  if (head >= nq && head < nh) blk = d.page_table[(int64_t)req * d.pt_stride + pos / kPage];
  if (head < nh) sum_splits8<S>(part + (int64_t)r * N + head * hd + i0, (int64_t)M * N, splits, v);
  // rotate-half partner values: thread t of a head pairs with thread (t + tph/2) mod tph
#pragma unroll
  for (int e = 0; e < 8; ++e) xch[threadIdx.x * 8 + e] = v[e];
  __syncthreads();
  const int partner = (threadIdx.x / tph) * tph + (threadIdx.x % tph + tph / 2) % tph;
  float w[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) w[e] = xch[partner * 8 + e];
  if (head >= nh) return;
  if (head < nq + nkv) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = lo ? v[e] * cn[e] - w[e] * sn[e] : v[e] * cn[e] + w[e] * sn[e];
  }
  if (head < nq) {
    store8_contig<T>(q + ((int64_t)r * nq + head) * hd + i0, v);
    return;
  }
  if (blk < 0 || blk >= d.n_blocks) {
    if (threadIdx.x % tph == 0) flag_error(d.err, kErrBlock);
    return;
  }
  const int slot = pos % kPage;
  const int page_elems = kPage * hd;
  if (head < nq + nkv) {
    T *pg = k_pool + ((int64_t)blk * nkv + (head - nq)) * page_elems;
    store8_contig<T>(pg + k_page_off(slot, i0), v);
  } else {
    T *pg = v_pool + ((int64_t)blk * nkv + (head - nq - nkv)) * page_elems;
#pragma unroll
    for (int e = 0; e < 8; ++e) Act<T>::store(pg, v_page_off(slot, i0 + e), v[e]);
  }
}

template <typename T>
void qkv_rope_append(const StepDesc &d, const float *part, int splits, const float *cs, T *q,
                     T *k_pool, T *v_pool, int M, int nq, int nkv, int hd, hipStream_t s) {
  const int nh = nq + 2 * nkv;
  dim3 grid(row_blocks(M), (nh + kRopeHeadsPerBlock - 1) / kRopeHeadsPerBlock);
  with_splits(splits, [&](auto S) {
    launch(qkv_rope_append_kernel<T, decltype(S)::value>, grid, kRopeHeadsPerBlock * hd / 8, 0, s, d, part, splits, cs, q,
           k_pool, v_pool, M, nq, nkv, hd);
  });
}

// ---------------------------------------------------------------------------------------
// SwiGLU: silu(gate) * up.  Gate/up partials are either stacked (columns [0, F) and
// [F, 2F): the fp32 path) or interleaved by 32-column fragments (bf16 weights packed by
// wisp_pack_gate_up: fragment 2b holds gate columns 32b .. 32b + 31, fragment 2b + 1 the
// up columns of the same b)
// ---------------------------------------------------------------------------------------
template <typename T, int S>
__global__ __launch_bounds__(256) void swiglu_kernel(const float *__restrict__ part, int splits,
                                                     T *__restrict__ out, bool packed, int M, int F,
                                                     bool interleaved) {
  const int64_t chunks = (int64_t)M * (F / 8);
  const int64_t stride = (int64_t)M * 2 * F;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < chunks;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = t / (F / 8), c = (t % (F / 8)) * 8;
    const float *pr = part + r * 2 * F;
    const int64_t gc = interleaved ? (c / 32) * 64 + c % 32 : c;
    const int64_t uc = interleaved ? gc + 32 : F + c;
    float g[8], u[8], v[8];
    sum_splits8<S>(pr + gc, stride, splits, g);
    sum_splits8<S>(pr + uc, stride, splits, u);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = silu_mul(g[e], u[e]);
    store8<T>(out, packed, r, c, F, v);
  }
}

template <typename T>
void swiglu(const float *part, int splits, T *out, bool packed, int M, int F, bool interleaved, hipStream_t s) {
  const int64_t chunks = (int64_t)M * (F / 8);
  int blocks = (int)((chunks + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  with_splits(splits, [&](auto S) {
    launch(swiglu_kernel<T, decltype(S)::value>, blocks, 256, 0, s, part, splits, out, packed, M, F, interleaved);
  });
}

template void embed_norm<float>(const StepDesc &, const float *, const float *, const int32_t *,
                                float *, float *, bool, int, int, int, float, hipStream_t);
template void embed_norm<uint16_t>(const StepDesc &, const uint16_t *, const uint16_t *,
                                   const int32_t *, float *, uint16_t *, bool, int, int, int, float,
                                   hipStream_t);
template void resid_norm<float>(const float *, int, float *, const float *, float *, bool, int, int,
                                float, hipStream_t, const int32_t *, int);
template void resid_norm<uint16_t>(const float *, int, float *, const uint16_t *, uint16_t *, bool,
                                   int, int, float, hipStream_t, const int32_t *, int);
template void qkv_rope_append<float>(const StepDesc &, const float *, int, const float *, float *,
                                     float *, float *, int, int, int, int, hipStream_t);
template void qkv_rope_append<uint16_t>(const StepDesc &, const float *, int, const float *,
                                        uint16_t *, uint16_t *, uint16_t *, int, int, int, int,
                                        hipStream_t);
template void swiglu<float>(const float *, int, float *, bool, int, int, bool, hipStream_t);
template void swiglu<uint16_t>(const float *, int, uint16_t *, bool, int, int, bool, hipStream_t);

}  // namespace wisp
