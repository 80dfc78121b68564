// Acceptance stage of the verification step (Sec. 2.4): Eq. (1) accept draft y_j with
// probability min(1, p/q), Eq. (2) stop at the first rejection R, Eq. (3) emit one extra
// token -- drawn from norm(max(0, p_R - q_R)) after a rejection (the residual that makes
// speculative sampling lossless) and from p after a fully accepted block.
//
// Three launches per batch: one pass over the logits in vocabulary chunks of 8192 entries
// (each chunk's maximum of z = logits / T and its fp64 sum of exp(z - maximum); the first
// argmax at T = 0), then one workgroup per (request, chunk of 2048) that decides every draft
// in parallel (thread j - 1 takes draft j; R is the smallest rejected j, an integer minimum)
// and runs its chunk of the exponential race that samples the extra token (argmax of score
// - ln(-ln u): no prefix sums, so the result does not depend on reduction order), and a last
// kernel, one wave per request, that combines the chunks' winners by a total
// order.  All random draws come from Philox4x32-10 keyed by the seed and counted by
// (index, row, request, purpose).
#pragma clang fp contract(off)
#include "common.h"
#include "kernels.h"

namespace wisp {

__device__ __forceinline__ Philox4 draw(uint64_t seed, uint32_t c0, uint32_t row, uint32_t req,
                                        uint32_t tag) {
  return philox4x32_10(c0, row, req, tag, (uint32_t)seed, (uint32_t)(seed >> 32));
}

// ---------------------------------------------------------------------------------------
// The vocabulary is cut into chunks: kVChunk entries per workgroup of the pass over the
// logits, kRaceChunk per workgroup of the race.  Partial results are combined in fixed order.
// ---------------------------------------------------------------------------------------
constexpr int kVChunk = 8192;
// The race takes chunks of 2048 entries (8 per thread), doubled up to 8192 while they make more
// than kRaceGroups workgroups (or, in a step, than fit into the GEMMs' partial sums, which are
// free by then): a workgroup also decides the request's drafts, which costs
// about as much as 2048 entries, but fewer than that many workgroups leave SIMDs idle (with
// 4-byte loads: B = 32 27.4 us with chunks of 8192, 18.3 with 2048; B = 256 119 against 143).
constexpr int kRaceChunk = 2048, kRaceChunkMax = 8192, kRaceGroups = 2560;

__device__ __forceinline__ bool better(float ka, int ia, float kb, int ib) {
  return ka > kb || (ka == kb && ia < ib);
}

// (key, index) argmax across a wave; ties go to the smaller index
__device__ __forceinline__ void wave_argmax(float &k, int &i) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ok = __shfl_xor(k, o);
    const int oi = __shfl_xor(i, o);
    if (better(ok, oi, k, i)) {
      k = ok;
      i = oi;
    }
  }
}

// (key, index) argmax across the 256 threads
__device__ __forceinline__ void block_argmax(float &k, int &i, float *shk, int *shi) {
  wave_argmax(k, i);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    shk[threadIdx.x >> 6] = k;
    shi[threadIdx.x >> 6] = i;
  }
  __syncthreads();
  k = shk[0];
  i = shi[0];
  for (int w = 1; w < 4; ++w)
    if (better(shk[w], shi[w], k, i)) {
      k = shk[w];
      i = shi[w];
    }
}

// Pass 1, per (row, chunk): the maximum m of z = l / T and the fp64 sum of exp(z - m) (T > 0),
// or the maximum and first argmax of l (T == 0).  A thread holds its 32 entries in registers,
// so the logits are read once.  Bound by the logits' bytes once the instructions per entry
// allow it: 16-byte loads where the rows are aligned (VEC) and no division at T = 1 (l / 1 is
// l).  B = 32 (171 rows of 128256): maximum and sum in separate passes of 4-byte loads took
// 28 + 30 us, together 18 (5 TB/s).
template <bool VEC>
__global__ __launch_bounds__(256) void row_stats_kernel(const float *__restrict__ logits, int V, float T, int CH,
                                                        float *__restrict__ part_m, int32_t *__restrict__ part_i,
                                                        double *__restrict__ part_s) {
  constexpr int PER = kVChunk / 256;
  __shared__ float shk[4];
  __shared__ int shi[4];
  __shared__ double shd[4];
  const int c = blockIdx.y;
  const int64_t r = blockIdx.x;
  const float *l = logits + r * V;
  const int k0 = c * kVChunk, n = min(V - k0, kVChunk);   // entries of this chunk
  // entry e of this thread: VEC: 4 (256 (e / 4) + thread) + e % 4, else 256 e + thread
  auto index = [&](int e) {
    return VEC ? 4 * (256 * (e >> 2) + (int)threadIdx.x) + (e & 3) : 256 * e + (int)threadIdx.x;
  };
  float z[PER];
  if constexpr (VEC) {   // V is a multiple of 4: a quadruple lies inside the chunk or outside
    const float4 *l4 = reinterpret_cast<const float4 *>(l + k0);
#pragma unroll
    for (int q = 0; q < PER / 4; ++q) {
      const int i4 = 256 * q + threadIdx.x;
      const float4 x = 4 * i4 < n ? __builtin_bit_cast(float4, ld16_stream(l4 + i4)) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      z[4 * q] = x.x;
      z[4 * q + 1] = x.y;
      z[4 * q + 2] = x.z;
      z[4 * q + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < PER; ++e) z[e] = index(e) < n ? l[k0 + index(e)] : -INFINITY;
  }
  if (T == 0.f) {
    float bk = -INFINITY;
    int bi = 0x7FFFFFFF;
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (z[e] > bk) {
        bk = z[e];
        bi = k0 + index(e);
      }
    block_argmax(bk, bi, shk, shi);
    if (threadIdx.x == 0) {
      part_m[r * CH + c] = bk;
      part_i[r * CH + c] = bi;
    }
    return;
  }
  if (T != 1.f) {
#pragma unroll
    for (int e = 0; e < PER; ++e) z[e] = z[e] / T;
  }
  float m = -INFINITY;
#pragma unroll
  for (int e = 0; e < PER; ++e) m = fmaxf(m, z[e]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) shk[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmaxf(fmaxf(shk[0], shk[1]), fmaxf(shk[2], shk[3]));
  const float mr = m == -INFINITY ? 0.f : m;   // a chunk of -inf sums to 0, not to exp(-inf + inf)
  double sum = 0.0;
#pragma unroll
  for (int e = 0; e < PER; ++e) sum += (double)expf(z[e] - mr);   // entries past the end: exp(-inf) = 0
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
  if ((threadIdx.x & 63) == 0) shd[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    part_m[r * CH + c] = m;
    part_s[r * CH + c] = (shd[0] + shd[1]) + (shd[2] + shd[3]);
  }
}

struct RowStat {
  float m, S;
  int amax;
};

// A row's statistics from its chunks' by 8 neighbouring lanes (lane `g` of them): the row's
// maximum, S = sum_c s_c exp(m_c - m) in fp64 rounded once, or (T == 0) the first argmax
__device__ RowStat row_stat8(const float *part_m, const int32_t *part_i, const double *part_s, int64_t r, int CH,
                             float T, int g) {
  RowStat st;
  float bk = -INFINITY;
  int bi = 0x7FFFFFFF;
  for (int c = g; c < CH; c += 8) {
    const float m = part_m[r * CH + c];
    const int i = T == 0.f ? part_i[r * CH + c] : 0;
    if (better(m, i, bk, bi)) {
      bk = m;
      bi = i;
    }
  }
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) {
    const float ok = __shfl_xor(bk, o);
    const int oi = __shfl_xor(bi, o);
    if (better(ok, oi, bk, bi)) {
      bk = ok;
      bi = oi;
    }
  }
  st.m = bk;
  st.S = 1.f;
  st.amax = bi;
  if (T == 0.f) return st;
  double s = 0.0;
  for (int c = g; c < CH; c += 8) {
    const float m = part_m[r * CH + c];
    s += m == bk && m != -INFINITY ? part_s[r * CH + c] : part_s[r * CH + c] * exp((double)m - (double)bk);
  }
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) s += __shfl_xor(s, o);
  st.S = (float)s;
  return st;
}

// entries 4 k4 .. 4 k4 + 3 of a row of V (VEC: the row is 16-byte aligned, V a multiple of 4;
// otherwise entries past the end repeat the last one)
template <bool VEC>
__device__ __forceinline__ void load_quad(const float *row, int k4, int V, float (&v)[4]) {
  if constexpr (VEC) {
    const float4 x = reinterpret_cast<const float4 *>(row)[k4];
    v[0] = x.x;
    v[1] = x.y;
    v[2] = x.z;
    v[3] = x.w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = row[min(4 * k4 + e, V - 1)];
  }
}

// pass 2: Eq. (1)-(2) acceptance (recomputed by every chunk's workgroup), then that chunk's
// part of the exponential race for the extra token (Eq. (3) / residual).  The <= 17 rows'
// statistics are combined by 8 lanes each; the <= 16 draft decisions are independent of one
// another, so thread j - 1 takes draft j's and R is the smallest rejected j (gamma + 1 when
// none is): one round of loads instead of a chain.  The race's logits and q come as 16-byte
// loads, two quadruples per thread at a time (4-byte loads inside the loop over entries: 13.4
// us at B = 1, 119 at B = 256; now 8.8 and 94).
template <bool VEC>
__global__ __launch_bounds__(256) void race_kernel(StepDesc d, int V, const float *__restrict__ logits,
                                                   const int32_t *__restrict__ tokens,
                                                   const float *__restrict__ q, float T, uint64_t seed,
                                                   int CH, int chunk, int RC, const float *__restrict__ part_m,
                                                   const int32_t *__restrict__ part_i,
                                                   const double *__restrict__ part_s,
                                                   float *__restrict__ race_k, int32_t *__restrict__ race_i,
                                                   int32_t *__restrict__ req_R) {
  __shared__ int R_sh;
  __shared__ float shk[4];
  __shared__ int shi[4];
  __shared__ int shany[4];
  __shared__ RowStat rows[32];
  const int c = blockIdx.y, i = blockIdx.x;
  const int gam = d.gamma[i], off = d.off[i], doff = d.doff[i];
  const uint32_t req = d.req_id[i];
  const int j = threadIdx.x + 1;   // gamma <= 16 < 256 threads
  // draft j's token, logit and probability: loaded before the statistics are combined
  int y = 0;
  float ly = 0.f, Q = 0.f;
  if (j <= gam) {
    y = tokens[off + j];
    if (y < 0 || y >= V) {
      if (c == 0) flag_error(d.err, kErrToken);
      y = 0;
    }
    ly = logits[(int64_t)(off + j - 1) * V + y];
    if (T != 0.f) Q = q[(int64_t)(doff + j - 1) * V + y];
  }
  const int g = threadIdx.x >> 3;   // row off + g of the request, 8 lanes each
  if (g <= gam) {
    const RowStat st = row_stat8(part_m, part_i, part_s, off + g, CH, T, threadIdx.x & 7);
    if ((threadIdx.x & 7) == 0) rows[g] = st;
  }
  if (threadIdx.x == 0) R_sh = gam + 1;
  __syncthreads();
  if (j <= gam) {
    const RowStat st = rows[j - 1];
    bool rejected_j;
    if (T == 0.f) {
      rejected_j = y != st.amax;
    } else {
      const float P = expf(ly / T - st.m) / st.S;
      const float a = Q > 0.f ? fminf(1.f, P / Q) : (P > 0.f ? 1.f : 0.f);
      const float u = uniform_from_word(draw(seed, 0u, (uint32_t)j, req, kTagAccept).v[0]);
      rejected_j = !(u <= a);
    }
    if (rejected_j) atomicMin(&R_sh, j);   // integer minimum: the order of arrival does not matter
  }
  __syncthreads();
  const int R = R_sh, r = R - 1;
  const RowStat st = rows[r];
  const int64_t o = ((int64_t)i * RC + c) * 2;
  if (c == 0 && threadIdx.x == 0) req_R[i] = R;
  if (T == 0.f) {   // one workgroup per request: the extra token is the row's argmax
    if (threadIdx.x == 0) race_i[o] = st.amax;
    return;
  }
  const int64_t lr = off + r;
  const float *l = logits + lr * V;
  const bool rejected = R <= gam;
  const float *qr = q + (int64_t)(doff + (rejected ? R - 1 : 0)) * V;
  float kR = -INFINITY, kP = -INFINITY;
  int iR = 0x7FFFFFFF, iP = 0x7FFFFFFF;
  int any = 0;
  // the chunk's quadruples in turns of 2 per thread, a turn's logits and q loaded together
  const int k4_1 = min((V + 3) / 4, (c + 1) * (chunk / 4));
  for (int base = c * (chunk / 4) + threadIdx.x; base < k4_1; base += 512) {
    float lv[2][4], qv[2][4];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int k4 = min(base + 256 * x, k4_1 - 1);   // past the end: loaded again, not used
      load_quad<VEC>(l, k4, V, lv[x]);
      if (rejected) load_quad<VEC>(qr, k4, V, qv[x]);
    }
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int k4 = base + 256 * x;
      if (k4 >= k4_1) break;
      const Philox4 w = draw(seed, (uint32_t)k4, (uint32_t)r, req, kTagRace);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = k4 * 4 + e;
        if (k >= V) break;
        const float z = T == 1.f ? lv[x][e] : lv[x][e] / T;
        const float gk = logf(-logf(uniform_from_word(w.v[e])));
        const float keyp = z - gk;
        if (keyp > kP) {
          kP = keyp;
          iP = k;
        }
        if (rejected) {
          const float wk = expf(z - st.m) / st.S - qv[x][e];
          if (wk > 0.f) {
            any = 1;
            const float keyr = logf(wk) - gk;
            if (keyr > kR) {
              kR = keyr;
              iR = k;
            }
          }
        }
      }
    }
  }
  block_argmax(kP, iP, shk, shi);
  if (rejected) {   // uniform over the workgroup; otherwise the residual race stays empty
    block_argmax(kR, iR, shk, shi);
#pragma unroll
    for (int x = 32; x > 0; x >>= 1) any |= __shfl_xor(any, x);
    if ((threadIdx.x & 63) == 0) shany[threadIdx.x >> 6] = any;
    __syncthreads();
    any = shany[0] | shany[1] | shany[2] | shany[3];
  }
  if (threadIdx.x == 0) {
    race_k[o] = kP;
    race_i[o] = iP;
    race_k[o + 1] = any ? kR : -INFINITY;
    race_i[o + 1] = any ? iR : 0x7FFFFFFF;
  }
}

// pass 3, one wave per request: the best of the chunks' race winners (a total order: key, then
// smaller index), and the outputs
__global__ __launch_bounds__(64) void finalize_kernel(StepDesc d, const int32_t *__restrict__ tokens, float T, int RC,
                                                      const float *__restrict__ race_k,
                                                      const int32_t *__restrict__ race_i,
                                                      const int32_t *__restrict__ req_R,
                                                      int32_t *__restrict__ accept_len,
                                                      int32_t *__restrict__ out_tokens) {
  const int i = blockIdx.x, lane = threadIdx.x;
  const int gam = d.gamma[i], off = d.off[i];
  const int R = req_R[i], L = R - 1;
  int extra;
  if (T == 0.f) {
    extra = race_i[(int64_t)i * RC * 2];
  } else {
    float kP = -INFINITY, kR = -INFINITY;
    int iP = 0x7FFFFFFF, iR = 0x7FFFFFFF;
    for (int c = lane; c < RC; c += 64) {
      const int64_t o = ((int64_t)i * RC + c) * 2;
      const float2 k = *reinterpret_cast<const float2 *>(race_k + o);
      const int2 x = *reinterpret_cast<const int2 *>(race_i + o);
      if (better(k.x, x.x, kP, iP)) {
        kP = k.x;
        iP = x.x;
      }
      if (x.y != 0x7FFFFFFF && better(k.y, x.y, kR, iR)) {
        kR = k.y;
        iR = x.y;
      }
    }
    wave_argmax(kP, iP);
    wave_argmax(kR, iR);
    extra = (R <= gam && iR != 0x7FFFFFFF) ? iR : iP;
  }
  if (lane <= gam) out_tokens[off + lane] = lane < L ? tokens[off + lane + 1] : (lane == L ? extra : -1);
  if (lane == 0) accept_len[i] = L;
}

int sampler_chunks(int V) { return (V + kVChunk - 1) / kVChunk; }
int sampler_race_chunk(int B, int V, size_t bytes) {
  auto chunks = [&](int chunk) { return (V + chunk - 1) / chunk; };
  int chunk = kRaceChunk;
  while (chunk < kRaceChunkMax && ((int64_t)B * chunks(chunk) > kRaceGroups || (size_t)B * chunks(chunk) * 16 > bytes)) chunk *= 2;
  return chunk;
}

void sampler(const StepDesc &d, int B, int M, int V, const float *logits, const int32_t *tokens,
             const float *q, float T, uint64_t seed, int chunk, SamplerScratch sc, int32_t *accept_len,
             int32_t *out_tokens, hipStream_t s) {
  if (B == 0) return;
  const int CH = sampler_chunks(V);
  const int RC = (V + chunk - 1) / chunk;
  const bool vec = V % 4 == 0 && ((uintptr_t)logits & 15) == 0;
  launch(vec ? row_stats_kernel<true> : row_stats_kernel<false>, dim3(M, CH), 256, 0, s, logits, V, T, CH, sc.part_m,
         sc.part_i, sc.part_s);
  const bool qvec = vec && ((uintptr_t)q & 15) == 0;
  launch(qvec ? race_kernel<true> : race_kernel<false>, dim3(B, T == 0.f ? 1 : RC), 256, 0, s, d, V, logits, tokens, q, T, seed, CH, chunk, RC, sc.part_m,
         sc.part_i, sc.part_s, sc.race_k, sc.race_i, sc.req_R);
  launch(finalize_kernel, B, 64, 0, s, d, tokens, T, RC, sc.race_k, sc.race_i, sc.req_R, accept_len, out_tokens);
}

__global__ void uniform_kernel(uint64_t seed, uint32_t req, uint32_t tag, uint32_t row, uint32_t n,
                               float *out) {
  for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x)
    out[k] = uniform_from_word(draw(seed, k >> 2, row, req, tag).v[k & 3]);
}

void uniform_draws(uint64_t seed, uint32_t req, uint32_t tag, uint32_t row, uint32_t n, float *out,
                   hipStream_t s) {
  if (n == 0) return;
  uint32_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  launch(uniform_kernel, blocks, 256, 0, s, seed, req, tag, row, n, out);
}

}  // namespace wisp
