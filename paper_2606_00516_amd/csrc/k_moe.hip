// Mixture-of-experts feed-forward block: routing, the expert-sorted order and
// the weighted combine (the expert products are the grouped GEMM kernel).
//
//   logits[t] = b[t] W_r^T (fp32 sums of bf16 products, kept in fp32)
//   S(t)      = the k largest logits (equal logits: lower expert first)
//   w[t, e]   = exp(logits[t, e] - max) over S(t), divided by its sum over
//               S(t) (renormalised) or over all E experts
//   out[t]    = bf16(residual[t] + sum_j w[t, j] y[t, j])
//
// with y[t, j] the fp32 output of expert S(t)_j for token t.
#include "device_common.h"
#include "eb_internal.h"

namespace eb {

constexpr int kMoeTokens = 16;  // tokens per logits wavefront

// Logits of a decode-sized batch: one wavefront per 16 tokens x 16 experts,
// the 16x16x32 MFMA with the experts as rows and the tokens as columns, both
// operands read straight from global memory (W_r is shared by every wave and
// stays in L2).  A wave's time is its chain of load latencies, so the next
// eight K steps' loads are in flight while the last eight multiply (64 tokens
// of 2048: 8.1 -> 5.4 us).  fp32 out [T, E].  Longer batches re-read every
// token row once per 16 experts here and take the weight-streaming GEMM
// instead (launch_moe_route).
__global__ __launch_bounds__(64) void k_moe_logits(const uint16_t *__restrict__ b, const uint16_t *__restrict__ wr,
                                                   int T, int d, int E, float *__restrict__ logits) {
  const int lane = threadIdx.x;
  const int t0 = blockIdx.x * kMoeTokens, e0 = blockIdx.y * 16;
  const int lr = lane & 15, lgp = lane >> 4;
  const buf_rsrc_t rb = make_rsrc(b, (int)min((size_t)T * d * 2, (size_t)0x7FFFFFFF));
  const buf_rsrc_t rr = make_rsrc(wr, (int)min((size_t)E * d * 2, (size_t)0x7FFFFFFF));
  const int tok = t0 + lr;
  const uint32_t boff = tok < T ? ((uint32_t)tok * (uint32_t)d + 8u * lgp) * 2u : 0x80000000u;
  const uint32_t woff = ((uint32_t)(e0 + lr) * (uint32_t)d + 8u * lgp) * 2u;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 8;
  u32x4_t wa[U], ba[U], wb[U], bb[U];
  auto load = [&](int kk, u32x4_t (&wf)[U], u32x4_t (&bf)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = kk + 32 * u;
      const bool ok = k < d;
      wf[u] = buf_ld_u32x4<0>(rr, (int)(ok ? woff + 2u * k : 0x80000000u));
      bf[u] = buf_ld_u32x4<0>(rb, (int)(ok && boff != 0x80000000u ? boff + 2u * k : 0x80000000u));
    }
  };
  load(0, wa, ba);
  for (int kk = 0; kk < d; kk += 64 * U) {
    load(kk + 32 * U, wb, bb);
#pragma unroll
    for (int u = 0; u < U; ++u) acc = mfma16x16x32(wa[u], ba[u], acc);
    load(kk + 64 * U, wa, ba);
#pragma unroll
    for (int u = 0; u < U; ++u) acc = mfma16x16x32(wb[u], bb[u], acc);
  }
  // lane holds experts e0 + 4 lgp .. + 3 of token lr
  if (tok < T) *reinterpret_cast<f32x4_t *>(logits + (size_t)tok * E + e0 + 4 * lgp) = acc;
}

// Top k of each token's logits: one wavefront per token, k rounds of a
// wave-wide arg-max (equal values: lower expert), then the weights.
__global__ __launch_bounds__(256) void k_moe_topk(const float *__restrict__ logits, int T, int E, int k,
                                                  int renormalize, int32_t *__restrict__ ids,
                                                  float *__restrict__ wts) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const float *row = logits + (size_t)t * E;
  float v[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = lane + 64 * c < E ? row[lane + 64 * c] : -INFINITY;
  float sel_v = 0.f, top = 0.f, sum_sel = 0.f;
  int sel_e = 0;
  for (int j = 0; j < k; ++j) {
    // this lane's best (value, lowest expert), then the wave's
    float bv = v[0];
    int be = lane;
#pragma unroll
    for (int c = 1; c < 4; ++c)
      if (v[c] > bv) {
        bv = v[c];
        be = lane + 64 * c;
      }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const float ov = __shfl_xor(bv, off, 64);
      const int oe = __shfl_xor(be, off, 64);
      if (ov > bv || (ov == bv && oe < be)) {
        bv = ov;
        be = oe;
      }
    }
    if (j == 0) top = bv;
    const float p = __expf(bv - top);
    sum_sel += p;
    if (lane == j) {
      sel_v = p;
      sel_e = be;
    }
    // the owner takes the chosen value out
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (lane + 64 * c == be) v[c] = -INFINITY;
  }
  float denom = sum_sel;
  if (!renormalize) {  // the softmax over all E experts (top is the largest logit)
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (lane + 64 * c < E) s += __expf(row[lane + 64 * c] - top);
    denom = wave_sum(s);
  }
  if (lane < k) {
    ids[(size_t)t * k + lane] = sel_e;
    wts[(size_t)t * k + lane] = sel_v / denom;
  }
}

// The sorted order: expert counts, their offsets in it, the row tiles (up to
// tile_rows rows of one expert) and each assignment's sorted position.
// Positions within an expert follow the order of the blocks' atomics; every
// later step is independent of that order (rows are independent in the
// products and the combine reads the slots in token order).
constexpr int kPlanThreads = 1024;
// assignments per block, from which on the plan runs on several blocks
constexpr int kPlanChunk = 1024;
constexpr int kPlanMaxBlocks = 256;

// (ids come from the routing kernel; clamped all the same, so that no input
// can steer a write outside the tables)
__device__ __forceinline__ int plan_expert(const int32_t *ids, int i, int E) { return min(max(ids[i], 0), E - 1); }

// Inclusive sums of v over the block's first 256 threads (4 wavefronts; every
// thread calls it, the others with v = 0).
__device__ __forceinline__ int scan256(int v, int *wsum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  if (lane == 63 && wave < 4) wsum[wave] = v;
  __syncthreads();
  for (int w = 0; w < min(wave, 4); ++w) v += wsum[w];
  __syncthreads();
  return v;
}

// Several blocks, first pass: block b counts its chunk's experts into
// counts[b][E].
__global__ __launch_bounds__(kPlanThreads) void k_moe_count(const int32_t *__restrict__ ids, int P, int E, int chunk,
                                                            int32_t *__restrict__ counts) {
  __shared__ int cnt[256];
  const int tid = threadIdx.x;
  if (tid < E) cnt[tid] = 0;
  __syncthreads();
  const int lo = blockIdx.x * chunk, hi = min(P, lo + chunk);
  for (int i = lo + tid; i < hi; i += kPlanThreads) atomicAdd(&cnt[plan_expert(ids, i, E)], 1);
  __syncthreads();
  if (tid < E) counts[(size_t)blockIdx.x * E + tid] = cnt[tid];
}

// One block over everything (counts null, chunk P), or the second pass of
// several: every block forms the totals and its own place in each expert's
// run from the counts, block 0 writes the tables.  The prefix sums over the
// experts run across threads; a single thread's walk over them took most of
// the time of a decode batch (64 tokens: 9.8 -> 5.0 us), one block's passes over
// all assignments that of a long one (65536 assignments: 67 -> 12 us).
__global__ __launch_bounds__(kPlanThreads) void k_moe_plan(const int32_t *__restrict__ ids, int P, int E, int k,
                                                           int tile_rows, int max_tiles, int chunk,
                                                           const int32_t *__restrict__ counts,
                                                           int32_t *__restrict__ offsets,
                                                           int32_t *__restrict__ sorted_tok,
                                                           int32_t *__restrict__ pos_of, int32_t *__restrict__ tiles,
                                                           int32_t *__restrict__ n_tiles) {
  __shared__ int cnt[256], cur[256], wsum[4];
  const int tid = threadIdx.x;
  const int lo = blockIdx.x * chunk, hi = min(P, lo + chunk);
  if (tid < 256) cnt[tid] = cur[tid] = 0;
  __syncthreads();
  if (counts) {
    const int nb = gridDim.x, G = kPlanThreads / E;  // G threads per expert share the blocks' counts
    const int e = tid % E, g = tid / E;
    if (g < G) {
      int tot = 0, before = 0;
      for (int b = g; b < nb; b += G) {
        const int c = counts[(size_t)b * E + e];
        tot += c;
        before += b < (int)blockIdx.x ? c : 0;
      }
      atomicAdd(&cnt[e], tot);
      atomicAdd(&cur[e], before);
    }
  } else {
    for (int i = lo + tid; i < hi; i += kPlanThreads) atomicAdd(&cnt[plan_expert(ids, i, E)], 1);
  }
  __syncthreads();
  const int n = tid < E ? cnt[tid] : 0, nt = (n + tile_rows - 1) / tile_rows;
  const int o1 = scan256(n, wsum), t1 = scan256(nt, wsum);
  if (tid < E) {
    cur[tid] += o1 - n;
    if (blockIdx.x == 0) {
      offsets[tid] = o1 - n;
      if (tid == E - 1) {
        offsets[E] = o1;
        *n_tiles = min(t1, max_tiles);
      }
      for (int j = 0, r = t1 - nt; j < n && r < max_tiles; j += tile_rows, ++r) {
        tiles[r] = tid;
        tiles[max_tiles + r] = o1 - n + j;
        tiles[2 * max_tiles + r] = min(tile_rows, n - j);
      }
    }
  }
  __syncthreads();
  for (int i = lo + tid; i < hi; i += kPlanThreads) {
    const int p = atomicAdd(&cur[plan_expert(ids, i, E)], 1);
    sorted_tok[p] = i / k;
    pos_of[i] = p;
  }
}

// out[t] = bf16(res[t] + sum_j w[t, j] y[pos_of[t k + j]]): one block per
// token and 1024 columns, four columns per thread.  Bound by reading y once:
// the token's positions and weights are fetched first, then the rows of
// eight experts are in flight together (the sum keeps the experts' order; a
// loop that waited for each position, then its row, read 8192 tokens' 537 MB
// in 146 us, this one in 138; 64 tokens 7.6 -> 4.8).  y is read once and, at
// thousands of tokens, larger than the caches: non-temporal loads leave them
// to the positions and the output (8192 tokens 137 -> 108 us, 5.6 TB/s; 64
// tokens, whose y does fit, 4.9 both).
__global__ __launch_bounds__(256) void k_moe_combine(const float *__restrict__ y, const int32_t *__restrict__ pos_of,
                                                     const float *__restrict__ wts, const uint16_t *__restrict__ res,
                                                     uint16_t *__restrict__ out, int d, int k) {
  const int t = blockIdx.x;
  const int c0 = blockIdx.y * 1024 + 4 * threadIdx.x;
  const int c = min(c0, d - 4);  // (lanes past the row work on its end: every lane stays active for the reads across lanes)
  const int lane = threadIdx.x & 63;
  // lane j holds expert j's position and weight (k <= 64)
  const int pv = lane < k ? pos_of[(size_t)t * k + lane] : 0;
  const float wv = lane < k ? wts[(size_t)t * k + lane] : 0.f;
  u32x2_t r = {0u, 0u};
  if (res) r = *reinterpret_cast<const u32x2_t *>(res + (size_t)t * d + c);
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  for (int j0 = 0; j0 < k; j0 += 8) {
    f32x4_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + u < k)
        v[u] = __builtin_nontemporal_load(
            reinterpret_cast<const f32x4_t *>(y + (size_t)__builtin_amdgcn_readlane(pv, j0 + u) * d + c));
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + u < k) acc += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wv), j0 + u)) * v[u];
  }
  acc += f32x4_t{bf16_lo(r[0]), bf16_hi(r[0]), bf16_lo(r[1]), bf16_hi(r[1])};
  if (c0 < d)
    *reinterpret_cast<u32x2_t *>(out + (size_t)t * d + c) =
        u32x2_t{pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3])};
}

hipError_t launch_moe_route(const uint16_t *b, const uint16_t *wr, int T, int d, int E, int k, int renormalize,
                            float *logits, int32_t *ids, float *wts, hipStream_t st) {
  if (T <= 0) return hipSuccess;
  hipError_t e;
  // The wavefronts read every token row once per 16 experts, the streaming
  // GEMM once per 128, in fewer and larger blocks: the line lies where T E
  // reaches 2^18 (whole blocks of experts 8 wide and top 1, us, wavefronts
  // against streamed, d 2048: 16 experts 8192 tokens 79 / 83, 16384 125 / 123;
  // 64 experts 3000 59 / 63, 4096 68 / 69, 8192 100 / 85; 128 experts 1536 57 /
  // 59, 2100 67 / 63; 256 experts 1024 69 / 68, 1536 79 / 70; d 512 and 4096
  // cross within a factor of 1.5 of it)
  if ((size_t)T * E > (size_t)1 << 18) {
    e = launch_gemm_f32(b, wr, logits, T, E, d, st);
  } else {
    hipLaunchKernelGGL(k_moe_logits, dim3((T + kMoeTokens - 1) / kMoeTokens, E / 16), dim3(64), 0, st, b, wr, T, d, E,
                       logits);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_moe_topk, dim3((T + 3) / 4), dim3(256), 0, st, logits, T, E, k, renormalize, ids, wts);
  return hipGetLastError();
}

hipError_t launch_moe_plan(const int32_t *ids, int P, int E, int k, int tile_rows, int max_tiles, int32_t *offsets,
                           int32_t *sorted_tok, int32_t *pos_of, int32_t *tiles, int32_t *n_tiles, int32_t *scratch,
                           hipStream_t st) {
  // several blocks once each has a full pass of assignments
  int nb = 1, chunk = P;
  const int32_t *counts = nullptr;
  if (P >= 4 * kPlanChunk) {
    nb = (P + kPlanChunk - 1) / kPlanChunk;
    if (nb > kPlanMaxBlocks) nb = kPlanMaxBlocks;
    chunk = (P + nb - 1) / nb;
    hipLaunchKernelGGL(k_moe_count, dim3(nb), dim3(kPlanThreads), 0, st, ids, P, E, chunk, scratch);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    counts = scratch;
  }
  hipLaunchKernelGGL(k_moe_plan, dim3(nb), dim3(kPlanThreads), 0, st, ids, P, E, k, tile_rows, max_tiles, chunk, counts,
                     offsets, sorted_tok, pos_of, tiles, n_tiles);
  return hipGetLastError();
}

hipError_t launch_moe_combine(const float *y, const int32_t *pos_of, const float *wts, const uint16_t *res,
                              uint16_t *out, int T, int d, int k, hipStream_t st) {
  if (T <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_moe_combine, dim3(T, (d + 1023) / 1024), dim3(256), 0, st, y, pos_of, wts, res, out, d, k);
  return hipGetLastError();
}

}  // namespace eb
