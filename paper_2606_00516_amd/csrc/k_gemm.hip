// Projection GEMMs of the layer: out = epilogue(A W^T), A [M, K] activations,
// W [N, K] weights, both K-contiguous bf16, fp32 accumulation on the
// 16x16x32 bf16 MFMA.
//
//  * stream: decode-sized batches (below 256 rows, and any number of them
//    against a W that one XCD's L2 holds) in blocks of 64 to 256 rows x 128
//    columns, one block per CU.  The product is bound by streaming W from HBM
//    once: W and A go straight into an LDS ring that fills the CU, all but one
//    stage of it in flight, and blocks may further split K, with a small
//    reduction kernel applying the epilogue.  Up to 64 rows, W may come from a
//    fragment-packed copy straight into registers.
//  * big: 256 x 256 tiles, larger M (and from 129 rows where its estimated
//    time is the least: plan_gemm).
//  * tiled: what neither takes.  128x128 output tiles, K tiles of 64
//    double-buffered in LDS, 4 waves each owning a 64x64 sub-tile.
//
// Epilogues: store; + residual; SiLU(gate) * up.  For SiLU the columns are
// processed in groups of 64 = 32 gate rows of W followed by the 32 matching
// up rows (gate rows 0..F-1, up rows F..2F-1 of W), so that every lane holds
// a gate accumulator and its up partner.
#include <algorithm>

#include "device_common.h"
#include "eb_internal.h"

namespace eb {

// W row feeding logical column c of the product (or -1 if none).
__device__ __forceinline__ int w_row_of(int c, int N, int epi) {
  if (epi != EPI_SILU_MUL) return c < N ? c : -1;
  const int F = N >> 1;
  const int g = c >> 6, w = c & 63;
  const int f = g * 32 + (w & 31);
  if (f >= F) return -1;
  return w < 32 ? f : F + f;
}

// Number of logical product columns for an epilogue.
__host__ __device__ static inline int logical_cols(int N, int epi) {
  if (epi != EPI_SILU_MUL) return N;
  const int F = N / 2;
  return ((F + 31) / 32) * 64;
}

// (a division: the reciprocal instruction is one unit in the last place less
// exact, and its result is flushed to zero for g below -87.3, where the value
// is still a normal bf16)
__device__ __forceinline__ float silu_f(float g) { return g / (1.0f + __expf(-g)); }

// 8-bit weights: the fp32 sums of logical columns c .. c + 3 (one W row
// each, consecutive within a column group) times their rows' scales.
__device__ __forceinline__ f32x4_t row_scaled(f32x4_t v, const float *__restrict__ wscale, int c, int N, int epi) {
  const int wr = w_row_of(c, N, epi);
  if (wr < 0) return v;
  const f32x4_t s = *reinterpret_cast<const f32x4_t *>(wscale + wr);
  return v * s;
}

// One 16-byte-per-lane buffer load straight into LDS at byte address lds +
// 16 lane (lds wave-uniform).  In assembly, so that the compiler does not
// take every later LDS read to depend on it and drain all loads in flight:
// the kernel counts its own loads (s_waitcnt vmcnt) instead.  The load
// writes no register.
__device__ __forceinline__ void dma_lds16(u32x4_t rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory", "m0");
}
// The same for data that nothing reads again (non-temporal).
__device__ __forceinline__ void dma_lds16_once(u32x4_t rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
               :
               : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory", "m0");
}
// The same with 4 bytes per lane (256 bytes per instruction).
__device__ __forceinline__ void dma_lds4(u32x4_t rsrc, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
               :
               : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wave_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ u32x4_t raw_rsrc(const void *base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  return u32x4_t{(uint32_t)a, (uint32_t)(a >> 32) & 0xFFFFu, bytes, 0x00020000u};
}

// ===========================================================================
// weight streaming from a fragment-packed copy
// ===========================================================================
constexpr int SK_BM = 64;                // rows per block
constexpr int SK_KC = 128;               // K per stage
constexpr int SK_ROWB = SK_KC * 2 + 16;  // LDS bytes per tile row (padded)

// The packed weight-streaming kernel's block is 128 logical columns x 64
// rows, one block per CU; each of the 4 waves owns 32 columns.
constexpr int SW_BN = 128;     // logical columns per block
constexpr int kPackedMaxRows = SK_BM;

// Where column tile ct of nct starts its walk over a K range of n 128-wide
// steps that no other block shares (it wraps around).  Blocks that all start
// at the first column read the same K offset of rows a power of two apart,
// and those addresses meet on few memory channels; an eighth of the range
// apart per XCD they spread, and the blocks of one XCD still share A's
// stages in its L2.  Gate/up at 64 rows (W 28672 x 4096): 51.5 -> 43.0 us on
// the row-major bf16 matrix, 31.8 -> 28.4 on 8-bit codes; split K ranges start
// apart by themselves (down: no change).  The order depends on the column
// tile alone, so a row's sums do not depend on the batch.
__device__ __forceinline__ int k_start(int ct, int nct, int n) { return ct * 8 / nct * n / 8; }

// Block-local logical column of row lr (0..15) of wave w's column fragment
// f (0, 1): wave w takes half w % 2 of SiLU group w / 2, fragment 0 its 16
// gate columns and fragment 1 their 16 up partners (32 further), so a lane
// holds a gate sum and its partner.
__device__ __forceinline__ int sw_col(int w, int f, int lr) { return (w >> 1) * 64 + f * 32 + (w & 1) * 16 + lr; }

// Fragment-packed weights.  A packed copy of W [N][K] (N % 16 == 0,
// K % 32 == 0) stores each 16-row x 32-column block as one contiguous
// 1 KiB run in the lane order of the MFMA's 16x16x32 operand: lane l holds
// row 16 g + l % 16, columns 32 c + 8 (l / 16) .. + 7, and block (g, c) sits
// at byte ((g * K / 32) + c) * 1024.  One 16-byte load per lane then fills an
// operand register with 1 KiB of contiguous memory.
__global__ __launch_bounds__(256) void k_pack_weight(const uint16_t *__restrict__ W, uint16_t *__restrict__ P, int N,
                                                     int K) {
  const size_t q = (size_t)blockIdx.x * 256 + threadIdx.x;  // 16-byte chunk of P
  const size_t nchunks = (size_t)N * K / 8;
  if (q >= nchunks) return;
  const int kc32 = K / 32;
  const size_t frag = q >> 6;
  const int l = (int)(q & 63);
  const size_t g = frag / kc32;
  const int c = (int)(frag - g * kc32);
  const size_t row = g * 16 + (l & 15);
  const size_t k = (size_t)c * 32 + (l >> 4) * 8;
  *reinterpret_cast<u32x4_t *>(P + q * 8) = *reinterpret_cast<const u32x4_t *>(W + row * K + k);
}

// The weight-streaming kernel on packed bf16 weights (four waves).  Same columns,
// split ranges, products and epilogues as k_gemm_stream<64, false>, but each
// wave loads its W operands straight into registers from the packed copy
// (every element of W is used by one wave only, so W needs no LDS), three
// 128-wide K stages ahead in a ring of three register sets; only A passes
// through LDS (three buffers).  The products take the same operands in the
// same order, so the sums are bitwise those of k_gemm_stream<64, false>.
// It stays for up to 64 rows because its split products are faster (8B down
// 24.7 against 29.7 us, qkv with the norm 15.6 against 18.2, o the same).  With
// more rows its 64-row blocks pass over W once each and the wider blocks of
// k_gemm_stream are faster on the row-major matrix (8B step at short contexts,
// 66 rows 195 us packed, 143 row-major; 128 rows 205, 177; 255 rows 306, 256;
// 70B layer, 80 rows 570, 382; 192 rows 734, 502).
constexpr int SP_LDS = 3 * SK_BM * SK_ROWB;
constexpr int SP_LDS_ONE = 96 * 1024;  // as launched: keeps one block per CU
static_assert(SP_LDS_ONE >= SP_LDS, "LDS");
template <bool PRENORM = false>
__global__ __launch_bounds__(256) void k_gemm_skinny_packed(const uint16_t *__restrict__ A, const uint16_t *__restrict__ Wp,
                                                            uint16_t *__restrict__ out, const uint16_t *__restrict__ res,
                                                            float *__restrict__ part, int M, int N, int K, int epi,
                                                            int ksteps_per_split, int tiles, int mt, int per_xcd,
                                                            const uint16_t *__restrict__ gamma = nullptr,
                                                            float *__restrict__ ssq = nullptr) {
  extern __shared__ __attribute__((aligned(16))) uint8_t sp_lds[];  // [3][64 A rows][SK_ROWB]
  const int t = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (t >= tiles) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = (t / mt) * SW_BN;
  const int split = blockIdx.y;
  const int m0 = (t % mt) * SK_BM;
  const int kbeg = split * ksteps_per_split * 32;
  const int kend = min(K, kbeg + ksteps_per_split * 32);
  const int nst = kend > kbeg ? (kend - kbeg + SK_KC - 1) / SK_KC : 0;
  const buf_rsrc_t ra = make_rsrc(A, (int)min((size_t)M * K * 2, (size_t)0x7FFFFFFF));
  const buf_rsrc_t rw = make_rsrc(Wp, (int)min((size_t)N * K * 2, (size_t)0x7FFFFFFF));

  // W: fragment f of this wave covers W rows wr_f .. wr_f + 15 (a 16-aligned
  // run, or none); its 32-wide K step kc is the 1 KiB run at
  // (wr_f / 16 * K / 32 + kc) * 1024, of which this lane reads 16 bytes.
  uint32_t wbase[2];
  bool wok[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int wr = w_row_of(n0 + sw_col(wave, f, 0), N, epi);
    wok[f] = wr >= 0;
    wbase[f] = wok[f] ? ((uint32_t)(wr >> 4) * (uint32_t)(K >> 5)) * 1024u + (uint32_t)lane * 16u : 0u;
  }
  const int kc0 = kbeg >> 5, kc_end = kend >> 5;
  u32x4_t w0[2][4], w1[2][4], w2[2][4];
  // stage s of the walk is K stage at(s) of the range (see k_start)
  const int rot = gridDim.y == 1 ? k_start(t / mt, tiles / mt, nst) : 0;
  auto at = [&](int s) { return s + rot < nst ? s + rot : s + rot - nst; };
  auto wload = [&](int s, u32x4_t (&wr)[2][4]) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int kc = kc0 + at(s) * 4 + ks;
#pragma unroll
      for (int f = 0; f < 2; ++f)
        wr[f][ks] = buf_ld_u32x4<kAuxNT>(
            rw, (int)(wok[f] && s < nst && kc < kc_end ? wbase[f] + (uint32_t)kc * 1024u : 0x80000000u));
    }
  };

  // A: thread t moves 16-byte chunk t % 16 of tile rows t / 16 + 16 j (j < 4)
  const int ch = tid & 15, r0 = tid >> 4;
  uint32_t aoff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int m = m0 + r0 + 16 * j;
    aoff[j] = m < M ? ((uint32_t)m * (uint32_t)K + (uint32_t)(ch * 8)) * 2u : 0x80000000u;
  }
  u32x4_t aa[4];
  u32x4_t ga = {0u, 0u, 0u, 0u};
  float ssacc[4] = {0.f, 0.f, 0.f, 0.f};
  const buf_rsrc_t rg = make_rsrc(PRENORM ? gamma : A, PRENORM ? K * 2 : 16);
  auto aload = [&](int s) {
    const int k = kbeg + at(s) * SK_KC + ch * 8;
    const bool ok = s < nst && k < kend;
    const uint32_t kb = (uint32_t)(kbeg + at(s) * SK_KC) * 2u;
#pragma unroll
    for (int j = 0; j < 4; ++j) aa[j] = buf_ld_u32x4<0>(ra, (int)(ok ? aoff[j] + kb : 0x80000000u));
    if constexpr (PRENORM) ga = buf_ld_u32x4<0>(rg, (int)(ok ? (uint32_t)(k * 2) : 0x80000000u));
  };
  const bool first_col_tile = n0 == 0;
  auto awrite = [&](int buf) {
    uint8_t *b = sp_lds + buf * SK_BM * SK_ROWB;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      u32x4_t av = aa[j];
      if constexpr (PRENORM) {
        if (first_col_tile) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float lo = bf16_lo(aa[j][e]), hi = bf16_hi(aa[j][e]);
            ssacc[j] += lo * lo + hi * hi;
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          av[e] = pack_bf16x2(bf16_lo(aa[j][e]) * bf16_lo(ga[e]), bf16_hi(aa[j][e]) * bf16_hi(ga[e]));
      }
      *reinterpret_cast<u32x4_t *>(b + (r0 + 16 * j) * SK_ROWB + ch * 16) = av;
    }
  };
  f32x4_t acc[2][4];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[f][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int lr = lane & 15, lg = lane >> 4;
  auto compute = [&](int buf, const u32x4_t (&wr)[2][4]) {
    const uint8_t *b = sp_lds + buf * SK_BM * SK_ROWB;
#pragma unroll
    for (int ks = 0; ks < SK_KC / 32; ++ks) {
      u32x4_t af[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        af[i] = *reinterpret_cast<const u32x4_t *>(b + (i * 16 + lr) * SK_ROWB + (ks * 4 + lg) * 16);
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[f][i] = mfma16x16x32(wr[f][ks], af[i], acc[f][i]);
    }
  };
  // Stage s: compute(s) from A buffer s % 3 and W set s % 3; write A(s + 2)
  // (loaded during stage s - 1) into buffer (s + 2) % 3; load A(s + 3), then
  // W(s + 3) into the set just consumed; one barrier.  A's loads go out
  // before W's so that waiting for A(s + 2) never waits for W(s + 2).
  aload(0);
  wload(0, w0);
  awrite(0);
  aload(1);
  wload(1, w1);
  awrite(1);
  aload(2);
  wload(2, w2);
  __syncthreads();
  auto stage = [&](int s, int buf, u32x4_t (&wr)[2][4]) {
    compute(buf, wr);
    awrite(buf == 0 ? 2 : buf - 1);
    aload(s + 3);
    wload(s + 3, wr);
    __syncthreads();
  };
  int s = 0;
  for (; s + 3 <= nst; s += 3) {
    stage(s, 0, w0);
    stage(s + 1, 1, w1);
    stage(s + 2, 2, w2);
  }
  // one or two stages left: A(s) and A(s + 1) already sit in buffers 0 and 1
  if (s < nst) compute(0, w0);
  if (s + 1 < nst) compute(1, w1);
  if constexpr (PRENORM) {
    if (first_col_tile) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = group_sum<16>(ssacc[j]);
        const int m = m0 + r0 + 16 * j;
        if (ch == 0 && m < M) ssq[(size_t)split * M + m] = v;
      }
    }
  }

  const int ncols = logical_cols(N, epi);
  int cf[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) cf[f] = n0 + sw_col(wave, f, 4 * lg);
  if (part) {
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = m0 + i * 16 + lr;
        if (m < M && cf[f] < ncols)
          *reinterpret_cast<f32x4_t *>(part + ((size_t)split * M + m) * ncols + cf[f]) = acc[f][i];
      }
    return;
  }
  if (epi == EPI_SILU_MUL) {
    const int F = N >> 1;
    const int fo = ((n0 + (wave >> 1) * 64) >> 1) + (wave & 1) * 16 + 4 * lg;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + i * 16 + lr;
      if (m < M && fo < F) {
        const f32x4_t g = acc[0][i], u = acc[1][i];
        const u32x2_t w = {pack_bf16x2(silu_f(g[0]) * u[0], silu_f(g[1]) * u[1]),
                           pack_bf16x2(silu_f(g[2]) * u[2], silu_f(g[3]) * u[3])};
        *reinterpret_cast<u32x2_t *>(out + (size_t)m * F + fo) = w;
      }
    }
    return;
  }
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int n = cf[f];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + i * 16 + lr;
      if (m < M && n < N) {
        f32x4_t v = acc[f][i];
        if (epi == EPI_RESIDUAL) {
          const u32x2_t r = *reinterpret_cast<const u32x2_t *>(res + (size_t)m * N + n);
          v[0] += bf16_lo(r[0]);
          v[1] += bf16_hi(r[0]);
          v[2] += bf16_lo(r[1]);
          v[3] += bf16_hi(r[1]);
        }
        const u32x2_t w = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
        *reinterpret_cast<u32x2_t *>(out + (size_t)m * N + n) = w;
      }
    }
  }
}

// Sum split-K partials (logical column space) and apply the epilogue.
__global__ __launch_bounds__(256) void k_gemm_splitk_epilogue(const float *__restrict__ part, int splits,
                                                              uint16_t *__restrict__ out,
                                                              const uint16_t *__restrict__ res, int M, int N,
                                                              int epi) {
  // two consecutive output columns per thread and step (N and F are even,
  // and a SiLU group of 32 never splits a pair; two rather than four columns
  // so that a decode batch's few rows still give the chip many waves), the
  // loads of up to eight splits issued before they are added; each element
  // sums its splits in order, then adds the residual
  typedef float f2_t __attribute__((ext_vector_type(2)));
  const int ncols = logical_cols(N, epi);
  const int outc = epi == EPI_SILU_MUL ? N / 2 : N;
  const long total2 = (long)M * (outc / 2);
  const size_t stride = (size_t)M * ncols;
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < total2; idx += (long)gridDim.x * blockDim.x) {
    const int m = (int)(idx / (outc / 2)), n = 2 * (int)(idx - (long)m * (outc / 2));
    const bool silu = epi == EPI_SILU_MUL;
    const int col = silu ? (n / 32) * 64 + (n & 31) : n;
    const float *p0 = part + (size_t)m * ncols + col;
    f2_t x = {0.f, 0.f}, u = {0.f, 0.f};
    for (int s0 = 0; s0 < splits; s0 += 8) {
      f2_t a[8], b[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const bool ok = s0 + q < splits;
        a[q] = ok ? *reinterpret_cast<const f2_t *>(p0 + (s0 + q) * stride) : f2_t{0.f, 0.f};
        b[q] = ok && silu ? *reinterpret_cast<const f2_t *>(p0 + (s0 + q) * stride + 32) : f2_t{0.f, 0.f};
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        x += a[q];
        u += b[q];
      }
    }
    uint32_t w;
    if (silu) {
      w = pack_bf16x2(silu_f(x[0]) * u[0], silu_f(x[1]) * u[1]);
    } else {
      if (epi == EPI_RESIDUAL) {
        const uint32_t r = *reinterpret_cast<const uint32_t *>(res + (size_t)m * N + n);
        x[0] += bf16_lo(r);
        x[1] += bf16_hi(r);
      }
      w = pack_bf16x2(x[0], x[1]);
    }
    *reinterpret_cast<uint32_t *>(out + (size_t)m * outc + n) = w;
  }
}

// Grouped use (the experts of a mixture-of-experts block): a row tile is some
// expert-sorted rows of one expert (tables [3][max_tiles]: expert, first
// sorted row, rows); its columns are those of that expert's W ([E][N][K]); A
// rows are gathered through a_rows (null: the sorted row itself); the store
// epilogue writes fp32.
struct GroupedArgs {
  const int32_t *a_rows, *tiles, *n_tiles;
  int max_tiles, a_nrows, f32_out;
};

// ===========================================================================
// stream: the weight-streaming kernel.  What bounds it is W's way from HBM,
// so all of the CU's LDS is a ring of K stages loaded straight into it (no
// register between, nothing for the compiler to wait on), and each stage waits
// for its own loads by count, leaving 4 or 5 stages (96-120 KiB per CU at up
// to 64 rows) in flight across the one barrier a stage has.  The kernel before
// it staged through registers, two 128-wide stages ahead, and drained at each
// barrier: 64 rows, qkv 22.3 -> 17.8 us, gate/up 51.2 -> 43.3; 8-bit W at 37
// rows, gate/up 41.0 -> 28.1, down 24.7 -> 20.4; more rows: stream_us.
//
// Eight waves, two on each SIMD, so that one issues loads or waits while the
// other multiplies (four waves, one a SIMD, before: 8-bit W at 37 rows, gate/up
// 28.5 -> 26.9 us, down 21.2 -> 20.0; 160 rows, qkv 26.2 -> 25.0, O 22.5 -> 21.6;
// 240 rows, gate/up 74 -> 71).  Wave grid: 2 x 4 (32 columns a wave, half the rows) to 64 rows, 4 x
// 2 (64 columns, a quarter of the rows) above, which reads each W fragment
// from LDS for fewer waves.  Measured and not taken: a ring of its own for W
// and for A, W's deeper, loaded by half of the waves each (one wave then
// issues twice the loads per stage: 8B O and down slower by 3 to 5 %).
//
// PRENORM (split-K partials only): A holds the rows x of an RMSNorm that
// precedes the product.  A landed stage's rows become bf16(x * gamma) in place
// one stage before they are multiplied, and the blocks of the first column
// tile write each row's partial sum of squares over their K range to
// ssq[split][M]; the row scale 1 / sqrt(mean(x^2) + eps) is applied to the
// summed partials by the consumer (RMSNorm(x) g W^T = inv * ((x g) W^T)).
//
// GROUPED (its waves a block): the experts of a mixture-of-experts block with a
// few rows each.  Half the LDS per block, so that a block's start is hidden by
// its neighbour (a block lasts 32 stages or less), an expert's column tiles
// side by side on one XCD.  128 experts of 768 over hidden 2048, 64 tokens: gate/up 151 -> 134
// us (6.0 TB/s), down 85 -> 73 against the register-staged 64 x 64 tiles it
// replaced; 512 tokens 172 + 100 -> 147 + 84.
// ===========================================================================
constexpr int ST_BN = 128;  // logical columns per block
// Rows per block, K per stage and ring depth: a stage holds 128 W rows and BM
// A rows of KC values (bf16: 64, rows of 128 bytes; 8-bit W: 128, W rows of
// 128 bytes of codes), the ring fills the CU's LDS (160 KiB less the norm
// gains), all but one stage of it in flight.
template <int BM, bool W8, bool PRENORM, int GROUPED = 0>
struct StreamTraits {
  static constexpr int KC = W8 ? 128 : 64;
  static constexpr int WROW = KC * (W8 ? 1 : 2);       // bytes of a W row
  static constexpr int AROW = KC * 2;                 // bytes of an A row
  static constexpr int W_BYTES = ST_BN * WROW;        // W part of a stage
  static constexpr int A_BYTES = BM * AROW;
  static constexpr int G_BYTES = PRENORM ? 256 : 0;   // the stage's norm gains
  static constexpr int STAGE = W_BYTES + A_BYTES + G_BYTES;
  static constexpr int R = (GROUPED ? 80 * 1024 : 160 * 1024) / STAGE;  // (grouped: two blocks per CU)
  static constexpr int LDS = R * STAGE;
  static_assert(R >= 2, "ring depth");
  static constexpr int NW = GROUPED ? GROUPED : 8;  // waves: two on each SIMD (grouped, 4: one of each of two blocks)
  static constexpr int WM = NW == 4 ? 1 : BM >= 128 ? 4 : 2, WN = NW / WM;  // wave grid
  static constexpr int NF = ST_BN / WN / 16;          // 16-column fragments per wave
  static constexpr int NI = BM / WM / 16;             // 16-row blocks per wave
  static constexpr int LA = A_BYTES / (NW * 1024), LW = W_BYTES / (NW * 1024);  // load instructions per wave and stage
  static_assert(LA * NW * 1024 == A_BYTES && LW * NW * 1024 == W_BYTES && NI * WM * 16 == BM, "wave shares");
};

template <int BM, bool W8, bool PRENORM, int GROUPED = 0, bool ONCE = false>
__global__ __launch_bounds__((64 * StreamTraits<BM, W8, PRENORM, GROUPED>::NW)) void k_gemm_stream(
    const uint16_t *__restrict__ A, const void *__restrict__ W, const float *__restrict__ wscale,
    uint16_t *__restrict__ out, const uint16_t *__restrict__ res, float *__restrict__ part, int M, int N, int K, int epi,
    int ksteps_per_split, int tiles, int mt, int per_xcd, const uint16_t *__restrict__ gamma, float *__restrict__ ssq,
    GroupedArgs ga = GroupedArgs{}) {
  using Tr = StreamTraits<BM, W8, PRENORM, GROUPED>;
  constexpr int KC = Tr::KC, R = Tr::R, NF = Tr::NF, NI = Tr::NI, LA = Tr::LA, LW = Tr::LW, AROW = Tr::AROW;
  constexpr int NL = LA + LW + (PRENORM ? 1 : 0);  // loads per wave and stage
  constexpr uint32_t WES = W8 ? 1u : 2u;
  extern __shared__ __attribute__((aligned(16))) uint8_t st_lds[];  // [R][W | A | gains]
  // block b takes tile (b % 8) * per_xcd + b / 8, so each XCD walks its own
  // contiguous tile range; the mt row blocks of one column tile are
  // neighbours there and share the W tile through that XCD's L2
  // (grouped: mt column tiles per row tile, so an expert's tiles stay on one XCD)
  if constexpr (GROUPED) {
    tiles = __builtin_amdgcn_readfirstlane(*ga.n_tiles) * mt;
    per_xcd = (tiles + 7) / 8;
    if ((int)(blockIdx.x / 8) >= per_xcd) return;
  }
  const int t = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (t >= tiles) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / Tr::WN, wn = wave % Tr::WN;
  const int ct = GROUPED ? t % mt : t / mt, nct = GROUPED ? mt : tiles / mt;  // column tile, of nct
  const int n0 = ct * ST_BN;
  int m0 = GROUPED ? 0 : (t % mt) * BM;
  if constexpr (GROUPED) {  // the tile's rows as a matrix of its own: M rows, W and the outputs at their places
    const int rt = t / mt;
    const int e = __builtin_amdgcn_readfirstlane(ga.tiles[rt]);
    const int row0 = __builtin_amdgcn_readfirstlane(ga.tiles[ga.max_tiles + rt]);
    M = __builtin_amdgcn_readfirstlane(ga.tiles[2 * ga.max_tiles + rt]);
    W = static_cast<const uint16_t *>(W) + (size_t)e * N * K;
    if (part) part += (size_t)row0 * N;
    if (out) out += (size_t)row0 * (epi == EPI_SILU_MUL ? N / 2 : N);
    m0 = row0;  // (of the sorted rows, for the loads below)
  }
  const int split = blockIdx.y;
  const int kbeg = split * ksteps_per_split * 32;
  const int kend = min(K, kbeg + ksteps_per_split * 32);
  const int nst = kend > kbeg ? (kend - kbeg + KC - 1) / KC : 0;
  const uint32_t a_bytes = (uint32_t)min((size_t)(GROUPED ? ga.a_nrows : M) * K * 2, (size_t)0x7FFFFFFF);
  const uint32_t w_bytes = (uint32_t)min((size_t)N * K * WES, (size_t)0x7FFFFFFF);

  // Loads.  A wave's load instruction i fills 1 KiB of LDS: rows of 128 bytes
  // (8 of them) or 256 (4); lane l writes 16-byte position l % 8 (l % 16) of
  // its row with the logical chunk swizzled there.  Rows outside the
  // operands and k past the block's range point past every descriptor's
  // range: they load zeros without traffic.
  auto swz = [](int row, int c, int rowb) { return rowb == 128 ? c ^ ((row >> 1) & 7) : c ^ (row & 15); };
  constexpr int RPI = 1024 / AROW, CPR = AROW / 16;  // A rows per load instruction, chunks per row
  constexpr int CK = W8 ? 16 : 8;                    // W values per chunk
  constexpr int WROW = Tr::WROW, WRPI = 1024 / WROW, WCPR = WROW / 16;
  uint32_t woff[LW], aoff[LA];
  auto wchunk = [&](int i) { return swz((wave * LW + i) * WRPI + lane / WCPR, lane % WCPR, WROW); };
  auto achunk = [&](int i) { return swz((wave * LA + i) * RPI + lane / CPR, lane % CPR, AROW); };
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int wr = w_row_of(n0 + (wave * LW + i) * WRPI + lane / WCPR, N, epi);
    woff[i] = wr >= 0 ? (uint32_t)wr * (uint32_t)K * WES + (uint32_t)wchunk(i) * 16u : 0x80000000u;
  }
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (wave * LA + i) * RPI + lane / CPR;
    int m = GROUPED ? (r < M ? m0 + r : -1) : (m0 + r < M ? m0 + r : -1);
    if constexpr (GROUPED) {
      if (m >= 0 && ga.a_rows) m = ga.a_rows[m];
      if (m >= ga.a_nrows) m = -1;
    }
    aoff[i] = m >= 0 ? (uint32_t)m * (uint32_t)K * 2u + (uint32_t)achunk(i) * 16u : 0x80000000u;
  }
  if constexpr (GROUPED) m0 = 0;  // the outputs' rows
  const u32x4_t ra = raw_rsrc(A, a_bytes), rw = raw_rsrc(W, w_bytes);
  const u32x4_t rg = raw_rsrc(PRENORM ? gamma : A, PRENORM ? (uint32_t)K * 2u : 0u);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)st_lds;
  constexpr auto dma_w = ONCE ? dma_lds16_once : dma_lds16;
  // stage s into the ring slot at byte `slot`
  const int rot = gridDim.y == 1 ? k_start(ct, nct, (kend - kbeg + 127) / 128) * (128 / KC) : 0;
  auto issue = [&](int s, uint32_t slot) {
    const int k0 = s >= nst ? kend : kbeg + (s + rot < nst ? s + rot : s + rot - nst) * KC;
    const uint32_t dw = lds0 + slot + (uint32_t)(wave * LW) * 1024u;
    const uint32_t da = lds0 + slot + Tr::W_BYTES + (uint32_t)(wave * LA) * 1024u;
    if constexpr (PRENORM) {
      // (all waves write the same values; gains past the range are zero like
      // the rows they meet there: an infinite one would make a NaN of them)
      const int k = k0 + 2 * lane;
      dma_lds4(rg, k < kend ? (uint32_t)(k * 2) : 0x80000000u, 0u, lds0 + slot + Tr::W_BYTES + Tr::A_BYTES);
    }
    if (k0 + KC <= kend) {
#pragma unroll
      for (int i = 0; i < LA; ++i) dma_lds16(ra, aoff[i], (uint32_t)k0 * 2u, da + i * 1024);
#pragma unroll
      for (int i = 0; i < LW; ++i) dma_w(rw, woff[i], (uint32_t)k0 * WES, dw + i * 1024);
    } else {  // the last stage of a ragged range, or past it (8-bit W: see clear_tail)
#pragma unroll
      for (int i = 0; i < LA; ++i)
        dma_lds16(ra, k0 + achunk(i) * 8 < kend && aoff[i] != 0x80000000u ? aoff[i] + (uint32_t)k0 * 2u : 0x80000000u, 0u,
                  da + i * 1024);
#pragma unroll
      for (int i = 0; i < LW; ++i)
        dma_w(rw, k0 + wchunk(i) * CK < kend && woff[i] != 0x80000000u ? woff[i] + (uint32_t)k0 * WES : 0x80000000u, 0u,
              dw + i * 1024);
    }
  };

  f32x4_t acc[NF][NI];
#pragma unroll
  for (int f = 0; f < NF; ++f)
#pragma unroll
    for (int i = 0; i < NI; ++i) acc[f][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int lr = lane & 15, lg = lane >> 4;
  // block-local logical column of fragment f's first W row
  auto fcol = [&](int f) { return NF == 2 ? sw_col(wn, f, 0) : wn * 64 + f * 16; };
  const int sw8 = (lr >> 1) & 7;
  auto compute = [&](uint32_t slot) {
    const uint8_t *w = st_lds + slot + lr * WROW;
    const uint8_t *a = st_lds + slot + Tr::W_BYTES + (wm * NI * 16 + lr) * AROW;
#pragma unroll
    for (int q = 0; q < KC / (W8 ? 64 : 32); ++q) {
      u32x4_t wc[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f)
        wc[f] = *reinterpret_cast<const u32x4_t *>(w + fcol(f) * WROW + (((q * 4 + lg) ^ (WROW == 128 ? sw8 : lr)) << 4));
#pragma unroll
      for (int h = 0; h < (W8 ? 2 : 1); ++h) {
        // 8-bit W: a lane's 16 codes are k = 16 (4 q + lg) .. + 15, A's chunks in the same order
        const int c = W8 ? (2 * (q * 4 + lg) + h) ^ lr : (q * 4 + lg) ^ (AROW == 128 ? sw8 : lr);
        u32x4_t wf[NF], af[NI];
#pragma unroll
        for (int f = 0; f < NF; ++f)
          wf[f] = W8 ? e4m3x8_to_bf16x8(u32x2_t{wc[f][2 * h], wc[f][2 * h + 1]}) : wc[f];
#pragma unroll
        for (int i = 0; i < NI; ++i) af[i] = *reinterpret_cast<const u32x4_t *>(a + i * 16 * AROW + (c << 4));
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
          for (int i = 0; i < NI; ++i) acc[f][i] = mfma16x16x32(wf[f], af[i], acc[f][i]);
      }
    }
  };
  // 8-bit W whose K ends 8 codes into a 16-code chunk: the chunk's other 8
  // are the next W row's first codes.  A is zero there, but a NaN code times
  // zero is NaN, so they are cleared in the landed stage before its products.
  const int tail_stage = W8 && (kend & 8) ? nst - 1 - rot : -1;  // walk position of the range's last stage
  auto clear_tail = [&](uint32_t slot) {
    const int c = ((kend - kbeg) % KC) / CK;  // (ranges begin at multiples of 32)
    if (tid < ST_BN) *reinterpret_cast<u32x2_t *>(st_lds + slot + tid * WROW + (swz(tid, c, WROW) << 4) + 8) = u32x2_t{0u, 0u};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wave_barrier();
  };
  // PRENORM: the A rows of a landed stage become bf16(x * gain) in place, the
  // blocks of the first column tile adding up their squares on the way
  constexpr int NT = 64 * Tr::NW, TJ = Tr::A_BYTES / (NT * 16);
  float ssacc[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) ssacc[j] = 0.f;
  const bool first_col_tile = n0 == 0;
  auto prenorm = [&](uint32_t slot) {
    const int p = tid % CPR, row = tid / CPR;  // rows + (NT / CPR) j: the same chunk for all j
    const int c = swz(row, p, AROW);
    uint8_t *a = st_lds + slot + Tr::W_BYTES + row * AROW + p * 16;
    const u32x4_t g = *reinterpret_cast<const u32x4_t *>(st_lds + slot + Tr::W_BYTES + Tr::A_BYTES + c * 16);
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      u32x4_t x = *reinterpret_cast<const u32x4_t *>(a + j * NT * 16);
      if (first_col_tile) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = bf16_lo(x[e]), hi = bf16_hi(x[e]);
          ssacc[j] += lo * lo + hi * hi;
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = pack_bf16x2(bf16_lo(x[e]) * bf16_lo(g[e]), bf16_hi(x[e]) * bf16_hi(g[e]));
      *reinterpret_cast<u32x4_t *>(a + j * NT * 16) = x;
    }
  };

  // Stage s: wait until it (PRENORM: and the A rows of stage s + 1) landed in
  // every wave, refill the slot read in stage s - 1 with stage s + R - 1, then
  // multiply.  The younger stages stay in flight across the barrier.
  auto next = [&](uint32_t slot) { return slot + Tr::STAGE == Tr::LDS ? 0u : slot + Tr::STAGE; };
  uint32_t fill = 0;
#pragma unroll
  for (int s = 0; s < R - 1; ++s) {
    issue(s, fill);
    fill += Tr::STAGE;
  }
  uint32_t slot = 0;
  if constexpr (PRENORM) {
    wait_loads<(R - 2) * NL + LW>();
    wave_barrier();
    prenorm(0);
  }
  for (int s = 0; s < nst; ++s) {
    wait_loads<PRENORM ? (R - 3) * NL + LW : (R - 2) * NL>();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wave_barrier();
    issue(s + R - 1, fill);
    fill = next(fill);
    if constexpr (PRENORM) prenorm(next(slot));
    if constexpr (W8) {
      if (s == tail_stage) clear_tail(slot);
    }
    compute(slot);
    slot = next(slot);
  }
  wait_loads<0>();
  if constexpr (PRENORM) {
    if (first_col_tile) {
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const float v = group_sum<CPR>(ssacc[j]);
        const int m = m0 + tid / CPR + (NT / CPR) * j;
        if (tid % CPR == 0 && m < M) ssq[(size_t)split * M + m] = v;
      }
    }
  }

  // lane: rows m = m0 + 16 (wm NI + i) + lr; fragment f holds logical columns
  // n0 + fcol(f) + 4 lg .. + 3
  const int ncols = logical_cols(N, epi);
  if constexpr (W8) {
#pragma unroll
    for (int f = 0; f < NF; ++f) {
      const int c = n0 + fcol(f) + 4 * lg;
      if (c < ncols) {
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[f][i] = row_scaled(acc[f][i], wscale, c, N, epi);
      }
    }
  }
  const int mrow = m0 + wm * NI * 16 + lr;
  if (part) {  // split-K partial, logical column space
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int m = mrow + i * 16, c = n0 + fcol(f) + 4 * lg;
        if (m < M && c < ncols) *reinterpret_cast<f32x4_t *>(part + ((size_t)split * M + m) * ncols + c) = acc[f][i];
      }
    return;
  }
  if (epi == EPI_SILU_MUL) {
    // fragment f holds gate sums, fragment f + NF / 2 their up partners
    const int F = N >> 1;
#pragma unroll
    for (int f = 0; f < NF / 2; ++f) {
      const int c = n0 + fcol(f);  // (32 gate columns, then 32 up, per group of 64)
      const int fo = (c >> 6) * 32 + (c & 31) + 4 * lg;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int m = mrow + i * 16;
        if (m < M && fo < F) {
          const f32x4_t g = acc[f][i], u = acc[f + NF / 2][i];
          *reinterpret_cast<u32x2_t *>(out + (size_t)m * F + fo) =
              u32x2_t{pack_bf16x2(silu_f(g[0]) * u[0], silu_f(g[1]) * u[1]),
                      pack_bf16x2(silu_f(g[2]) * u[2], silu_f(g[3]) * u[3])};
        }
      }
    }
    return;
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int n = n0 + fcol(f) + 4 * lg;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int m = mrow + i * 16;
      if (m < M && n < N) {
        f32x4_t v = acc[f][i];
        if (epi == EPI_RESIDUAL) {
          const u32x2_t r = *reinterpret_cast<const u32x2_t *>(res + (size_t)m * N + n);
          v += f32x4_t{bf16_lo(r[0]), bf16_hi(r[0]), bf16_lo(r[1]), bf16_hi(r[1])};
        }
        *reinterpret_cast<u32x2_t *>(out + (size_t)m * N + n) =
            u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
      }
    }
  }
}

// ===========================================================================
// tiled
// ===========================================================================
constexpr int TL_BM = 128, TL_BN = 128, TL_BK = 64, TL_LDK = TL_BK + 8;

__global__ __launch_bounds__(256) void k_gemm_tiled(const uint16_t *__restrict__ A, const uint16_t *__restrict__ W,
                                                    uint16_t *__restrict__ out, const uint16_t *__restrict__ res,
                                                    int M, int N, int K, int epi, int tiles_m, int tiles_n) {
  __shared__ __attribute__((aligned(16))) uint16_t sA[2][TL_BM * TL_LDK];
  __shared__ __attribute__((aligned(16))) uint16_t sB[2][TL_BN * TL_LDK];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  // tile order: column-major over M inside groups of 8 N tiles, so that
  // consecutive blocks share the same A rows and a small band of W rows
  const int bid = blockIdx.x;
  const int group = 8;
  const int per_group = group * tiles_m;
  const int gidx = bid / per_group;
  const int first_n = gidx * group;
  const int gsz = min(group, tiles_n - first_n);
  const int inb = bid - gidx * per_group;
  const int tn = first_n + inb % gsz;
  const int tm = inb / gsz;
  const int m0 = tm * TL_BM, n0 = tn * TL_BN;
  const int nk = (K + TL_BK - 1) / TL_BK;

  // global -> register staging: 4 chunks of 16 B for A and for W per thread
  const int ldr = threadIdx.x >> 3;        // row 0..31 within a pass
  const int ldc = (threadIdx.x & 7) * 8;   // k offset
  const uint16_t *ga[4];
  const uint16_t *gb[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int m = m0 + p * 32 + ldr;
    ga[p] = m < M ? A + (size_t)m * K : nullptr;
    const int wr = w_row_of(n0 + p * 32 + ldr, N, epi);
    gb[p] = wr >= 0 ? W + (size_t)wr * K : nullptr;
  }
  u32x4_t ra[4], rb[4];
  auto gload = [&](int kt) {
    const int k = kt * TL_BK + ldc;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      ra[p] = (ga[p] && k < K) ? ld_u32x4(ga[p] + k) : u32x4_t{0, 0, 0, 0};
      rb[p] = (gb[p] && k < K) ? ld_u32x4(gb[p] + k) : u32x4_t{0, 0, 0, 0};
    }
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      st_u32x4(&sA[buf][(p * 32 + ldr) * TL_LDK + ldc], ra[p]);
      st_u32x4(&sB[buf][(p * 32 + ldr) * TL_LDK + ldc], rb[p]);
    }
  };
  f32x4_t acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int lr = lane & 15, lk = (lane >> 4) * 8;
  gload(0);
  sstore(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < nk) gload(kt + 1);
#pragma unroll
    for (int kk = 0; kk < TL_BK; kk += 32) {
      u32x4_t a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = ld_u32x4(&sA[buf][(wm * 64 + i * 16 + lr) * TL_LDK + kk + lk]);
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = ld_u32x4(&sB[buf][(wn * 64 + j * 16 + lr) * TL_LDK + kk + lk]);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma16x16x32(a[i], b[j], acc[i][j]);
    }
    if (kt + 1 < nk) sstore(buf ^ 1);
    __syncthreads();
  }
  // epilogue straight from the accumulator layout: lane holds rows
  // 4 (lane/16) + e, column lane % 16 of each 16x16 block
  const int cbase = n0 + wn * 64;
  if (epi == EPI_SILU_MUL) {
    const int F = N >> 1;
    const int f0 = cbase >> 1;  // 64-group -> 32 ffn columns
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = m0 + wm * 64 + i * 16 + (lane >> 4) * 4 + e;
          const int f = f0 + j * 16 + lr;
          if (m < M && f < F)
            out[(size_t)m * F + f] = (uint16_t)f32_to_bf16_bits(silu_f(acc[i][j][e]) * acc[i][j + 2][e]);
        }
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + wm * 64 + i * 16 + (lane >> 4) * 4 + e;
        const int n = cbase + j * 16 + lr;
        if (m < M && n < N) {
          float x = acc[i][j][e];
          if (epi == EPI_RESIDUAL) x += bf16_to_f32(res[(size_t)m * N + n]);
          out[(size_t)m * N + n] = (uint16_t)f32_to_bf16_bits(x);
        }
      }
}

// ===========================================================================
// big: 256 x 256 output tiles for large M (prefill-sized batches).  K tiles
// of 64 stream straight from global memory (buffer loads with an LDS
// destination: no register round trip) into two LDS buffers, each cut into
// four half tiles (rows 0..63 and 64..127 of every wave's 128 A rows, columns
// 0..31 and 32..63 of its 64 W columns).  8 waves (2 along M x 4 along N) each
// own a 128 x 64 sub-tile.
//
// What bounds it is latency on the way to the matrix cores, so two things
// are kept apart from them.  (1) A K tile is four phases of 16 products, one
// per quadrant (half of A x half of W); each phase reads from LDS the one
// half tile that the next products need (W0, W1, A1, then A0 of the next K
// tile) and issues the load of one half tile into the place that was read
// two phases before, so six half tiles' worth of phases lie between a load
// and its use, and the wait in each phase leaves the five youngest half tiles
// (80 KiB per CU) in flight: the load stream never drains.  (2) The two
// wave rows, one wave of each on every SIMD, run half a phase apart
// (the second passes one extra barrier first): while one multiplies, the
// other reads LDS and issues loads (raising the multiplying wave's priority
// adds nothing).  Against one barrier and a full drain
// per K tile: gate/up at 8192 rows (N 28672, K 4096) 1456 -> 1365 us, down
// (N 4096, K 14336) 800 -> 691, qkv at 2048 rows 106 -> 92, 70B gate/up at
// 256 rows 253 -> 221; without the half-phase offset 1614 / 804 us.
//
// Safety of the reuse: a half tile read in phase p is complete in every
// wave (lgkmcnt(0) before its products) before the barrier that ends phase
// p of the later wave row, and refilled in phase p + 2; a half tile read in
// phase p was waited for by every wave before the barrier in its phase p - 1.
//
// The product is formed transposed, C^T = W A^T, so that each lane's
// accumulators hold 4 consecutive output columns of one row and the epilogue
// stores 8 bytes at a time.  LDS rows are 128 bytes (64 bf16 of K); the
// 16-byte chunk c of row r sits at chunk c ^ ((r >> 1) & 7), which makes the
// MFMA operand reads of 16 consecutive rows conflict free.  8-bit W tiles
// stay codes in LDS (64-byte rows, chunk c at c ^ ((r >> 2) & 3)) and are
// converted when read (835 rows: gate/up 218 -> 196 us; 8192 rows 1570 ->
// 1394), instead of passing through registers on their way in.
// With fewer tiles than CUs (decode-sized M of 256 against a few thousand
// columns) blocks split K (gridDim.y splits of kt_per K tiles) and write
// fp32 partials in logical column space for the split-K epilogue kernel.
// Requires K % 64 == 0, N % 8 == 0 and both operands under 2 GiB (32-bit
// offsets).
// ===========================================================================
constexpr int BG_BM = 256, BG_BN = 256, BG_BK = 64;
constexpr int BG_THREADS = 512;
constexpr int BG_TILE_BYTES = 256 * BG_BK * 2;  // one operand tile: 32 KiB
constexpr int BG_HALF_BYTES = BG_TILE_BYTES / 2;

__device__ __forceinline__ int bg_swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

template <int epi, bool W8, bool GROUPED>
__global__ __launch_bounds__(BG_THREADS) void k_gemm_big(const uint16_t *__restrict__ A, const void *__restrict__ W,
                                                         const float *__restrict__ wscale, uint16_t *__restrict__ out,
                                                         const uint16_t *__restrict__ res, float *__restrict__ part,
                                                         int M, int N, int K, int tiles_m, int tiles_n,
                                                         int per_xcd, int kt_per, GroupedArgs ga) {
  extern __shared__ __attribute__((aligned(16))) uint8_t bg_lds[];  // [2][A0 | A1 | W0 | W1]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;  // 128 rows of M, 64 columns of N
  // XCD-aware tile order: blocks are dealt round-robin to the 8 XCDs, so
  // block b works on tile (b % 8) * per_xcd + b / 8: each XCD walks its own
  // contiguous run of the (grouped) tile order and its L2 keeps the shared
  // A and W panels.
  int total = tiles_m * tiles_n;
  if constexpr (GROUPED) {
    total = __builtin_amdgcn_readfirstlane(*ga.n_tiles) * tiles_n;
    per_xcd = (total + 7) / 8;
  }
  const int t = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (blockIdx.x / 8 >= per_xcd || t >= total) return;
  int m0, n0, mlim;  // first row, first logical column, rows of the tile in use
  const uint8_t *Wt = static_cast<const uint8_t *>(W);
  if constexpr (GROUPED) {
    const int rt = t / tiles_n;
    const int e = __builtin_amdgcn_readfirstlane(ga.tiles[rt]);
    m0 = __builtin_amdgcn_readfirstlane(ga.tiles[ga.max_tiles + rt]);
    mlim = __builtin_amdgcn_readfirstlane(ga.tiles[2 * ga.max_tiles + rt]);
    n0 = (t - rt * tiles_n) * BG_BN;
    Wt += (size_t)e * N * K * 2;
  } else {
    const int group = 8;
    const int per_group = group * tiles_m;
    const int gidx = t / per_group;
    const int first_n = gidx * group;
    const int gsz = min(group, tiles_n - first_n);
    const int inb = t - gidx * per_group;
    const int tm = inb / gsz;
    n0 = (first_n + inb - tm * gsz) * BG_BN;
    m0 = tm * BG_BM;
    mlim = min(BG_BM, M - m0);
  }
  const int split = blockIdx.y;
  const int kt0 = split * kt_per, kt1 = min(K / BG_BK, kt0 + kt_per);

  constexpr uint32_t WES = W8 ? 1u : 2u;  // bytes per W element
  const int a_nrows = GROUPED ? ga.a_nrows : M;
  const uint32_t a_bytes = (uint32_t)min((size_t)a_nrows * K * 2, (size_t)0x7FFFFFFF);
  const uint32_t w_bytes = (uint32_t)min((size_t)N * K * WES, (size_t)0x7FFFFFFF);
  // Loads.  A half tile is 128 LDS rows: A half h holds rows wm 128 + 64 h +
  // 0..63 of both wave rows, W half h columns wn 64 + 32 h + 0..31 of the four
  // wave columns, so every wave reads each half once per K tile.  Wave w
  // fills LDS rows 16 w .. 16 w + 15 of a half: two instructions of 8 rows x
  // 128 bytes (8-bit W: one of 16 rows x 64 bytes); lane l writes 16-byte
  // position l % 8 (l % 4) of its row with the logical chunk swizzled there.
  // Rows outside the operands point 2 GiB in, past every descriptor's range,
  // so they load zeros.
  uint32_t aoff[2][2], woff[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int i = wave * 16 + j * 8 + (lane >> 3);  // LDS row of the half
      const int row = (i >> 6) * 128 + h * 64 + (i & 63);
      int ar = row < mlim ? m0 + row : -1;
      if constexpr (GROUPED)
        if (ar >= 0 && ga.a_rows) ar = ga.a_rows[ar];
      aoff[h][j] = ar >= 0 && ar < a_nrows ? ((uint32_t)ar * (uint32_t)K + (uint32_t)(bg_swz(i, lane & 7) * 8)) * 2u
                                           : 0x80000000u;
    }
#pragma unroll
    for (int j = 0; j < (W8 ? 1 : 2); ++j) {
      const int i = W8 ? wave * 16 + (lane >> 2) : wave * 16 + j * 8 + (lane >> 3);
      const int wr = w_row_of(n0 + (i >> 5) * 64 + h * 32 + (i & 31), N, epi);
      const int cb = (W8 ? (lane & 3) ^ ((i >> 2) & 3) : bg_swz(i, lane & 7)) * 16;
      woff[h][j] = wr >= 0 ? (uint32_t)wr * (uint32_t)K * WES + (uint32_t)cb : 0x80000000u;
    }
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)bg_lds;
  // half h of K tile kt into the buffer at dst_buf (past the last K tile: an
  // empty range, no traffic)
  auto dma_a = [&](int kt, int h, uint32_t dst_buf) {
    const u32x4_t r = raw_rsrc(A, kt < kt1 ? a_bytes : 0u);
    const uint32_t kb = kt < kt1 ? (uint32_t)kt * (BG_BK * 2u) : 0u;
    const uint32_t dst = lds0 + dst_buf + (uint32_t)(h * BG_HALF_BYTES + wave * 2048);
    dma_lds16(r, aoff[h][0], kb, dst);
    dma_lds16(r, aoff[h][1], kb, dst + 1024);
  };
  auto dma_w = [&](int kt, int h, uint32_t dst_buf) {
    const u32x4_t r = raw_rsrc(Wt, kt < kt1 ? w_bytes : 0u);
    const uint32_t kb = kt < kt1 ? (uint32_t)kt * (BG_BK * WES) : 0u;
    const uint32_t dst =
        lds0 + dst_buf + (uint32_t)(BG_TILE_BYTES + h * BG_HALF_BYTES + wave * (W8 ? 1024 : 2048));
    dma_lds16(r, woff[h][0], kb, dst);
    if constexpr (!W8) dma_lds16(r, woff[h][1], kb, dst + 1024);
  };

  f32x4_t acc[4][8];  // [W block jn][A block im]: rows n, cols m
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Operand reads: LDS row 16 i + lr of a half, for both 32-wide K steps.
  // 8-bit W: a lane takes the 16 codes of chunk lg, so lane group lg holds k
  // = 16 lg + 8 ks .. + 7 in step ks, and A is read in the same order.
  const int lr = lane & 15, lg = lane >> 4;
  const int sw = (lr >> 1) & 7;
  const uint32_t apos = (uint32_t)(lr * 128 + ((W8 ? 2 * lg : lg) ^ sw) * 16);
  const uint32_t wpos = W8 ? (uint32_t)(lr * 64 + (lg ^ ((lr >> 2) & 3)) * 16) : apos;
  constexpr uint32_t KSX = W8 ? 16u : 64u;  // position of step 1 = that of step 0 ^ KSX
  uint32_t abase = (uint32_t)(wm * 64 * 128) + apos;
  uint32_t wbase = (uint32_t)(BG_TILE_BYTES + wn * 32 * (W8 ? 64 : 128)) + wpos;
  u32x4_t ax[4][2], ay[4][2];  // A halves 0 and 1: [16-row block][K step]
  u32x4_t w0[2][2], w1[2][2];  // W halves
  auto read_a = [&](uint32_t base, int h, u32x4_t (&f)[4][2]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        f[i][ks] = *reinterpret_cast<const u32x4_t *>(bg_lds + ((base ^ (ks ? KSX : 0u)) + h * BG_HALF_BYTES + i * 2048));
  };
  auto read_w = [&](uint32_t base, int h, u32x4_t (&f)[2][2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if constexpr (W8) {
        const u32x4_t c = *reinterpret_cast<const u32x4_t *>(bg_lds + (base + h * BG_HALF_BYTES + j * 1024));
        f[j][0] = e4m3x8_to_bf16x8(u32x2_t{c[0], c[1]});
        f[j][1] = e4m3x8_to_bf16x8(u32x2_t{c[2], c[3]});
      } else {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
          f[j][ks] =
              *reinterpret_cast<const u32x4_t *>(bg_lds + ((base ^ (ks ? KSX : 0u)) + h * BG_HALF_BYTES + j * 2048));
      }
    }
  };
  auto products = [&](const u32x4_t (&wf)[2][2], const u32x4_t (&af)[4][2], int hw, int ha) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[hw * 2 + j][ha * 4 + i] = mfma16x16x32(wf[j][ks], af[i][ks], acc[hw * 2 + j][ha * 4 + i]);
    wave_barrier();
  };
  constexpr int NW_ = W8 ? 1 : 2;  // load instructions of a W half (an A half has 2)
  constexpr uint32_t BUF = 2 * BG_TILE_BYTES;
  uint32_t buf = 0;  // LDS buffer of the K tile in use
  dma_a(kt0, 0, 0);
  dma_w(kt0, 0, 0);
  dma_w(kt0, 1, 0);
  dma_a(kt0, 1, 0);
  dma_a(kt0 + 1, 0, BUF);
  dma_w(kt0 + 1, 0, BUF);
  dma_w(kt0 + 1, 1, BUF);
  wait_loads<4 + 3 * NW_>();
  wave_barrier();
  read_a(abase, 0, ax);
  if (wm == 1) wave_barrier();
  for (int kt = kt0; kt < kt1; ++kt) {
    read_w(wbase, 0, w0);
    dma_a(kt + 1, 1, buf ^ BUF);
    wait_loads<6 + 2 * NW_>();
    wave_barrier();
    products(w0, ax, 0, 0);

    read_w(wbase, 1, w1);
    dma_a(kt + 2, 0, buf);
    wait_loads<6 + 2 * NW_>();
    wave_barrier();
    products(w1, ax, 1, 0);

    read_a(abase, 1, ay);
    dma_w(kt + 2, 0, buf);
    wait_loads<4 + 3 * NW_>();
    wave_barrier();
    products(w1, ay, 1, 1);

    abase ^= BUF;
    wbase ^= BUF;
    read_a(abase, 0, ax);
    dma_w(kt + 2, 1, buf);
    wait_loads<4 + 3 * NW_>();
    wave_barrier();
    products(w0, ay, 0, 1);
    buf ^= BUF;
  }
  wait_loads<0>();
  if (wm == 0) wave_barrier();

  // Epilogue: lane holds out[m][n .. n + 3] with m = m0 + wm 128 + 16 im + lr,
  // n = n0 + wn 64 + 16 jn + 4 lg (N and F are multiples of 4, so a group of
  // 4 columns is either wholly inside or wholly outside).  Rows and columns
  // outside are dropped by the buffer range over the tile's rows (columns
  // point 2 GiB in), so there is no branch per store and the residual's
  // loads go out sixteen at a time.
  const int ncols = logical_cols(N, epi);
  const int nl = n0 + wn * 64 + lg * 4;
  const uint32_t row = wm * 128 + lr;  // of the tile, at im = 0
  auto at = [&](int ld, int es, int col, int lim) -> uint32_t {  // byte of (row, col) in a tile of ld columns
    return col < lim ? (row * (uint32_t)ld + (uint32_t)col) * (uint32_t)es : 0x80000000u;
  };
  if constexpr (W8) {  // the rows' scales, before any epilogue or partial
#pragma unroll
    for (int jn = 0; jn < 4; ++jn)
      if (nl + jn * 16 < ncols) {
#pragma unroll
        for (int im = 0; im < 8; ++im) acc[jn][im] = row_scaled(acc[jn][im], wscale, nl + jn * 16, N, epi);
      }
  }
  if (part || (GROUPED && ga.f32_out)) {  // fp32: a split-K partial (logical column space), or the product itself
    float *base = part ? part + ((size_t)split * M + m0) * ncols : reinterpret_cast<float *>(out) + (size_t)m0 * N;
    const buf_rsrc_t ro = make_rsrc(base, mlim * ncols * 4);
#pragma unroll
    for (int jn = 0; jn < 4; ++jn) {
      const uint32_t o = at(ncols, 4, nl + jn * 16, ncols);
#pragma unroll
      for (int im = 0; im < 8; ++im) buf_st_b128(ro, o + (uint32_t)im * 64u * (uint32_t)ncols, acc[jn][im]);
    }
    return;
  }
  if constexpr (epi == EPI_SILU_MUL) {
    // the wave's 64 columns are one [32 gate | 32 up] group: blocks jn and
    // jn + 2 pair up
    const int F = N >> 1;
    const buf_rsrc_t ro = make_rsrc(out + (size_t)m0 * F, mlim * F * 2);
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      const uint32_t o = at(F, 2, ((n0 + wn * 64) >> 1) + jj * 16 + lg * 4, F);
#pragma unroll
      for (int im = 0; im < 8; ++im) {
        const f32x4_t gv = acc[jj][im], uv = acc[jj + 2][im];
        buf_st_b64(ro, o + (uint32_t)im * 32u * (uint32_t)F,
                   u32x2_t{pack_bf16x2(silu_f(gv[0]) * uv[0], silu_f(gv[1]) * uv[1]),
                           pack_bf16x2(silu_f(gv[2]) * uv[2], silu_f(gv[3]) * uv[3])});
        if (im % 2) __builtin_amdgcn_sched_barrier(0);
      }
    }
    return;
  }
  const buf_rsrc_t ro = make_rsrc(out + (size_t)m0 * N, mlim * N * 2);
  uint32_t o[4];
#pragma unroll
  for (int jn = 0; jn < 4; ++jn) o[jn] = at(N, 2, nl + jn * 16, N);
  if constexpr (epi == EPI_RESIDUAL) {
    const buf_rsrc_t rr = make_rsrc(res + (size_t)m0 * N, mlim * N * 2);
#pragma unroll
    for (int j2 = 0; j2 < 4; j2 += 2) {  // (half of them at a time: registers)
      u32x2_t r[2][8];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int im = 0; im < 8; ++im)
          r[j][im] = buf_ld_u32x2<0>(rr, (int)(o[j2 + j] + (uint32_t)im * 32u * (uint32_t)N));
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int im = 0; im < 8; ++im)
          acc[j2 + j][im] +=
              f32x4_t{bf16_lo(r[j][im][0]), bf16_hi(r[j][im][0]), bf16_lo(r[j][im][1]), bf16_hi(r[j][im][1])};
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // (unknown to the compiler from here: it would keep all 32 addresses of the
  // residual's loads in registers for the stores, and spill)
#pragma unroll
  for (int jn = 0; jn < 4; ++jn) asm volatile("" : "+v"(o[jn]));
#pragma unroll
  for (int im = 0; im < 8; ++im) {
#pragma unroll
    for (int jn = 0; jn < 4; ++jn)
      buf_st_b64(ro, o[jn] + (uint32_t)im * 32u * (uint32_t)N,
                 u32x2_t{pack_bf16x2(acc[jn][im][0], acc[jn][im][1]), pack_bf16x2(acc[jn][im][2], acc[jn][im][3])});
    __builtin_amdgcn_sched_barrier(0);
  }
}

// ===========================================================================
// planning and launch
// ===========================================================================
// The split-K sum of a residual GEMM and the RMSNorm of its rows in one
// pass: h = bf16(sum_s part[s] + res) is stored (the splits summed in order,
// as the split-K epilogue does), then out = bf16(h * inv * g) with inv from
// the rounded h.  One block of kFuseThreads per row (a decode batch has few
// rows, so the row's loads are spread over many waves): thread t takes the
// 8-column chunks t, t + kFuseThreads, .. (rows up to kFuseThreads *
// kFuseMaxChunks chunks wide), issues the loads of eight splits before
// adding them, and the sum of squares is reduced across the block.
constexpr int kFuseThreads = 512;
constexpr int kFuseMaxChunks = 2;
__global__ __launch_bounds__(kFuseThreads) void k_splitk_residual_rmsnorm(const float *__restrict__ part, int splits,
                                                                 const uint16_t *__restrict__ res,
                                                                 uint16_t *__restrict__ h,
                                                                 const uint16_t *__restrict__ g,
                                                                 uint16_t *__restrict__ out, int M, int N,
                                                                 float eps) {
  __shared__ float red[kFuseThreads / 64];
  const int row = blockIdx.x;
  const int tid = threadIdx.x;
  const int nch = N >> 3;
  u32x4_t v[kFuseMaxChunks];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < kFuseMaxChunks; ++j) {
    const int c = tid + kFuseThreads * j;
    v[j] = u32x4_t{0u, 0u, 0u, 0u};
    if (c < nch) {
      f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
      const float *pp = part + (size_t)row * N + c * 8;
      const size_t stride = (size_t)M * N;
      for (int s0i = 0; s0i < splits; s0i += 8) {
        f32x4_t a[8], b[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const bool ok = s0i + q < splits;
          a[q] = ok ? *reinterpret_cast<const f32x4_t *>(pp + (s0i + q) * stride) : f32x4_t{0.f, 0.f, 0.f, 0.f};
          b[q] = ok ? *reinterpret_cast<const f32x4_t *>(pp + (s0i + q) * stride + 4) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          s0 += a[q];
          s1 += b[q];
        }
      }
      const u32x4_t r = ld_u32x4(res + (size_t)row * N + c * 8);
      s0[0] += bf16_lo(r[0]);
      s0[1] += bf16_hi(r[0]);
      s0[2] += bf16_lo(r[1]);
      s0[3] += bf16_hi(r[1]);
      s1[0] += bf16_lo(r[2]);
      s1[1] += bf16_hi(r[2]);
      s1[2] += bf16_lo(r[3]);
      s1[3] += bf16_hi(r[3]);
      v[j] = u32x4_t{pack_bf16x2(s0[0], s0[1]), pack_bf16x2(s0[2], s0[3]), pack_bf16x2(s1[0], s1[1]),
                     pack_bf16x2(s1[2], s1[3])};
      st_u32x4(h + (size_t)row * N + c * 8, v[j]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = bf16_lo(v[j][i]), y = bf16_hi(v[j][i]);
        ss += x * x + y * y;
      }
    }
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < kFuseThreads / 64; ++w) tot += red[w];
  const float inv = 1.0f / sqrtf(tot / (float)N + eps);
#pragma unroll
  for (int j = 0; j < kFuseMaxChunks; ++j) {
    const int c = tid + kFuseThreads * j;
    if (c < nch) {
      const u32x4_t gv = ld_u32x4(g + c * 8);
      u32x4_t o;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        o[i] = pack_bf16x2(bf16_lo(v[j][i]) * inv * bf16_lo(gv[i]), bf16_hi(v[j][i]) * inv * bf16_hi(gv[i]));
      st_u32x4(out + (size_t)row * N + c * 8, o);
    }
  }
}

// The split-K sum and epilogue, or with nf (residual epilogue, rows fit) the
// sum fused with the RMSNorm of the result rows (nf->done set).
static hipError_t finish_splitk(const float *part, int splits, uint16_t *out, const uint16_t *res, int M, int N,
                                int epi, NormFuse *nf, hipStream_t st);

static hipError_t launch_splitk_epilogue(const float *part, int splits, uint16_t *out, const uint16_t *res, int M,
                                         int N, int epi, hipStream_t st) {
  const int outc = epi == EPI_SILU_MUL ? N / 2 : N;
  const long total = (long)M * (outc / 2);
  const int blocks = (int)((total + 255) / 256 < 8192 ? (total + 255) / 256 : 8192);
  hipLaunchKernelGGL(k_gemm_splitk_epilogue, dim3(blocks), dim3(256), 0, st, part, splits, out, res, M, N, epi);
  return hipGetLastError();
}

static hipError_t finish_splitk(const float *part, int splits, uint16_t *out, const uint16_t *res, int M, int N,
                                int epi, NormFuse *nf, hipStream_t st) {
  if (nf && nf->gamma && epi == EPI_RESIDUAL && N % 8 == 0 && N / 8 <= kFuseThreads * kFuseMaxChunks) {
    hipLaunchKernelGGL(k_splitk_residual_rmsnorm, dim3(M), dim3(kFuseThreads), 0, st, part, splits, res, out, nf->gamma,
                       nf->out, M, N, nf->eps);
    nf->done = true;
    return hipGetLastError();
  }
  return launch_splitk_epilogue(part, splits, out, res, M, N, epi, st);
}

constexpr int kMaxSplits = 8;
static int stream_splits(int M, int N, int K, int bm) {
  const int tiles = ((N + ST_BN - 1) / ST_BN) * ((M + bm - 1) / bm);
  const int nsteps = (K + 31) / 32;
  // one block per CU (256 CUs).  A grid that covers at least 3/4 of the CUs
  // is not split; otherwise K is split into the count whose rounds of 256
  // blocks take the least time per split (ceil(tiles s / 256) / s; fewer
  // splits on ties), at most 8 (the fp32 partials are written and read back
  // once per split) and each split keeping 4 or more 128-wide K stages
  if (tiles >= 192) return 1;
  int best = 1;
  for (int s = 2; s <= kMaxSplits && nsteps / s >= 16; ++s) {
    const long rs = ((long)tiles * s + 255) / 256, rb = ((long)tiles * best + 255) / 256;
    if (rs * best < rb * s) best = s;  // rs / s < rb / best
  }
  return best;
}

// What a plan takes, in microseconds, less what all plans share: rounds of 256
// blocks (one per CU), each a start and its K stages, or W's way from HBM
// where that is longer, and for a split K the sum's launch and the fp32
// partials written and read.  More rows per block mean fewer bytes of W
// through a CU's LDS, fewer mean more blocks at work and less K to split, and
// which of them decides depends on how the blocks fill their rounds, so the
// plans are compared by these estimates.  Their constants are fitted to every
// choice timed at 65 to 256 rows of 17 products (K 256 to 28672, N 256 to
// 57344, 0.1 MB to 0.9 GB) of both weight types: the plan chosen is within
// 1.3 % (8-bit W 0.6 %) of the fastest of them on average, 20 % at worst (rows
// that are no whole cache lines).  The lines drawn through a few 8B and 70B
// shapes before had 8-bit W on 256 x 256 tiles from 129 rows on (a W of 0.1 MB
// at 200 rows: 20.5 us, now 6; 8B qkv at 255 rows 38, now 26), and as few
// blocks as possible elsewhere (2048 x 2048 at 255 rows 24, now 17; 8208 x
// 1048 at 192 rows 26, now 15; 8B gate/up at 160 rows 60 us then and now).
static float split_us(int splits, int M, int ncols) {
  return splits > 1 ? 4.f + (float)splits * (float)M * (float)ncols * (8.f / 6e6f) : 0.f;
}
static float w_us(int N, int K, bool w8, bool once) {
  return (float)N * (float)K * (w8 ? 1.f : 2.f) / (once ? 5.5e6f : 4.5e6f);
}
static float stream_us(int M, int N, int K, int ncols, bool w8, int bm, int splits) {
  const int mt = (M + bm - 1) / bm, tiles = (ncols + ST_BN - 1) / ST_BN * mt;
  const int rounds = (tiles * splits + 255) / 256;
  const int range = ((K + 31) / 32 + splits - 1) / splits * 32, stages = (range + (w8 ? 127 : 63)) / (w8 ? 128 : 64);
  float stage = w8 ? (bm == 64 ? 0.65f : 1.08f) : bm == 64 ? 0.45f : bm == 128 ? 0.65f : bm == 192 ? 0.83f : 0.97f;
  // a 128-byte run of a row that is no whole number of cache lines touches two
  // of them: more so, the more rows of A a block loads
  if (!w8 && bm > 64 && K % 64) stage *= 1.6f;
  const float blocks = (float)rounds * ((w8 ? 3.2f : 2.f) + (float)stages * stage);
  return std::max(blocks, w_us(N, K, w8, mt == 1)) + split_us(splits, M, ncols);
}
static float big_us(int M, int N, int K, int ncols, bool w8, const GemmPlan &p) {
  const long tiles = (long)((M + BG_BM - 1) / BG_BM) * ((ncols + BG_BN - 1) / BG_BN);
  const float blocks = (float)((tiles * p.splits + 255) / 256) * ((w8 ? 7.f : 4.f) + (float)p.kt_per * (w8 ? 1.3f : 1.5f));
  return std::max(blocks, w_us(N, K, w8, true)) + split_us(p.splits, M, ncols);
}

GemmPlan plan_gemm(int M, int N, int K, int epi, bool w8, size_t max_ws) {
  GemmPlan none{};
  none.splits = 1;
  if (M <= 0 || N <= 0 || K <= 0) return none;  // nothing to plan (kind 0, no workspace)
  const int ncols = logical_cols(N, epi);
  const size_t one = (size_t)M * ncols * sizeof(float);  // the partials of one split
  // the big kernel addresses W through a 32-bit buffer range; A is cut into
  // row chunks that each fit one (launch_gemm)
  // (and a tile's rows of the output through another)
  const bool big_fits = K % BG_BK == 0 && N % 8 == 0 && (size_t)N * K * 2 < ((size_t)1 << 31) &&
                        (size_t)BG_BM * K * 2 < ((size_t)1 << 31) && (size_t)BG_BM * ncols * 4 < ((size_t)1 << 31);
  // the weight-streaming kernels address both operands through 32-bit buffer ranges
  const bool stream_fits = (size_t)N * K * (w8 ? 1 : 2) < ((size_t)1 << 31) && (size_t)M * K * 2 < ((size_t)1 << 31);
  // A W that one XCD's L2 holds costs nothing to read again, and many small
  // blocks have the shorter chain at any number of rows (256 x 256 at 512
  // rows: 21 us in 256 x 256 tiles, 5.6 in blocks of 64 rows)
  const bool small_w = (size_t)N * K * (w8 ? 1 : 2) <= ((size_t)4 << 20);
  // (the tiled kernel, for what the others do not take, reads bf16 weights only)
  const bool stream = stream_fits && (M < BG_BM || small_w || (!big_fits && (M == BG_BM || w8)));
  GemmPlan best = none;
  best.kind = w8 ? -1 : 1;  // -1: no kernel here addresses 8-bit operands this large
  float best_us = 0.f;
  if (big_fits && (M >= BG_BM || (M > 128 && stream))) {
    // one block per CU: split K while the tiles cover at most half the CUs,
    // keeping at least 8 K tiles per split
    const long big_tiles = (long)((M + BG_BM - 1) / BG_BM) * ((ncols + BG_BN - 1) / BG_BN);
    GemmPlan p = none;
    p.kind = 2;
    const int nk = K / BG_BK;
    int splits = 1;
    if (big_tiles <= 128 && (size_t)M * K * 2 < ((size_t)1 << 31)) {
      const long by_cus = 256 / big_tiles, by_k = nk / 8;
      splits = (int)(by_cus < by_k ? by_cus : by_k);
    }
    if (splits < 1) splits = 1;
    // (the scratch's limit binds only where the other kernels are a choice)
    while (stream && splits > 1 && splits * one > max_ws) --splits;
    p.kt_per = (nk + splits - 1) / splits;
    p.splits = (nk + p.kt_per - 1) / p.kt_per;
    p.ws_bytes = p.splits > 1 ? p.splits * one : 0;
    if (!stream) return p;
    best = p;
    best_us = big_us(M, N, K, ncols, w8, p);
  }
  if (!stream) return best;
  // up to 64 rows one block row holds the batch; above, the rows per block
  // (to the batch's own; 8-bit W stops at 128, where its ring is three stages
  // deep) with the least time, each with the splits that there is room for
  for (int bm = 64; bm <= (w8 ? 128 : 256) && (bm == 64 || bm - 64 < M); bm += 64) {
    GemmPlan p = none;
    p.bm = bm;
    p.splits = stream_splits(M, ncols, K, bm);
    while (p.splits > 1 && p.splits * one > max_ws) --p.splits;
    p.ws_bytes = p.splits > 1 ? p.splits * one : 0;
    const float us = stream_us(M, N, K, ncols, w8, bm, p.splits);
    if (best.kind == 1 || best.kind == -1 || us < best_us) {
      best = p;
      best_us = us;
    }
  }
  return best;
}

bool packed_ok(int N, int K, int epi) {
  if (N <= 0 || K <= 0 || N % 16 || K % 32) return false;
  if (epi == EPI_SILU_MUL && (N / 2) % 16) return false;  // gate and up runs must stay 16-aligned
  return (size_t)N * K * 2 < ((size_t)1 << 31);
}

size_t packed_weight_bytes(int N, int K) { return (size_t)N * K * 2; }

hipError_t pack_weight(const uint16_t *W, uint16_t *P, int N, int K, hipStream_t st) {
  if (!W || !P || N <= 0 || K <= 0 || N % 16 || K % 32) return hipErrorInvalidValue;
  const size_t chunks = (size_t)N * K / 8;
  const size_t blocks = (chunks + 255) / 256;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pack_weight, dim3((unsigned)blocks), dim3(256), 0, st, W, P, N, K);
  return hipGetLastError();
}

// One 256 x 256 launch: the kernel of the epilogue and weight type.
template <bool W8, bool GROUPED>
static void launch_big(dim3 grid, hipStream_t st, const uint16_t *A, const void *W, const float *wscale, uint16_t *out,
                       const uint16_t *res, float *part, int M, int N, int K, int epi, int tm, int tn, int per_xcd,
                       int kt_per, const GroupedArgs &ga) {
  auto k = epi == EPI_SILU_MUL               ? k_gemm_big<EPI_SILU_MUL, W8, GROUPED>
           : epi == EPI_RESIDUAL && !GROUPED ? k_gemm_big<GROUPED ? EPI_STORE : EPI_RESIDUAL, W8, GROUPED>
                                             : k_gemm_big<EPI_STORE, W8, GROUPED>;
  hipLaunchKernelGGL(k, grid, dim3(BG_THREADS), 4 * BG_TILE_BYTES, st, A, W, wscale, out, res, part, M, N, K, tm, tn,
                     per_xcd, kt_per, ga);
}

// W by non-temporal loads: with one block row (mt) every byte of W is used
// once and only takes cache from the activations and partials.  70B gate/up
// (940 MB) at one row 157 -> 144 us, 8B gate/up (235 MB) at 64 rows 43.8 ->
// 40.0, of 8-bit codes 29.7 -> 28.0.  To 32 rows for every W larger than one
// XCD's L2; above, where activations and partials weigh more, from 96 MiB (8B
// qkv, 50 MB, at 64 rows 15.6 -> 17.4 with them, 8B down, 117 MB, 31.0 -> 28.8).
// Between the two sizes it depends on what the caches hold: passes over one 8B
// layer, 64 requests, 213 -> 218 us with them; twelve layers in turn 1684 -> 1707,
// with 8-bit W at 37 rows 1294 -> 1271; after a flush that left the caches
// full of written data 251 -> 239.
static bool w_read_once(int mt, int M, int N, int K, bool w8) {
  const size_t bytes = (size_t)N * K * (w8 ? 1 : 2);
  return mt == 1 && bytes > (M <= 32 ? (size_t)4 << 20 : (size_t)96 << 20);
}

template <bool PRENORM>
static hipError_t launch_stream(const uint16_t *A, const void *W, const float *wscale, uint16_t *out,
                                const uint16_t *res, float *part, int M, int N, int K, int epi, int splits, int bm,
                                hipStream_t st, const uint16_t *gamma, float *ssq) {
  const bool w8 = wscale != nullptr;
  const int ncols = logical_cols(N, epi);
  const int nsteps = (K + 31) / 32;
  const int per = (nsteps + splits - 1) / splits;
  const int mt = (M + bm - 1) / bm;
  const int tiles = ((ncols + ST_BN - 1) / ST_BN) * mt;
  const int per_xcd = (tiles + 7) / 8;
  const dim3 grid(8 * per_xcd, splits);
  const bool once = w_read_once(mt, M, N, K, w8);
#define EB_STREAM(BM_, W8_)                                                                                         \
  hipLaunchKernelGGL((once ? k_gemm_stream<BM_, W8_, PRENORM, 0, true> : k_gemm_stream<BM_, W8_, PRENORM>), grid, \
                     dim3(64 * StreamTraits<BM_, W8_, PRENORM>::NW), (StreamTraits<BM_, W8_, PRENORM>::LDS), st, A, W, \
                     wscale, out, res, part, M, N, K, epi, per, tiles, mt, per_xcd, gamma, ssq, GroupedArgs{})
  if (bm == 64) {
    if (w8)
      EB_STREAM(64, true);
    else
      EB_STREAM(64, false);
    return hipGetLastError();
  }
  if constexpr (PRENORM) {
    return hipErrorInvalidValue;
  } else if (w8) {
    EB_STREAM(128, true);
  } else if (bm == 128) {
    EB_STREAM(128, false);
  } else if (bm == 192) {
    EB_STREAM(192, false);
  } else {
    EB_STREAM(256, false);
  }
#undef EB_STREAM
  return hipGetLastError();
}

hipError_t launch_gemm_f32(const uint16_t *A, const uint16_t *W, float *out, int M, int N, int K, hipStream_t st) {
  return launch_stream<false>(A, W, nullptr, nullptr, nullptr, out, M, N, K, (int)EPI_STORE, 1, 64, st, nullptr, nullptr);
}

hipError_t launch_gemm(const GemmPlan &p, const uint16_t *A, const void *W, const float *wscale, uint16_t *out,
                       const uint16_t *res, int M, int N, int K, int epi, void *ws, hipStream_t st, NormFuse *nf,
                       const uint16_t *Wp) {
  if (nf) nf->done = false;
  if (M <= 0) return hipSuccess;
  const bool w8 = wscale != nullptr;
  if (p.kind < 0 || (w8 && p.kind == 1)) return hipErrorInvalidValue;
  const int ncols = logical_cols(N, epi);
  if (p.kind == 0) {
    const int nsteps = (K + 31) / 32;
    const int splits = p.splits;
    const int per = (nsteps + splits - 1) / splits;
    float *part = splits > 1 ? reinterpret_cast<float *>(ws) : nullptr;
    const int mt = (M + SK_BM - 1) / SK_BM;
    const int tiles = ((ncols + SW_BN - 1) / SW_BN) * mt;
    const int per_xcd = (tiles + 7) / 8;
    dim3 grid(8 * per_xcd, splits);
    if (!(Wp && packed_ok(N, K, epi) && M <= kPackedMaxRows)) {
      const hipError_t e =
          launch_stream<false>(A, W, wscale, out, res, part, M, N, K, epi, splits, p.bm, st, nullptr, nullptr);
      if (e != hipSuccess || splits == 1) return e;
      return finish_splitk(part, splits, out, res, M, N, epi, nf, st);
    }
    hipLaunchKernelGGL(k_gemm_skinny_packed<false>, grid, dim3(256), SP_LDS_ONE, st, A, Wp, out, res, part, M, N, K, epi,
                       per, tiles, mt, per_xcd);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || splits == 1) return e;
    return finish_splitk(part, splits, out, res, M, N, epi, nf, st);
  }
  if (p.kind == 2) {
    if (p.splits > 1) {  // one launch (the plan only splits a few tiles), then the partial sums
      const int tm = (M + BG_BM - 1) / BG_BM, tn = (ncols + BG_BN - 1) / BG_BN;
      const int per_xcd = (tm * tn + 7) / 8;
      float *part = reinterpret_cast<float *>(ws);
      auto launch = w8 ? launch_big<true, false> : launch_big<false, false>;
      launch(dim3(8 * per_xcd, p.splits), st, A, W, wscale, out, res, part, M, N, K, epi, tm, tn, per_xcd, p.kt_per,
             GroupedArgs{});
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      return finish_splitk(part, p.splits, out, res, M, N, epi, nf, st);
    }
    // rows per launch: A's slice must stay inside a 32-bit buffer range
    const size_t rows_fit = ((((size_t)1 << 31) - 1) / ((size_t)K * 2)) / BG_BM * BG_BM;
    const int chunk = (int)(rows_fit < (size_t)M ? rows_fit : (size_t)M);
    const size_t out_cols = epi == EPI_SILU_MUL ? (size_t)N / 2 : (size_t)N;
    for (int m0 = 0; m0 < M; m0 += chunk) {
      const int mc = M - m0 < chunk ? M - m0 : chunk;
      const int tm = (mc + BG_BM - 1) / BG_BM, tn = (ncols + BG_BN - 1) / BG_BN;
      const int per_xcd = (tm * tn + 7) / 8;
      auto launch = w8 ? launch_big<true, false> : launch_big<false, false>;
      launch(dim3(8 * per_xcd), st, A + (size_t)m0 * K, W, wscale, out + (size_t)m0 * out_cols,
             res ? res + (size_t)m0 * N : nullptr, nullptr, mc, N, K, epi, tm, tn, per_xcd, K / BG_BK, GroupedArgs{});
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const int tiles_m = (M + TL_BM - 1) / TL_BM, tiles_n = (ncols + TL_BN - 1) / TL_BN;
  hipLaunchKernelGGL(k_gemm_tiled, dim3(tiles_m * tiles_n), dim3(256), 0, st, A,
                     static_cast<const uint16_t *>(W), out, res, M, N, K, epi, tiles_m,
                     tiles_n);
  return hipGetLastError();
}

hipError_t launch_gemm_prenorm(const GemmPlan &p, const uint16_t *x, const uint16_t *gamma, const void *W,
                               const float *wscale, int M, int N, int K, float *part, float *ssq, hipStream_t st,
                               const uint16_t *Wp) {
  if (M <= 0) return hipSuccess;
  if (p.kind != 0 || p.splits < 2) return hipErrorInvalidValue;
  if (!(Wp && packed_ok(N, K, EPI_STORE) && M <= kPackedMaxRows))
    return launch_stream<true>(x, W, wscale, nullptr, nullptr, part, M, N, K, (int)EPI_STORE, p.splits, p.bm, st, gamma,
                               ssq);
  const int nsteps = (K + 31) / 32;
  const int per = (nsteps + p.splits - 1) / p.splits;
  const int mt = (M + SK_BM - 1) / SK_BM;
  const int tiles = ((N + SW_BN - 1) / SW_BN) * mt;
  const int per_xcd = (tiles + 7) / 8;
  hipLaunchKernelGGL((k_gemm_skinny_packed<true>), dim3(8 * per_xcd, p.splits), dim3(256), SP_LDS_ONE, st, x, Wp, nullptr,
                     nullptr, part, M, N, K, (int)EPI_STORE, per, tiles, mt, per_xcd, gamma, ssq);
  return hipGetLastError();
}

hipError_t launch_gemm_grouped_big(const uint16_t *A, int a_nrows, const int32_t *a_rows, const uint16_t *W,
                                   void *out, bool f32_out, const int32_t *tiles, const int32_t *n_tiles, int max_tiles,
                                   int N, int K, int epi, hipStream_t st) {
  if (max_tiles <= 0) return hipSuccess;
  if (K % BG_BK) return hipErrorInvalidValue;
  const int tiles_n = (logical_cols(N, epi) + BG_BN - 1) / BG_BN;
  const GroupedArgs ga{a_rows, tiles, n_tiles, max_tiles, a_nrows, f32_out ? 1 : 0};
  const unsigned grid = ((unsigned)max_tiles * (unsigned)tiles_n + 7) / 8 * 8;
  launch_big<false, true>(dim3(grid), st, A, W, nullptr, static_cast<uint16_t *>(out), nullptr, nullptr, 0, N, K, epi, 0,
                          tiles_n, 0, K / BG_BK, ga);
  return hipGetLastError();
}

hipError_t launch_gemm_grouped(const uint16_t *A, int a_nrows, const int32_t *a_rows, const uint16_t *W, void *out,
                               bool f32_out, const int32_t *tiles, const int32_t *n_tiles, int max_tiles, int N, int K,
                               int epi, bool once, hipStream_t st) {
  if (max_tiles <= 0) return hipSuccess;
  const int nct = (logical_cols(N, epi) + ST_BN - 1) / ST_BN;
  const unsigned grid = ((unsigned)max_tiles * (unsigned)nct + 7) / 8 * 8;
  const GroupedArgs ga{a_rows, tiles, n_tiles, max_tiles, a_nrows, f32_out ? 1 : 0};
  uint16_t *o16 = f32_out ? nullptr : static_cast<uint16_t *>(out);
  float *o32 = f32_out ? static_cast<float *>(out) : nullptr;
  // Eight waves a block where all blocks are on the chip at once, two per CU, and
  // each one's own latency counts (16 experts of 512 over 1024: one token 24.8 ->
  // 23.4 us, 16 tokens 29.3 -> 28.5; 32 experts the same 26.4 -> 25.0, 33.2 -> 32.3);
  // with more, four (16 experts of 2048 over 4096, 64 tokens: 176 against 178).
  const bool wide = grid <= 512;
  auto k = wide ? (once ? k_gemm_stream<64, false, false, 8, true> : k_gemm_stream<64, false, false, 8>)
                : (once ? k_gemm_stream<64, false, false, 4, true> : k_gemm_stream<64, false, false, 4>);
  static_assert(StreamTraits<64, false, false, 8>::LDS == StreamTraits<64, false, false, 4>::LDS, "one LDS size");
  hipLaunchKernelGGL(k, dim3(grid), dim3(wide ? 512 : 256), (StreamTraits<64, false, false, 4>::LDS), st, A, W, nullptr,
                     o16, nullptr, o32, 0, N, K, epi, (K + 31) / 32, 0, nct, 0, nullptr, nullptr, ga);
  return hipGetLastError();
}

}  // namespace eb
