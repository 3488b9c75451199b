// Weight-streaming path of the expert computation for small token counts (Sec. 3.2).
// With only a handful of tokens per cluster the layer is bound by reading every base
// matrix once from HBM, so the two shared-base products are pure streams: a workgroup owns
// 32 weight rows of one cluster and 16 or 32 of its tokens (128 rows and up to 64 tokens: skinny_wide), its four wavefronts split the
// contraction dimension, and both operands travel global -> LDS by DMA into per-wavefront
// rings.  The per-expert rank-r terms (INT4 factors dequantised on the fly, Sec. 3.4) are
// small kernels of their own or ride along in the stream launches.
#include <algorithm>
#include <type_traits>

#include "cmoe_device.h"

namespace {

constexpr int SK_ROWS = 32;   // weight rows per workgroup
constexpr int SK_RB = SK_ROWS / 32;  // 32-row blocks per workgroup
constexpr int SK_OCC = 3;     // workgroups per CU the LDS budget is sized for
constexpr int SK_WAVES = 4;   // wavefronts splitting the contraction

// Weight rows of a workgroup in the form of `cols` tokens (64: skinny_wide)
__host__ __device__ constexpr int stream_rows(int cols) { return cols == 64 ? 128 : SK_ROWS; }
constexpr int SK_A_BYTES = SK_ROWS * 128;           // weight rows x 64 elements
// Ring geometry of one wavefront for COLS token rows per pass (16, or 32 when the caller
// has more than 16 rows per group: all 32 accumulator columns are then distinct).
template <int COLS>
struct SkRing {
  static constexpr int B_BYTES = COLS * 128;            // token rows x 64 elements
  static constexpr int STAGE = SK_A_BYTES + B_BYTES;    // one wavefront stage
  static constexpr int RING = 2 * STAGE;                // two stages per wavefront
  static constexpr int DMA = (SK_ROWS + COLS) / 8;      // 1-KiB loads per stage (8 rows x 128 B each)
  static constexpr int OCC = COLS == 16 ? SK_OCC : 2;   // workgroups per CU that fit the LDS
};

// acc[rb] += sum_k W[row(rb)][k] X[col][k] over the 64-element steps [it0, it1) of this
// wavefront.  Both operands stream global -> LDS one step ahead of the matrix-core work,
// as whole 128-byte lines per row, into a two-stage ring private to the wavefront (so no
// barrier is needed, only vmcnt), chunks XOR-swizzled with (row >> 1) & 7.
//   wrow / brow: the lane's row (lane / 8) of the first 8-row group of the weight / token
//                tile at step 0, WITHOUT the chunk offset (the swizzle depends on the row);
//                w_stride: elements between 8-row groups; brow[i]: the lane's row of token
//                row group i (rows beyond the pass are clamped by the caller)
//   w_blk:       elements between consecutive 32-element contraction blocks of a weight row:
//                32 for row-major rows, rows * 32 for a matrix stored as [K / 32][rows][32]
//                (the re-tiled copy of the bases); a step of 64 elements is two blocks
// With COLS = 16 accumulator columns 16..31 repeat columns 0..15.  NT: weight loads carry the
// non-temporal hint (the token rows never do: they are re-read by every row block).
template <int COLS, bool NT>
__device__ __forceinline__ void skinny_stream(const half_t* wrow, size_t w_stride, size_t w_blk,
                                              const half_t* const (&brow)[COLS / 8], char* ring, unsigned ring_lds,
                                              int lane, int it0, int it1, float16v (&acc)[SK_RB]) {
  using RG = SkRing<COLS>;
  if (it0 >= it1) return;
  const int fr = lane & 31, h = lane >> 5;
  int offa[SK_RB][4], offb[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int rb = 0; rb < SK_RB; ++rb) {
      const int row = rb * 32 + fr;
      offa[rb][s] = row * 128 + (((2 * s + h) ^ ((row >> 1) & 7)) << 4);
    }
    const int br = fr & (COLS - 1);
    offb[s] = SK_A_BYTES + br * 128 + (((2 * s + h) ^ ((br >> 1) & 7)) << 4);
  }
  // lane l of load i fills row 8i + l/8, chunk position l%8, with source chunk position ^ swizzle(row)
  const int lrow = lane >> 3, lpos = lane & 7;
  const int c0 = (lpos ^ (lrow >> 1)) << 3, c1 = (lpos ^ (lrow >> 1) ^ 4) << 3;  // even / odd groups
  // the same chunks of the weight rows: chunk c = block c / 4 of the step, 8 (c % 4) elements into it
  const size_t wc0 = (size_t)(c0 >> 5) * w_blk + (c0 & 31), wc1 = (size_t)(c1 >> 5) * w_blk + (c1 & 31);
  const size_t w_step = 2 * w_blk;
  auto issue = [&](int it, int stage) {
    const unsigned dst = ring_lds + stage * RG::STAGE;
#pragma unroll
    for (int i = 0; i < SK_ROWS / 8; ++i) {
      const half_t* src = wrow + ((i & 1) ? wc1 : wc0) + (size_t)i * w_stride + (size_t)it * w_step;
      if (NT) dma16_nt(src, dst + i * 1024); else dma16(src, dst + i * 1024);
    }
#pragma unroll
    for (int i = 0; i < COLS / 8; ++i)
      dma16(brow[i] + ((i & 1) ? c1 : c0) + (size_t)it * 64, dst + SK_A_BYTES + i * 1024);
  };
  auto compute = [&](int stage) {
    const char* sb = ring + stage * RG::STAGE;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      half8 fa[SK_RB];
#pragma unroll
      for (int rb = 0; rb < SK_RB; ++rb) fa[rb] = *(const half8*)(sb + offa[rb][s]);
      const half8 fb = *(const half8*)(sb + offb[s]);
#pragma unroll
      for (int rb = 0; rb < SK_RB; ++rb) acc[rb] = mfma16(fa[rb], fb, acc[rb]);
    }
    wait_lds();  // the stage has been read: it may be refilled
  };
  issue(it0, 0);
  for (int it = it0; it < it1; it += 2) {
    if (it + 1 < it1) {
      issue(it + 1, 1);
      wait_vm<RG::DMA>();
    } else {
      wait_vm<0>();
    }
    compute(0);
    if (it + 1 < it1) {
      if (it + 2 < it1) {
        issue(it + 2, 0);
        wait_vm<RG::DMA>();
      } else {
        wait_vm<0>();
      }
      compute(1);
    }
  }
}

// Sum of the four wavefronts' partial accumulators through LDS; wavefront w < SK_RB returns
// with block w in hb.  red: [SK_WAVES][SK_RB][16][64] floats.
__device__ __forceinline__ void skinny_reduce(float* red, int wave, int lane, const float16v (&acc)[SK_RB],
                                              float16v& hb) {
#pragma unroll
  for (int rb = 0; rb < SK_RB; ++rb)
#pragma unroll
    for (int v = 0; v < 16; ++v) red[((wave * SK_RB + rb) * 16 + v) * 64 + lane] = acc[rb][v];
  __syncthreads();
  if (wave < SK_RB) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < SK_WAVES; ++w) s += red[((w * SK_RB + wave) * 16 + v) * 64 + lane];
      hb[v] = s;
    }
  }
}

// ---------------------------------------------------------------- more than 32 tokens of a cluster
// acc[a][b] += rows 16 a of this wavefront's 32 x tokens 16 b of the workgroup's up to 64, over the 32-element blocks [b0, b1)
// of the contraction, so that a cluster of up to 64 tokens reads its weights once.  A weight row is read by one
// wavefront only: it goes straight to registers as the matrix-core operand (16 rows x 64 bytes of the re-tiled base are
// 1 KiB of contiguous memory), 16 blocks ahead; the tokens come through LDS, once for the four wavefronts' 128 rows, 256
// elements at a time.  A row's products are one chain of FP32 sums (four shorter ones in skinny_stream): y of 256 tokens of 8
// clusters of 2048 x 8192 against 64 bits 3.8e-4 (4.4e-4 there, whose second stream is not in parts and rounds to FP16 first).
// row_of(i): row of X of token i of the pass; n_tok: tokens of the pass.
constexpr int SW_CH = 8;   // blocks of a chunk of tokens; two chunks of weights in flight
constexpr int SW_CHUNK = SW_CH * 64 * 64, SW_LDS = 2 * SW_CHUNK;
template <bool NT, class RowOf>
__device__ __forceinline__ void skinny_wide(const half_t* const (&wrow)[2], size_t w_step, const half_t* X, int Kc, RowOf row_of,
                                            int n_tok, char* smem, int b0, int b1, float4v (&acc)[2][4]) {
  const int tid = threadIdx.x, lane = tid & 63, t16 = lane & 15, q = lane >> 4;
  if (b0 >= b1) return;   // uniform over the workgroup
  const int chunks = (b1 - b0 + SW_CH - 1) / SW_CH;
  // tokens: a thread takes 64 bytes, block tid % 8 of the chunk, of tokens tid / 8 and, past 32 tokens, tid / 8 + 32
  const int xt = tid >> 3, xb = tid & 7;
  const bool two = n_tok > 32;
  const half_t* xrow[2] = {X + (size_t)row_of(xt) * Kc, X + (size_t)row_of(xt + 32) * Kc};
  char* xdst = smem + xb * 4096 + xt * 64;
  half8 xv[2][4];
  auto load_x = [&](int c) {
    const size_t at = (size_t)min(b0 + c * SW_CH + xb, b1 - 1) * 32;
#pragma unroll
    for (int i = 0; i < 4; ++i) xv[0][i] = *(const half8*)(xrow[0] + at + 8 * i);
    if (two) {
#pragma unroll
      for (int i = 0; i < 4; ++i) xv[1][i] = *(const half8*)(xrow[1] + at + 8 * i);
    }
  };
  auto put_x = [&](int buf) {
#pragma unroll
    for (int r = 0; r < 2; ++r)
      if (r == 0 || two) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *(half8*)(xdst + buf * SW_CHUNK + r * 2048 + ((i ^ swz(xt)) << 4)) = xv[r][i];
      }
  };
  auto load_w = [&](half8 (&w)[2], int c, int i) {
    const size_t at = (size_t)min(b0 + c * SW_CH + i, b1 - 1) * w_step;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const half8* p = (const half8*)(wrow[a] + at);
      w[a] = NT ? __builtin_nontemporal_load(p) : *p;
    }
  };
  half8 w[2][SW_CH][2];
  load_x(0);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < SW_CH; ++i) load_w(w[h][i], h, i);
  put_x(0);
  const int frag = t16 * 64 + ((q ^ swz(t16)) << 4), nb = (n_tok + 15) / 16;
  // Chunk c, from half h of the registers; more: chunk c + 2 follows and takes their place.  (Loads under a condition in one loop
  // for all chunks make the compiler wait for every load before each use: three to four times as slow.)
  auto chunk = [&](int c, auto h_, auto more) {
    constexpr int h = decltype(h_)::value;
    // the chunk's tokens are there; the other buffer has been read
    wait_lds();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (more || c + 1 < chunks) load_x(c + 1);
    const char* sx = smem + h * SW_CHUNK + frag;
#pragma unroll
    for (int i = 0; i < SW_CH; ++i) {
      if (more || b0 + c * SW_CH + i < b1) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if (b < nb) {
            const half8 fb = *(const half8*)(sx + i * 4096 + b * 1024);
#pragma unroll
            for (int a = 0; a < 2; ++a) acc[a][b] = mfma32(w[h][i][a], fb, acc[a][b]);
          }
      }
      if (more) load_w(w[h][i], c + 2, i);
    }
    if (more || c + 1 < chunks) put_x(h ^ 1);
  };
  constexpr std::integral_constant<int, 0> H0{};
  constexpr std::integral_constant<int, 1> H1{};
  int c = 0;
  for (; c + 2 < chunks; c += 2) {   // of an odd number the second loads nothing new, once
    chunk(c, H0, std::true_type{});
    chunk(c + 1, H1, std::true_type{});
  }
  chunk(c, H0, std::false_type{});
  if (c + 1 < chunks) chunk(c + 1, H1, std::false_type{});
}

struct SkinnyTile {
  int c, n0, m0, m_end, s;
};
// Stream workgroup `id` of a launch of nx row blocks x 2^split parts of the contraction (t.s) x slots (row
// block fastest).  A slot is a pass over `cols` tokens of a cluster, m_end the end of the pass; the slots
// are the passes that exist, found from the offsets.
__device__ __forceinline__ bool skinny_tile(const int* offsets, int id, int nx, int split, int G, int cols, int rows,
                                            SkinnyTile& t) {
  int xb = id % nx;
  const int slot = id / nx >> split;
  t.s = id / nx & ((1 << split) - 1);
  // Workgroups are dealt round-robin to the 8 XCDs.  The INT4 factor rows are 128-byte
  // lines shared by 8 neighbouring row blocks, so inside every run of 64 blocks the 8
  // workgroups that land on one XCD take 8 neighbouring row blocks: each line is then
  // fetched into one L2 instead of eight.  (The caller keeps id congruent to the dispatch
  // index modulo 8.)
  if ((nx & 7) == 0 && xb < (nx & ~63)) xb = (xb & ~63) + ((xb & 7) << 3) + ((xb >> 3) & 7);
  t.n0 = xb * rows;
  int hi;
  if (!find_tile(offsets, G, cols, slot, t.c, t.m0, hi)) return false;
  t.m_end = min(hi, t.m0 + cols);
  return t.m0 < hi;
}

// ---------------------------------------------------------------- t1 = V1_e x
// t1[tok][j][:] for token tok and its selected expert j, by the calling workgroup of four wavefronts: a wavefront
// takes ROWS rank rows at a time and U chunks of eight elements a lane, all loads of a step in flight before the first
// is used; INT4 codes dequantised on the fly (Sec. 3.4).
template <int ROWS, int U>
__device__ __forceinline__ void skinny_t1_rows(int tok, int j, const half_t* __restrict__ x,
                                               const int* __restrict__ expert_idx,
                                               const uint8_t* __restrict__ v1_q, const half_t* __restrict__ v1_s,
                                               int d, int q, int r, int k, int x_div, int n_exp,
                                               half_t* __restrict__ t1) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int e = min(max(expert_idx[(size_t)tok * k + j], 0), n_exp - 1);
  const half_t* xr = x + (size_t)(tok / x_div) * d;
  for (int rho0 = wave * ROWS; rho0 < r; rho0 += nw * ROWS) {   // r is a multiple of ROWS
    float acc[ROWS] = {};
    for (int ch0 = lane; ch0 < d / 8; ch0 += 64 * U) {   // 8 elements per chunk: 4 code bytes, one scale
      unsigned bytes[ROWS][U];
      half_t sc[ROWS][U];
      half8 xv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int ch = ch0 + 64 * u;
        const bool in = ch < d / 8;
        xv[u] = in ? *(const half8*)(xr + ch * 8) : half8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
          const size_t row = (size_t)e * r + rho0 + i;
          bytes[i][u] = in ? *(const unsigned*)(v1_q + row * (d / 2) + ch * 4) : 0u;
          sc[i][u] = in ? v1_s[row * (d / q) + (ch * 8) / q] : (half_t)0.f;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < ROWS; ++i) acc[i] = fmaf((float)sc[i][u], code_dot8(bytes[i][u], xv[u]), acc[i]);
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const float sum = wave_sum(acc[i]);
      if (lane == 0) t1[((size_t)tok * k + j) * r + rho0 + i] = (half_t)sum;
    }
  }
}
// Four rows a wavefront from rank 16 on, as many as give all four wavefronts work below, and no more chunks in flight
// than a row of up to 1024 elements has: with four rows and chunks always, half the wavefronts idled at rank 8 and half
// the products were of zeros at width 1024 (expert computation of 256 tokens, four experts of rank 8 each, 4 clusters
// of 1024 x 4096: 49.8 -> 47.0 us, a wavefront per rank row 47.4).
__device__ __forceinline__ void skinny_t1_job(int tok, int j, const half_t* __restrict__ x,
                                              const int* __restrict__ expert_idx,
                                              const uint8_t* __restrict__ v1_q, const half_t* __restrict__ v1_s,
                                              int d, int q, int r, int k, int x_div, int n_exp,
                                              half_t* __restrict__ t1) {
  auto go = [&](auto rows, auto u) {
    skinny_t1_rows<decltype(rows)::value, decltype(u)::value>(tok, j, x, expert_idx, v1_q, v1_s, d, q, r, k, x_div, n_exp,
                                                              t1);
  };
  auto pick = [&](auto u) {
    if (r == 4) go(std::integral_constant<int, 1>{}, u);
    else if (r == 8) go(std::integral_constant<int, 2>{}, u);
    else go(std::integral_constant<int, 4>{}, u);
  };
  if (d <= 1024) pick(std::integral_constant<int, 2>{}); else pick(std::integral_constant<int, 4>{});
}

// ---------------------------------------------------------------- residual-down
// ures[tok][n] = sum_j g_j sum_rho U2_{e_j}[rho][n] s_j[rho] for token tok and a chunk of
// 2048 output columns, s_j summed here from its n_parts partials in fixed order.
__device__ __forceinline__ void skinny_ures_job(int tok, int chunk, const int* __restrict__ expert_idx,
                                                const float* __restrict__ gate,
                                                const uint8_t* __restrict__ u2_q, const half_t* __restrict__ u2_s,
                                                const float* __restrict__ spart, int n_parts, int T, int d, int q,
                                                int r, int k, int n_exp, float* __restrict__ ures) {
  __shared__ float gs[8 * 32];
  __shared__ int es[8];
  const int tid = threadIdx.x;
  const int kr = k * r;
  if (tid < kr) {
    float sum = 0.f;
    for (int part = 0; part < n_parts; ++part) sum += spart[((size_t)part * T + tok) * kr + tid];
    gs[tid] = gate[(size_t)tok * k + tid / r] * sum;
  }
  if (tid < k) es[tid] = min(max(expert_idx[(size_t)tok * k + tid], 0), n_exp - 1);
  __syncthreads();
  const int ch = chunk * 256 + tid;  // 8 output columns
  if (ch >= d / 8) return;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  for (int j = 0; j < k; ++j) {
    const size_t row0 = (size_t)es[j] * r;
    for (int rho0 = 0; rho0 < r; rho0 += 4) {   // r is a multiple of 4: four rows per batch of loads
      unsigned bytes[4];
      float sc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const size_t row = row0 + rho0 + u;
        bytes[u] = *(const unsigned*)(u2_q + row * (d / 2) + ch * 4);
        sc[u] = (float)u2_s[row * (d / q) + (ch * 8) / q] * gs[j * r + rho0 + u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned b = (bytes[u] >> (8 * i)) & 0xffu;
          acc[2 * i] = fmaf(sc[u], nib_lo(b), acc[2 * i]);
          acc[2 * i + 1] = fmaf(sc[u], nib_hi(b), acc[2 * i + 1]);
        }
    }
  }
  float* dst = ures + (size_t)tok * d + ch * 8;
  *(float4v*)dst = float4v{acc[0], acc[1], acc[2], acc[3]};
  *(float4v*)(dst + 4) = float4v{acc[4], acc[5], acc[6], acc[7]};
}

// y[tok] = base[inv_perm[tok]] + ures[tok], base being y_base_sorted, or with SPLIT > 1 the sum of the parts
// of the contraction.
template <int SPLIT>
__global__ __launch_bounds__(256) void skinny_add_kernel(const half_t* __restrict__ yb, const float* __restrict__ parts,
                                                         const float* __restrict__ ures, const int* __restrict__ inv_perm,
                                                         int T, int d, half_t* __restrict__ y) {
  const int tok = blockIdx.x, ch = blockIdx.y * 256 + threadIdx.x;
  if (ch >= d / 4) return;
  const float4v u = *(const float4v*)(ures + (size_t)tok * d + ch * 4);
  const size_t at = (size_t)inv_perm[tok] * d + ch * 4;
  float4v b;
  if (SPLIT == 1) {
    const half4 h = *(const half4*)(yb + at);
#pragma unroll
    for (int i = 0; i < 4; ++i) b[i] = (float)h[i];
  } else {
    float4v v[SPLIT];
#pragma unroll
    for (int s = 0; s < SPLIT; ++s) v[s] = *(const float4v*)(parts + (size_t)s * T * d + at);
    b = v[0];
#pragma unroll
    for (int s = 1; s < SPLIT; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) b[i] += v[s][i];
  }
  half4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = (half_t)(b[i] + u[i]);
  *(half4*)(y + (size_t)tok * d + ch * 4) = o;
}

// Small jobs that ride along with a weight stream as the first workgroups of its grid:
// they are dispatched first, finish within a few microseconds and leave their slots to
// the stream, instead of costing a launch of their own on the critical path.
enum { SIDE_NONE = 0, SIDE_T1 = 1, SIDE_URES = 2 };
struct SideArgs {
  const half_t* x;
  const int* expert_idx;
  const float* gate;
  const uint8_t* fq;     // V1 codes (SIDE_T1) or U2 codes (SIDE_URES)
  const half_t* fs;      // their scales
  const float* spart;
  half_t* t1;
  float* ures;
  int T, d, q, r, k, n_parts, n_jobs;
  int x_div;             // row of x of a token index = index / x_div (>= 1)
  int n_exp;             // G * K: expert slots are clamped to [0, n_exp)
  int n_side;            // workgroups reserved for the jobs (n_jobs rounded up to 8)
};

// The permutation of up to 256 tokens (T <= SKINNY_T, G <= 64), by every workgroup for itself from the cluster
// ids, as in sort_few_kernel.  That kernel takes 4.7 us between two large ones, 1.6 us between small ones; the ballots
// add nothing to a stream of HBM size and 0.5 to 1 us to the smallest (768 x 3072, one token: 4.4 -> 5.2 us).
struct FewSort {
  int wc[4][64], perm[256], off[65];
};
struct FewSortArgs {
  const int* ids;
  int T;
  int *perm, *inv_perm, *offsets;   // written by one workgroup
};
__device__ __forceinline__ void few_sort(const FewSortArgs& a, int G, FewSort& s, bool write) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool in = tid < a.T;
  const int id = in ? min(max(a.ids[tid], 0), G - 1) : 0;
  unsigned long long same = __ballot(in), of_lane = same;   // lanes with this lane's cluster; with cluster `lane`
  for (int b = 0; b < 32 - __builtin_clz(G); ++b) {
    const unsigned long long m = __ballot((id >> b) & 1);
    same &= ((id >> b) & 1) ? m : ~m;
    of_lane &= ((lane >> b) & 1) ? m : ~m;
  }
  s.wc[wave][lane] = lane < G ? __popcll(of_lane) : 0;
  __syncthreads();
  int total = 0, before = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int v = s.wc[w][lane];
    total += v;
    before += w < wave ? v : 0;
  }
  const int first = wave_inclusive_sum(total) - total;
  const int row = __shfl(first + before, id, 64) + __popcll(same & ((1ull << lane) - 1ull));
  if (wave == 0 && lane < G) s.off[lane] = first;
  if (tid == 0) s.off[G] = a.T;
  if (in) s.perm[row] = tid;
  if (write) {
    if (wave == 0 && lane < G) a.offsets[lane] = first;
    if (tid == 0) a.offsets[G] = a.T;
    if (in) {
      a.perm[row] = tid;
      a.inv_perm[tid] = row;
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------- shared-base products
// out[p][n] = sum_k W[c][n][k] X[row(p)][k] for the sorted rows p of cluster c (the product
// the experts of a cluster share, Sec. 3.2): up-projection with W = W1_base, X = x gathered
// through perm, out = Hb; down-projection with W = W2_base, X = A, out = y_base_sorted.
// N: rows of W per cluster, Kc: contraction length, gather: row index of X per sorted row
// or NULL for the identity.  w_blk = 0: W[c] is row-major [N][Kc]; otherwise W[c] is stored
// as [Kc / 32][N][32] and w_blk = N * 32 (the re-tiled copy of the bases): an 8-row load is
// then two contiguous 256-byte pieces instead of eight 128-byte pieces a row apart.
// SORT: the permutation is made here (few_sort) and gathers through it.
template <int SIDE, int COLS, bool NT, bool SORT>
__global__ __launch_bounds__(256, (COLS == 64 ? 2 : SkRing<COLS>::OCC)) void skinny_base_kernel(
    const half_t* __restrict__ X, const int* __restrict__ gather, const half_t* __restrict__ W,
    const int* __restrict__ offsets, int N, int Kc, half_t* __restrict__ out, float* __restrict__ parts, int split,
    int T, int nx, int G, long w_blk, SideArgs sa, FewSortArgs fs) {
  // The jobs for t1 before the stream's workgroups, those for ures after them: 203 tokens of 8 clusters of
  // 2048 x 8192, down-projection 65.4 us with them before, 62 after, 65 to 70 in between; up-projection 64 before and in
  // between, 63 after, but 153 instead of 138 us for 64 tokens of 8 of 4096 x 14336.
  const int first = SIDE == SIDE_T1 ? sa.n_side : 0, job = (int)blockIdx.x - (SIDE == SIDE_T1 ? 0 : (int)gridDim.x - sa.n_side);
  const int id = (int)blockIdx.x - first;
  if (SIDE == SIDE_T1 ? id < 0 : SIDE == SIDE_URES && job >= 0) {
    if (job >= sa.n_jobs) return;
    if (SIDE == SIDE_T1) {
      skinny_t1_job(job / sa.k, job % sa.k, sa.x, sa.expert_idx, sa.fq, sa.fs, sa.d, sa.q, sa.r, sa.k, sa.x_div, sa.n_exp,
                    sa.t1);
    } else {
      const int nch = (sa.d + 2047) / 2048;
      skinny_ures_job(job / nch, job % nch, sa.expert_idx, sa.gate, sa.fq, sa.fs, sa.spart, sa.n_parts, sa.T, sa.d, sa.q,
                      sa.r, sa.k, sa.n_exp, sa.ures);
    }
    return;
  }
  __shared__ FewSort order[1];
  if (SORT) few_sort(fs, G, order[0], id == 0);
  constexpr int RED_BYTES = SK_WAVES * SK_RB * 16 * 64 * 4;
  using RG = SkRing<COLS == 64 ? 16 : COLS>;
  constexpr int RINGS = SK_WAVES * RG::RING;
  __shared__ __attribute__((aligned(1024))) char smem[COLS == 64 ? SW_LDS : RED_BYTES > RINGS ? RED_BYTES : RINGS];
  SkinnyTile t;
  if (!skinny_tile(SORT ? order[0].off : offsets, id, nx, split, G, COLS, stream_rows(COLS), t)) return;
  if constexpr (COLS == 64) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t16 = lane & 15, q = lane >> 4;
    const half_t* wrow[2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
      wrow[a] = W + (size_t)t.c * N * Kc + (size_t)min(t.n0 + wave * 32 + a * 16 + t16, N - 1) * (w_blk ? 32 : Kc) + 8 * q;
    float4v acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = float4v{0.f, 0.f, 0.f, 0.f};
    const int blocks = Kc / 32;
    skinny_wide<NT>(wrow, w_blk ? (size_t)w_blk : 32, X, Kc,
                    [&](int i) {
                      const int p = min(t.m0 + i, t.m_end - 1);
                      return SORT ? order[0].perm[p] / sa.x_div : gather != nullptr ? gather[p] / sa.x_div : p;
                    },
                    t.m_end - t.m0, smem, t.s * blocks >> split, (t.s + 1) * blocks >> split, acc);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int p = t.m0 + b * 16 + t16;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int n = t.n0 + wave * 32 + a * 16 + 4 * q;
        if (p >= t.m_end || n >= N) continue;
        const size_t at = (size_t)p * N + n;
        if (parts != nullptr)
          *(float4v*)(parts + (size_t)t.s * T * N + at) = acc[a][b];
        else
          *(half4*)(out + at) = half4{(half_t)acc[a][b][0], (half_t)acc[a][b][1], (half_t)acc[a][b][2], (half_t)acc[a][b][3]};
      }
    }
  } else {
    float* red = (float*)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, fr = lane & 31, h = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const unsigned smem_lds = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
    const int lrow = lane >> 3;
    const size_t w_ld = w_blk ? 32 : Kc;   // elements between consecutive weight rows
    const half_t* wrow = W + (size_t)t.c * N * Kc + (size_t)(t.n0 + lrow) * w_ld;
    const int p = t.m0 + fr;
    const half_t* brow[COLS / 8];
#pragma unroll
    for (int i = 0; i < COLS / 8; ++i) {
      int r = min(t.m0 + 8 * i + lrow, t.m_end - 1);
      if (SORT) r = order[0].perm[r] / sa.x_div;
      else if (gather != nullptr) r = gather[r] / sa.x_div;
      brow[i] = X + (size_t)r * Kc;
    }
    float16v acc[SK_RB];
#pragma unroll
    for (int rb = 0; rb < SK_RB; ++rb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[rb][v] = 0.f;
    static_assert(SK_WAVES == 4, "shares of the contraction");
    const int iters = Kc / 64, share = t.s * SK_WAVES + wv;
    skinny_stream<COLS, NT>(wrow, 8 * w_ld, w_blk ? (size_t)w_blk : 32, brow, smem + wv * RG::RING,
                            smem_lds + wv * RG::RING, lane, share * iters >> (2 + split), (share + 1) * iters >> (2 + split), acc);
    __syncthreads();  // every ring has been consumed: its space becomes red
    float16v hb;
    skinny_reduce(red, wave, lane, acc, hb);
    if (wave < SK_RB && fr < COLS && p < t.m_end) {
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const size_t at = (size_t)p * N + t.n0 + wave * 32 + 8 * qd + 4 * h;
        if (parts != nullptr)
          *(float4v*)(parts + (size_t)t.s * T * N + at) = float4v{hb[4 * qd], hb[4 * qd + 1], hb[4 * qd + 2], hb[4 * qd + 3]};
        else
          *(half4*)(out + at) = to_half4(hb, qd);
      }
    }
  }
}

// ---------------------------------------------------------------- residual-up, GELU, gated sum, V2 product
// In place on A (which holds Hb on entry), for sorted row p and a chunk of RU_CH columns:
//   A[p][n] = sum_j g_j GELU(Hb[p][n] + sum_rho U1_{e_j}[rho][n] t1_j[rho])       (Sec. 3.2)
//   spart[chunk][row][j][rho] = sum_{n in chunk} V2_{e_j}[rho][n] GELU(...)_j[n]
// with the INT4 factors dequantised on the fly (Sec. 3.4).  A workgroup takes sorted row p = blockIdx.x and its
// token perm[p], row = p; or, with inv_perm given, token blockIdx.x, p = inv_perm of it, row = the
// token, so that the loads by token do not wait for p.  t1 is in token order.  A thread owns 8 consecutive
// columns (one 32-bit word of codes per rank row); the k*r partial dot products of a thread
// are summed over the wavefront by a halving exchange, then over the 4 wavefronts in fixed order.
// Bound by vector instructions (three quarters of the time they issue): 203 tokens, two experts of rank 16, 8192
// columns 20.0 us with an exchange of always 64 values through LDS, in registers of which two workgroups
// fit a CU; 16.8 us with 32 values, register swaps and four workgroups.
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
// The 8 INT4 codes c_0..c_7 of one 32-bit word as f16 pairs WITHOUT their offsets removed.
// Flipping bit 3 of every nibble turns a two's-complement code c into c + 8 in [0, 16); a
// nibble masked in place into the mantissa of 1024.0 then reads 1024 + (c + 8) at mantissa
// bit 0 and 1024 + 16 (c + 8) at mantissa bit 4:
//   o[0] = 1032 + (c_0, c_4)        o[1] = 16 (72 + (c_1, c_5))
//   o[2] = 1032 + (c_2, c_6)        o[3] = 16 (72 + (c_3, c_7))
// The users fold the factor 16 into the other operand and subtract the offsets once per
// sum (FP32 accumulation keeps that exact enough: the offsets are < 2^11 times the terms).
constexpr float DQ_OFF_EVEN = 1032.f, DQ_OFF_ODD = 72.f;
__device__ __forceinline__ unsigned and_or(unsigned a, unsigned mask, unsigned bits) {
  unsigned r;
  asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(mask), "v"(bits));
  return r;
}
__device__ __forceinline__ void decode8_raw(unsigned w, half2v (&o)[4]) {
  const unsigned magic = 0x64006400u;
  w ^= 0x88888888u;
  const unsigned w8 = w >> 8;
  o[0] = __builtin_bit_cast(half2v, and_or(w, 0x000f000fu, magic));
  o[1] = __builtin_bit_cast(half2v, and_or(w, 0x00f000f0u, magic));
  o[2] = __builtin_bit_cast(half2v, and_or(w8, 0x000f000fu, magic));
  o[3] = __builtin_bit_cast(half2v, and_or(w8, 0x00f000f0u, magic));
}

// The same with the offsets removed exactly (f16 subtraction of representable values):
// o[0] = (c_0, c_4), o[1] = 16 (c_1, c_5), o[2] = (c_2, c_6), o[3] = 16 (c_3, c_7).
__device__ __forceinline__ void decode8_x16(unsigned w, half2v (&o)[4]) {
  decode8_raw(w, o);
  const half2v even = {(_Float16)1032.f, (_Float16)1032.f}, odd = {(_Float16)1152.f, (_Float16)1152.f};
  o[0] -= even;
  o[1] -= odd;
  o[2] -= even;
  o[3] -= odd;
}

constexpr int RU_N = 8;
constexpr int RU_CH = RU_N * 256;
static_assert(RU_CH == SKINNY_SN, "s partial chunk");

// One step of the halving exchange: N values a lane, lanes OFF apart.  Across halves and rows of the wavefront
// one swap instruction moves both values of a pair.
template <int OFF, int N, int NV>
__device__ __forceinline__ void halving_step(float (&v)[NV], int lane) {
  if constexpr (N == 1) {
    v[0] += __shfl_xor(v[0], OFF, 64);
  } else {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      if constexpr (OFF >= 16) {
        const unsigned a = __float_as_uint(v[i]), b = __float_as_uint(v[i + N / 2]);
        const auto sw = OFF == 32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false)
                                  : __builtin_amdgcn_permlane16_swap(a, b, false, false);
        v[i] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
      } else {
        const bool up = (lane & OFF) != 0;
        const float keep = up ? v[i + N / 2] : v[i];
        const float send = up ? v[i] : v[i + N / 2];
        v[i] = keep + __shfl_xor(send, OFF, 64);
      }
    }
  }
}
// v[0] of lane l becomes the wavefront's sum of value l / (64 / NV).
template <int NV>
__device__ __forceinline__ void halving_sum(float (&v)[NV], int lane) {
  constexpr auto left = [](int steps) { return (NV >> steps) > 1 ? NV >> steps : 1; };
  halving_step<32, left(0)>(v, lane);
  halving_step<16, left(1)>(v, lane);
  halving_step<8, left(2)>(v, lane);
  halving_step<4, left(3)>(v, lane);
  halving_step<2, left(4)>(v, lane);
  halving_step<1, left(5)>(v, lane);
}

// EPG experts at a time (k rounded up to a power of two, at most 64 values in all)
template <int R, int EPG>
__global__ __launch_bounds__(256) void skinny_resid_up_kernel(
    half_t* __restrict__ A, const half_t* __restrict__ t1, const int* __restrict__ perm,
    const int* __restrict__ inv_perm, const int* __restrict__ expert_idx, const float* __restrict__ gate, const uint8_t* __restrict__ u1_q,
    const half_t* __restrict__ u1_s, const uint8_t* __restrict__ v2_q, const half_t* __restrict__ v2_s, int T,
    int d_ff, int k, int q, int n_exp, float* __restrict__ spart) {
  constexpr int NV = EPG * R;    // (expert, rank row) values of a group
  __shared__ int srow[8];        // first factor row e_j R of selected expert j
  __shared__ float st1[256];     // t1_j[rho]
  __shared__ float sg[8];
  __shared__ float red[4][64];
  const int row = blockIdx.x, chunk = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kr = k * R;
  const int tok = inv_perm != nullptr ? row : perm[row], p = inv_perm != nullptr ? inv_perm[row] : row;
  if (tid < kr) st1[tid] = (float)t1[(size_t)tok * kr + tid];
  if (tid < k) {
    srow[tid] = min(max(expert_idx[(size_t)tok * k + tid], 0), n_exp - 1) * R;
    sg[tid] = gate[(size_t)tok * k + tid];
  }
  const int n = chunk * RU_CH + tid * RU_N;
  const bool in = n < d_ff;
  const size_t qrow = (size_t)(d_ff / 2), srw = (size_t)(d_ff / q);
  float hbv[8], av[8];
  {
    half8 h8 = {0, 0, 0, 0, 0, 0, 0, 0};
    if (in) h8 = *(const half8*)(A + (size_t)p * d_ff + n);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      hbv[i] = (float)h8[i];
      av[i] = 0.f;
    }
  }
  __syncthreads();
  for (int j0 = 0; j0 < k; j0 += EPG) {
    float part[NV];
#pragma unroll
    for (int jj = 0; jj < EPG; ++jj) {
      const int j = j0 + jj;
#pragma unroll
      for (int rho = 0; rho < R; ++rho) part[jj * R + rho] = 0.f;
      if (in && j < k) {
        // the expert's rows are uniform over the workgroup: scalar row bases, one 32-bit
        // lane offset; every code word and scale is requested before the first is used
        const size_t row0 = (size_t)__builtin_amdgcn_readfirstlane(srow[j]);
        const uint8_t* ub = u1_q + row0 * qrow;
        const uint8_t* vb = v2_q + row0 * qrow;
        const half_t* usb = u1_s + row0 * srw;
        const half_t* vsb = v2_s + row0 * srw;
        const unsigned qoff = (unsigned)n / 2, soff = (unsigned)n / (unsigned)q;
        unsigned uw[R], vw[R];
        half_t us[R], vs[R];
#pragma unroll
        for (int rho = 0; rho < R; ++rho) {
          uw[rho] = *(const unsigned*)(ub + rho * qrow + qoff);
          us[rho] = usb[rho * srw + soff];
        }
#pragma unroll
        for (int rho = 0; rho < R; ++rho) {
          vw[rho] = *(const unsigned*)(vb + rho * qrow + qoff);
          vs[rho] = vsb[rho * srw + soff];
        }
        float hj[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) hj[i] = hbv[i];
        float ssum = 0.f;
#pragma unroll
        for (int rho = 0; rho < R; ++rho) {
          const float sc = (float)us[rho] * st1[j * R + rho], sc16 = sc * 0.0625f;
          ssum += sc;
          half2v c[4];
          decode8_raw(uw[rho], c);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float m = (i & 1) ? sc16 : sc;
            hj[i] = fmaf((float)c[i][0], m, hj[i]);
            hj[i + 4] = fmaf((float)c[i][1], m, hj[i + 4]);
          }
        }
        const float g = sg[j];
        half2v g2[4];   // GELU values as f16 pairs (element i, element i + 4), odd i scaled by 1/16
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float off = (i & 1) ? DQ_OFF_ODD : DQ_OFF_EVEN;
          const float lo = gelu_erf(fmaf(-off, ssum, hj[i])), hi = gelu_erf(fmaf(-off, ssum, hj[i + 4]));
          av[i] = fmaf(g, lo, av[i]);
          av[i + 4] = fmaf(g, hi, av[i + 4]);
          const half2v gg = half2v{(_Float16)lo, (_Float16)hi};
          g2[i] = (i & 1) ? gg * half2v{(_Float16)0.0625f, (_Float16)0.0625f} : gg;
        }
        // the two-element dot product instruction is fed exact codes: its accumulation is
        // not a correctly rounded FP32 chain, so large offsets must not pass through it
#pragma unroll
        for (int rho = 0; rho < R; ++rho) {
          half2v c[4];
          decode8_x16(vw[rho], c);
          float dot = 0.f;
#pragma unroll
          for (int i = 0; i < 4; ++i) dot = __builtin_amdgcn_fdot2(c[i], g2[i], dot, false);
          part[jj * R + rho] = (float)vs[rho] * dot;
        }
      }
    }
    halving_sum<NV>(part, lane);
    if (lane % (64 / NV) == 0) red[wave][lane / (64 / NV)] = part[0];
    __syncthreads();
    if (wave == 0 && lane < NV && j0 * R + lane < kr)
      spart[((size_t)chunk * T + row) * kr + j0 * R + lane] =
          ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    __syncthreads();
  }
  if (in) {
    half8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (half_t)av[i];
    *(half8*)(A + (size_t)p * d_ff + n) = o;
  }
}

// ---------------------------------------------------------------- residual-down + un-permute
// y[t] = y_base_sorted[inv_perm[t]] + sum_j g_j U2_{e_j} s_j with U2 dequantised on the
// fly: one workgroup per token, a thread per 8 output columns.
__global__ __launch_bounds__(256) void skinny_combine_kernel(const half_t* __restrict__ yb,
                                                             const float* __restrict__ s_down,
                                                             const int* __restrict__ inv_perm,
                                                             const int* __restrict__ expert_idx,
                                                             const float* __restrict__ gate,
                                                             const uint8_t* __restrict__ u2_q,
                                                             const half_t* __restrict__ u2_s, int d, int q, int r,
                                                             int k, int n_exp, half_t* __restrict__ y) {
  __shared__ float gs[8 * 32];
  __shared__ int es[8];
  const int t = blockIdx.x, tid = threadIdx.x;
  if (tid < k * r) gs[tid] = gate[(size_t)t * k + tid / r] * s_down[(size_t)t * k * r + tid];
  if (tid < k) es[tid] = min(max(expert_idx[(size_t)t * k + tid], 0), n_exp - 1);
  __syncthreads();
  const int ch = blockIdx.y * 256 + tid;  // 8 output columns
  if (ch >= d / 8) return;
  const half8 b8 = *(const half8*)(yb + (size_t)inv_perm[t] * d + ch * 8);
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = (float)b8[i];
  for (int j = 0; j < k; ++j) {
    const size_t row0 = (size_t)es[j] * r;
    for (int rho0 = 0; rho0 < r; rho0 += 4) {   // r is a multiple of 4: four rows per batch of loads
      unsigned bytes[4];
      float sc[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const size_t row = row0 + rho0 + u;
        bytes[u] = *(const unsigned*)(u2_q + row * (d / 2) + ch * 4);
        sc[u] = (float)u2_s[row * (d / q) + (ch * 8) / q] * gs[j * r + rho0 + u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned b = (bytes[u] >> (8 * i)) & 0xffu;
          acc[2 * i] = fmaf(sc[u], nib_lo(b), acc[2 * i]);
          acc[2 * i + 1] = fmaf(sc[u], nib_hi(b), acc[2 * i + 1]);
        }
    }
  }
  half8 o;
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] = (half_t)acc[i];
  *(half8*)(y + (size_t)t * d + ch * 8) = o;
}

}  // namespace

// Base matrices larger than this are streamed with the non-temporal hint: they cannot stay in
// the last-level cache (256 MB) from one call to the next anyway, and keeping them out of it
// leaves the routers, the tokens and the factors there.  Smaller layers are left cacheable.
static bool stream_once(const cmoe_dims& dm) {
  return (size_t)dm.G * dm.d * dm.d_ff * sizeof(half_t) > ((size_t)96 << 20);
}

// Parts of the contraction of the down-projection, as a power of two.  A launch that leaves CUs idle lasts as long as a wavefront's
// chain of steps; parts shorten the chain, until the launch has 192 workgroups (256 where the base comes from HBM
// and the loads take longer), two steps a wavefront are left or the parts no longer fit the space of the factor
// panels, which this path does not use.  Down-projection of 1, 2 and 4 parts, one token: 768 x 3072 6.7, 5.8 and
// 4.6 us, of 8 clusters of 2048 x 8192 16.9, 11.6 and 9.2 us; one part and two: two tokens there (128 workgroups) 18.9
// and 14.7 us, one of 4096 x 14336 30 and 21 us, but 8 tokens of 4 clusters of 1024 x 4096 (128) 9.5 and 10.7 us.
// The form of 64 tokens has a quarter of the row blocks and is cut up to 1024 workgroups: 256 tokens of 8 clusters of 4096 x 14336
// whole and in two parts (704) 163 and 161 us, of 2048 x 8192 in two and in four (768) 57.8 and 58.2.
inline int down_split(const cmoe_dims& dm, int T, int cols) {
  const int slots = T < dm.G + T / cols ? T : dm.G + T / cols, most = cols == 64 ? 1024 : stream_once(dm) ? 256 : 192;
  const int nx = (dm.d + stream_rows(cols) - 1) / stream_rows(cols);
  const size_t room = sizeof(half_t) * 2 * dm.G * dm.KRp * ((size_t)dm.d + dm.d_ff);
  int split = 2;
  while (split > 0 && ((nx * slots << split) > most || dm.d_ff / 64 < 2 * SK_WAVES << split ||
                       sizeof(float) * (T * (size_t)dm.d << split) > room))
    --split;
  return split;
}

// Tokens of a cluster that a workgroup of a weight stream takes: 16, 32 or 64; 32 (two workgroups per CU
// instead of three) where the second reading of a matrix by the passes of a cluster costs more.
//   - Up to 16 tokens no cluster has a second pass.
//   - A matrix that the caches keep is not read twice from memory, and while the workgroups of the
//     16-token form are at most four per CU the passes of a cluster run side by side.  Whole forward
//     of the 32-token and the 16-token form: one cluster of 768 x 3072, 32 tokens 27.9 and 27.1 us;
//     one of 2048 x 8192, 32 tokens 48.5 and 46.7 us, 128 tokens (2304 workgroups) 61 and 69 us; four of
//     1024 x 4096, 50 tokens 41.9 and 40.0 us, 128 tokens (1536 workgroups) 43.8 and 47 us.
//   - Else the expected load of a cluster decides, above 12 tokens for the down-projection and above 13
//     for the up-projection, whose launch also holds a workgroup per token and expert: 8 clusters of
//     4096 x 14336, 104 tokens: both 32-token 345 us, the down-projection alone 338, neither 339;
//     112 tokens: 352, 381, 410; of 2048 x 8192, 97 tokens: 126.7, 126.1, 134.
// And 64 (skinny_wide) for a matrix that the caches do not keep:
//   - Where some cluster is likely to hold more than 32 tokens, so that its second pass would read the matrix again: above 28
//     tokens a cluster on average (a single cluster: above 32), while the launch keeps most CUs busy.  32- and 64-token form,
//     down-projection of 8 clusters of 2048 x 8192: 256 tokens 81.9 and 57.0 us, 203 with a cluster of 37 64.3 and 57.1, with
//     none above 32 54.7 and 57.1; of 4096 x 14336: 230 186 and 159, 130 (at most 27) 145 and 155; one of 4096 x 14336: 70
//     69.8 and 46.4, 64 (128 workgroups) 40.3 and 42.6, 20 23.5 and 29.5; one of 2048 x 32768: 100 (128) 84.1 and 84.1, 150
//     (192) 145 and 86.  Up-projection: one of 8192 x 8192, 60 (64 workgroups) 52.7 and 84.9, 100 (128) 95.6 and 85.6; of
//     4096 x 14336, 64 (112) 50.0 and 47.7.
//   - In the up-projection from 18 tokens a cluster on: in the form of 32 rows the tokens that a workgroup reads from the caches are
//     as many bytes as its weights, here a quarter.  8 clusters of 2048 x 8192: 140 tokens 55.3 and 51.1 us, 165 54.7 and 50.9;
//     of 12: 256 80.5 and 72.6; 4 of 4096 x 14336: 64 79.7 and 77.3; 2: 30 43.4 and 40.5; 3 of 3072 x 8192 (192 workgroups) 58 33.2
//     and 30.5.  Not where that leaves CUs idle, in the first round of workgroups or in the second: 1 of 4096 x 14336 (112), 20 25.9
//     and 32.4; 2 of 4096 x 8192 (128), 40 31.1 and 32.8; 3 of 4096 x 14336 (336) 58 63.8 and 69.4; 5 of 2048 x 8192 (320) 95
//     37.3 and 39.5; but 6 (384) 115 42.6 and 39.9.
static bool stream_wide(const cmoe_dims& dm, int T, bool down) {
  if (!stream_once(dm)) return false;
  const int N = down ? dm.d : dm.d_ff;
  const long row_blocks = (N + stream_rows(64) - 1) / stream_rows(64), once = row_blocks * dm.G;   // workgroups of a pass per cluster
  if (T > 28 * dm.G && T > 32) {
    const long least = row_blocks * std::max(dm.G, (T + 63) / 64);
    return down ? least << down_split(dm, T, 64) >= 192 : least >= 112;
  }
  return !down && T > 18 * dm.G && ((once >= 192 && once <= 256) || once >= 384);
}
int stream_cols(const cmoe_dims& dm, int T, bool down) {
  if (T <= 16 || T <= (down ? 12 : 13) * dm.G) return 16;
  if (stream_wide(dm, T, down)) return 64;
  const long narrow = (long)(dm.d_ff / SK_ROWS) * (dm.G + T / 16);   // workgroups, at most
  return !stream_once(dm) && narrow <= 1024 ? 16 : 32;
}

// One weight stream of the layer.
template <int SIDE, bool SORT>
hipError_t launch_stream(const cmoe_dims& dm, int cols, const half_t* X, const int* gather, const half_t* W,
                         const int* offsets, int N, int Kc, half_t* out, float* parts, int split, int T, long w_blk,
                         const SideArgs& sa, const FewSortArgs& fs, hipStream_t st) {
  const int nx = (N + stream_rows(cols) - 1) / stream_rows(cols);
  const int slots = T < dm.G + T / cols ? T : dm.G + T / cols;   // at most: a slot holds a token, all but G of them `cols`
  const dim3 grid(((unsigned)nx * slots << split) + sa.n_side), block(256);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, 0, st, X, gather, W, offsets, N, Kc, out, parts, split, T, nx, dm.G, w_blk, sa, fs);
  };
  if (cols == 64) {
    go(skinny_base_kernel<SIDE, 64, true, SORT>);   // bases that the caches do not keep
  } else if (cols == 32) {
    if (stream_once(dm)) go(skinny_base_kernel<SIDE, 32, true, SORT>); else go(skinny_base_kernel<SIDE, 32, false, SORT>);
  } else {
    if (stream_once(dm)) go(skinny_base_kernel<SIDE, 16, true, SORT>); else go(skinny_base_kernel<SIDE, 16, false, SORT>);
  }
  return hipGetLastError();
}

// Hb = W1_base(c) x for every sorted row; with t1 != NULL the t1 = V1 x jobs ride along.  cluster_id != NULL: the
// permutation (perm, inv_perm, offsets) is made in the same launch.
hipError_t launch_skinny_hb(const cmoe_dims& dm, const cmoe_weights& w, const half_t* x, int x_div, int T,
                            const int* cluster_id, int* perm, int* inv_perm, int* offsets, const int* expert_idx,
                            half_t* t1, half_t* hb, hipStream_t st) {
  SideArgs sa{};
  sa.x_div = x_div > 1 ? x_div : 1;
  // the re-tiled copy of W1 when the caller keeps one, else the canonical array
  const half_t* w1 = w.packed ? (const half_t*)((const char*)w.packed + cmoe_packed(dm).w1) : (const half_t*)w.w1_base;
  const long w_blk = w.packed ? (long)dm.d_ff * 32 : 0;
  const int cols = stream_cols(dm, T, false);
  const FewSortArgs fs{cluster_id, T, perm, inv_perm, offsets};
  auto go = [&](auto side) {
    constexpr int SIDE = decltype(side)::value;
    if (cluster_id != nullptr)
      return launch_stream<SIDE, true>(dm, cols, x, perm, w1, offsets, dm.d_ff, dm.d, hb, nullptr, 0, T, w_blk, sa, fs, st);
    return launch_stream<SIDE, false>(dm, cols, x, perm, w1, offsets, dm.d_ff, dm.d, hb, nullptr, 0, T, w_blk, sa, fs, st);
  };
  if (t1 == nullptr) return go(std::integral_constant<int, SIDE_NONE>{});
  sa.x = x;
  sa.expert_idx = expert_idx;
  sa.fq = w.v1_q;
  sa.fs = (const half_t*)w.v1_s;
  sa.t1 = t1;
  sa.T = T;
  sa.d = dm.d;
  sa.q = dm.q;
  sa.r = dm.r;
  sa.k = dm.k;
  sa.n_exp = dm.G * dm.K;
  sa.n_jobs = T * dm.k;
  sa.n_side = (sa.n_jobs + 7) & ~7;
  return go(std::integral_constant<int, SIDE_T1>{});
}

hipError_t launch_skinny_resid_up(const cmoe_dims& dm, const cmoe_weights& w, int T, const int* perm,
                                  const int* inv_perm, const int* expert_idx, const float* gate, const half_t* t1, half_t* a,
                                  float* spart, hipStream_t st) {
  dim3 grid(T, (dm.d_ff + SKINNY_SN - 1) / SKINNY_SN), block(256);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, 0, st, a, t1, perm, inv_perm, expert_idx, gate, w.u1_q, (const half_t*)w.u1_s,
                       w.v2_q, (const half_t*)w.v2_s, T, dm.d_ff, dm.k, dm.q, dm.G * dm.K, spart);
  };
  auto pick = [&](auto rank) {
    constexpr int R = decltype(rank)::value;
    if (dm.k == 1) go(skinny_resid_up_kernel<R, 1>);
    else if (dm.k == 2 || R == 32) go(skinny_resid_up_kernel<R, 2>);
    else if (dm.k <= 4 || R == 16) go(skinny_resid_up_kernel<R, R <= 16 ? 4 : 2>);
    else go(skinny_resid_up_kernel<R, R <= 8 ? 8 : R == 16 ? 4 : 2>);
  };
  switch (dm.r) {
    case 4: pick(std::integral_constant<int, 4>{}); break;
    case 8: pick(std::integral_constant<int, 8>{}); break;
    case 16: pick(std::integral_constant<int, 16>{}); break;
    default: pick(std::integral_constant<int, 32>{}); break;
  }
  return hipGetLastError();
}

// y_base_sorted = W2_base(c) A.  With ures != NULL the residual-down jobs ride along (ures[tok] = sum_j g_j U2
// s_j from the s partials in token order), and the base product may come in parts of the contraction
// (parts [split][T][d] FP32, sorted rows) instead: launch_skinny_add adds them all.
hipError_t launch_skinny_down(const cmoe_dims& dm, const cmoe_weights& w, const half_t* a, int T, const int* offsets,
                              half_t* y_base_sorted, float* parts, const int* expert_idx, const float* gate,
                              const float* spart, int n_parts, float* ures, hipStream_t st) {
  SideArgs sa{};
  sa.x_div = 1;
  const half_t* w2 = w.packed ? (const half_t*)((const char*)w.packed + cmoe_packed(dm).w2) : (const half_t*)w.w2_base;
  const long w_blk = w.packed ? (long)dm.d * 32 : 0;
  const int cols = stream_cols(dm, T, true);
  if (ures == nullptr)
    return launch_stream<SIDE_NONE, false>(dm, cols, a, nullptr, w2, offsets, dm.d, dm.d_ff, y_base_sorted, nullptr, 0, T,
                                           w_blk, sa, FewSortArgs{}, st);
  sa.expert_idx = expert_idx;
  sa.gate = gate;
  sa.fq = w.u2_q;
  sa.fs = (const half_t*)w.u2_s;
  sa.spart = spart;
  sa.ures = ures;
  const int split = down_split(dm, T, cols);
  sa.T = T;
  sa.d = dm.d;
  sa.q = dm.q;
  sa.r = dm.r;
  sa.k = dm.k;
  sa.n_exp = dm.G * dm.K;
  sa.n_parts = n_parts;
  sa.n_jobs = T * ((dm.d + 2047) / 2048);
  sa.n_side = (sa.n_jobs + 7) & ~7;
  return launch_stream<SIDE_URES, false>(dm, cols, a, nullptr, w2, offsets, dm.d, dm.d_ff, y_base_sorted,
                                         split > 0 ? parts : nullptr, split, T, w_blk, sa,
                                         FewSortArgs{}, st);
}

hipError_t launch_skinny_add(const cmoe_dims& dm, const half_t* y_base_sorted, const float* parts, const float* ures,
                             const int* inv_perm, int T, half_t* y, hipStream_t st) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(T, (dm.d / 4 + 255) / 256), dim3(256), 0, st, y_base_sorted, parts, ures, inv_perm, T,
                       dm.d, y);
  };
  switch (down_split(dm, T, stream_cols(dm, T, true))) {
    case 0: go(skinny_add_kernel<1>); break;
    case 1: go(skinny_add_kernel<2>); break;
    default: go(skinny_add_kernel<4>); break;
  }
  return hipGetLastError();
}

hipError_t launch_skinny_combine(const cmoe_dims& dm, const cmoe_weights& w, const half_t* y_base_sorted,
                                 const float* s_down, const int* inv_perm, const int* expert_idx, const float* gate,
                                 int T, half_t* y, hipStream_t st) {
  hipLaunchKernelGGL(skinny_combine_kernel, dim3(T, (dm.d / 8 + 255) / 256), dim3(256), 0, st, y_base_sorted, s_down, inv_perm, expert_idx,
                     gate, w.u2_q, (const half_t*)w.u2_s, dm.d, dm.q, dm.r, dm.k, dm.G * dm.K, y);
  return hipGetLastError();
}
