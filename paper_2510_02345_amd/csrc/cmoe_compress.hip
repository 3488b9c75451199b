// Construction of the compressed form from dense expert matrices (Sec. 3.2, 3.4):
//   base(c)   = mean of the cluster's K expert matrices                       (Eq. 6)
//   Delta_e   = W_e - base(c), factorised as U_e V_e of rank r                (Eq. 7)
//   U_e, V_e  -> INT4 codes with one FP16 scale per q codes                   (Sec. 3.4)
//   optional gate: an expert whose residual has cosine similarity to the base below a
//   threshold keeps no residual                                              (Sec. 3.4)
// The rank-r factors are the best ones inside the subspace found by a randomised subspace
// iteration (sketch of l >= r rows, Rayleigh-Ritz on the sketch), which for the decaying
// residual spectra of clustered experts is the truncated SVD of Sec. 3.2 to within a
// fraction of a percent of its Frobenius error.  The heavy steps are products of the
// residual (or its transpose) with l sketch rows: streams of a materialised FP16 copy of Delta_e.
#include <type_traits>

#include "cmoe_device.h"

namespace {

constexpr int CP_LMAX = 48;   // widest sketch

// ---------------------------------------------------------------- base, residuals, norms
// One 64 x 64 tile of cluster c: the base tile (Eq. 6: FP32 sum of the K experts in index
// order, divided by K, rounded to FP16), then for each expert e of the cluster
// D = f16(W_e - base) and the tile's share of sum D^2, sum D base, sum base^2, sum W_e^2 (FP32, fixed
// order), one partial per wavefront -> part[e][tile][wave][4].  The tiles of the first CR_KEEP experts
// stay in registers between the two passes; those of further experts are read a second time (from
// cache).  Bound by the 4.5 GB it reads and writes for 64 experts of 8192 x 2048: 0.99 ms (with a
// transposed copy of the residuals beside D, 6.4 GB, 1.51 ms).
constexpr int CR_KEEP = 8;
__global__ __launch_bounds__(256) void cmp_residual_kernel(const half_t* __restrict__ W, int K, int out_d, int in_d,
                                                           half_t* __restrict__ base, half_t* __restrict__ D,
                                                           float* __restrict__ part) {
  const int c = blockIdx.z;
  const int o0 = blockIdx.y * 64, i0 = blockIdx.x * 64;
  const int tid = threadIdx.x;
  const size_t me = (size_t)out_d * in_d;
  const size_t tix = (size_t)blockIdx.y * gridDim.x + blockIdx.x, nt = (size_t)gridDim.x * gridDim.y;
  const int row0 = tid >> 3, ch = tid & 7;   // rows row0 and row0 + 32, 8 columns per thread
  size_t off[2];
  float bsum[2][8];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    off[u] = (size_t)(o0 + row0 + 32 * u) * in_d + i0 + ch * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) bsum[u][i] = 0.f;
  }
  half8 keep[CR_KEEP][2];
#pragma unroll
  for (int j = 0; j < CR_KEEP; ++j)
#pragma unroll
    for (int u = 0; u < 2; ++u)
      keep[j][u] = j < K ? *(const half8*)(W + ((size_t)c * K + j) * me + off[u]) : half8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < CR_KEEP; ++j)
    if (j < K)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 8; ++i) bsum[u][i] += (float)keep[j][u][i];
  for (int j = CR_KEEP; j < K; ++j)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const half8 w8 = *(const half8*)(W + ((size_t)c * K + j) * me + off[u]);
#pragma unroll
      for (int i = 0; i < 8; ++i) bsum[u][i] += (float)w8[i];
    }
  const float kf = (float)K;
  half8 b8[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
#pragma unroll
    for (int i = 0; i < 8; ++i) b8[u][i] = (half_t)(bsum[u][i] / kf);
    *(half8*)(base + (size_t)c * me + off[u]) = b8[u];
  }
  auto one = [&](int j, const half8 (&w)[2]) {
    const int e = c * K + j;
    float s_dd = 0.f, s_db = 0.f, s_bb = 0.f, s_ww = 0.f;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      half8 d8;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float wv = (float)w[u][i], b = (float)b8[u][i];
        d8[i] = (half_t)(wv - b);
        const float dv = (float)d8[i];
        s_dd = fmaf(dv, dv, s_dd);
        s_db = fmaf(dv, b, s_db);
        s_bb = fmaf(b, b, s_bb);
        s_ww = fmaf(wv, wv, s_ww);
      }
      *(half8*)(D + (size_t)e * me + off[u]) = d8;
    }
    // wavefront sums in a fixed order (lanes by halving); the four wavefronts' partials are
    // added, in order, by cmp_stats_kernel
    float v[4] = {s_dd, s_db, s_bb, s_ww};
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int o2 = 32; o2 > 0; o2 >>= 1) v[a] += __shfl_xor(v[a], o2, 64);
    if ((tid & 63) < 4) {
      const int a = tid & 3;
      part[(((size_t)e * nt + tix) * 4 + (tid >> 6)) * 4 + a] = a == 0 ? v[0] : a == 1 ? v[1] : a == 2 ? v[2] : v[3];
    }
  };
#pragma unroll
  for (int j = 0; j < CR_KEEP; ++j)
    if (j < K) one(j, keep[j]);
  for (int j = CR_KEEP; j < K; ++j) {
    half8 w[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) w[u] = *(const half8*)(W + ((size_t)c * K + j) * me + off[u]);
    one(j, w);
  }
}

// stats[e][a] = sum over the n_tiles (tile, wavefront) partials part[e][.][a] (FP64, fixed
// order), a = dd, db, bb, ww.
__global__ __launch_bounds__(256) void cmp_stats_kernel(const float* __restrict__ part, int n_tiles,
                                                        double* __restrict__ stats) {
  __shared__ double red[256];
  const int e = blockIdx.x, a = threadIdx.x & 3, lane4 = threadIdx.x >> 2;   // 64 strided readers per quantity
  const float* src = part + (size_t)e * n_tiles * 4 + a;
  double s = 0.0;
  int t = lane4;
  for (; t + 7 * 64 < n_tiles; t += 8 * 64) {   // eight loads in flight, added in index order
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = src[(size_t)(t + 64 * u) * 4];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += (double)v[u];
  }
  for (; t < n_tiles; t += 64) s += (double)src[(size_t)t * 4];
  red[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x < 4) {
    double tot = 0.0;
    for (int i = 0; i < 64; ++i) tot += red[i * 4 + threadIdx.x];
    stats[(size_t)e * 4 + threadIdx.x] = tot;
  }
}

// ---------------------------------------------------------------- sketch bookkeeping
// X[e l + a][:] = omega[a][:] for every expert
__global__ __launch_bounds__(256) void cmp_tile_rows_kernel(const half_t* __restrict__ omega, int l, int n,
                                                            half_t* __restrict__ X) {
  const int row = blockIdx.y, col = (blockIdx.x * 256 + threadIdx.x) * 8;
  if (col >= n) return;
  *(half8*)(X + (size_t)row * n + col) = *(const half8*)(omega + (size_t)(row % l) * n + col);
}

// ---------------------------------------------------------------- Gram matrix of the l sketch rows
// gpart[e][chunk][i] = sum over the chunk's 512 columns, in order, of X[e l + a][n] X[e l + b][n]; symmetric: the
// lower triangle is kept, (a, b <= a) at i = a (a + 1) / 2 + b.
__host__ __device__ inline int tri_size(int l) { return l * (l + 1) / 2; }
constexpr int GR_COLS = 512, GR_LD = GR_COLS + 8;
// From the tile xs [l][GR_LD], by 256 threads.  A thread takes a block of 2 x 2 elements, so that a value
// read from LDS and widened serves two products.
__device__ __forceinline__ void gram_tile(const half_t* xs, int l, float* __restrict__ dst) {
  const int h = (l + 1) / 2;
  for (int i = threadIdx.x; i < tri_size(h); i += 256) {
    int a2 = (int)((sqrtf(8.f * i + 1.f) - 1.f) * 0.5f);
    while (tri_size(a2) > i) --a2;
    while (tri_size(a2 + 1) <= i) ++a2;
    const int b2 = i - tri_size(a2);
    const half_t *xa[2], *xb[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      xa[u] = xs + min(2 * a2 + u, l - 1) * GR_LD;
      xb[u] = xs + min(2 * b2 + u, l - 1) * GR_LD;
    }
    float s[2][2] = {};
#pragma unroll 2
    for (int n = 0; n < GR_COLS; n += 8) {
      const half8 a0 = *(const half8*)(xa[0] + n), a1 = *(const half8*)(xa[1] + n);
      const half8 b0 = *(const half8*)(xb[0] + n), b1 = *(const half8*)(xb[1] + n);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float fa0 = (float)a0[u], fa1 = (float)a1[u], fb0 = (float)b0[u], fb1 = (float)b1[u];
        s[0][0] = fmaf(fa0, fb0, s[0][0]);
        s[0][1] = fmaf(fa0, fb1, s[0][1]);
        s[1][0] = fmaf(fa1, fb0, s[1][0]);
        s[1][1] = fmaf(fa1, fb1, s[1][1]);
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int a = 2 * a2 + u, b = 2 * b2 + v;
        if (a < l && b <= a) dst[tri_size(a) + b] = s[u][v];
      }
  }
}
// Block (ceil(n / 512), E); LR: l rounded up to 8.
template <int LR>
__global__ __launch_bounds__(256) void cmp_gram_kernel(const half_t* __restrict__ X, int l, int n,
                                                       float* __restrict__ gpart) {
  __shared__ __attribute__((aligned(16))) half_t xs[LR * GR_LD];
  const int e = blockIdx.y, n0 = blockIdx.x * GR_COLS, tid = threadIdx.x;
  for (int idx = tid; idx < l * (GR_COLS / 8); idx += 256) {
    const int a = idx / (GR_COLS / 8), ch = idx % (GR_COLS / 8);
    half8 v = {0, 0, 0, 0, 0, 0, 0, 0};
    if (n0 + ch * 8 < n) v = *(const half8*)(X + ((size_t)e * l + a) * n + n0 + ch * 8);
    *(half8*)(xs + a * GR_LD + ch * 8) = v;
  }
  __syncthreads();
  gram_tile(xs, l, gpart + ((size_t)e * gridDim.x + blockIdx.x) * tri_size(l));
}

// ---------------------------------------------------------------- a residual times the sketch rows
// Per expert e, with D [out][in] its residual:
//   TRANS = false: Y[a][o] = sum_i D[o][i] X[a][i]       TRANS = true: Y[a][i] = sum_o D[o][i] X[a][o]
// both from the ONE row-major D (the contraction along its columns reads fragments by transposing LDS
// reads), FP16 rows out.  The contraction is summed in four quarters, added in order.
// Bound by the stream of D.  A workgroup takes 128 output positions, a wavefront 32 of them, and the X tile is
// shared by the wavefronts, so that of the loads in flight (three stages ahead, two workgroups per CU)
// four fifths are D.  SPLIT = 2: 64 output positions and two wavefront pairs that take half of the
// contraction each, for launches whose 128-position workgroups would not fill the CUs twice.
// 64 experts of 8192 x 2048, 24 rows: 0.39 and 0.37 ms (the second from a transposed copy of D, written
// by the residual kernel for 0.5 ms, 0.40).
template <int BR, int SPLIT>   // BR: rows of X in LDS, l rounded up (16, 24, 32 or 48)
struct CmpTile {
  static constexpr int WN = 4 / SPLIT, ROWS = 32 * WN;              // wavefronts along the output; positions
  static constexpr int A_BYTES = ROWS * 128, STEP = A_BYTES + BR * 128, STAGE = SPLIT * STEP;
  static constexpr int NS = 4 * STAGE <= 80 * 1024 ? 4 : 3;
  static constexpr int PER_A = 4, B_PIECES = SPLIT * BR / 8, PER_B = (B_PIECES + 3) / 4, PER = PER_A + PER_B;
  static constexpr int SMEM = NS * STAGE, OCC = SMEM <= 80 * 1024 ? 2 : 1;   // workgroups per CU
  static constexpr int NP = BR > 32 ? 2 : 1;                        // passes of 32 accumulator columns
};
template <int BR, int SPLIT, bool TRANS>
__global__ __launch_bounds__(256, (CmpTile<BR, SPLIT>::OCC)) void cmp_stream_kernel(const half_t* __restrict__ D,
                                                                                    const half_t* __restrict__ X, int out_d,
                                                                                    int in_d, int l, int n_blocks,
                                                                                    half_t* __restrict__ Y) {
  using TL = CmpTile<BR, SPLIT>;
  constexpr int NP = TL::NP;
  __shared__ __attribute__((aligned(1024))) char smem[TL::SMEM];
  static_assert(SPLIT == 1 || 2 * 2 * NP * 4096 <= TL::SMEM, "exchange area");
  const int tid = threadIdx.x, lane = tid & 63, fr = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wave % TL::WN, half = wave / TL::WN;
  const int e = blockIdx.x / n_blocks, blk = blockIdx.x % n_blocks;
  const int N = TRANS ? in_d : out_d, Kc = TRANS ? out_d : in_d, n0 = blk * TL::ROWS;
  D += (size_t)e * out_d * in_d;
  X += (size_t)e * l * Kc;
  const int steps = Kc / 64;
  // steps of this wavefront's half: [s0, s0 + mine)
  const int mid = steps / 2, stages = SPLIT == 1 ? steps : steps - mid;
  const int s0 = SPLIT == 2 && half ? mid : 0, mine = SPLIT == 1 ? steps : half ? steps - mid : mid;
  const unsigned base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
  // chunk keys: rows of 128 bytes (X, D rows, and D columns with 64 positions): two rows span the banks
  auto key8 = [](int row) { return (row >> 1) & 7; };
  const half_t* src[TL::PER];
  unsigned dst[TL::PER];
  int last[TL::PER];   // last step of the piece's half
#pragma unroll
  for (int i = 0; i < TL::PER; ++i) {
    const bool is_a = i < TL::PER_A;
    const int g = is_a ? wave * TL::PER_A + i : min(wave * TL::PER_B + i - TL::PER_A, TL::B_PIECES - 1);
    const int per = is_a ? TL::ROWS / 8 : BR / 8, hf = g / per, pc = g % per;   // half; 1-KiB piece of its step
    const int first = SPLIT == 2 && hf ? mid : 0;
    last[i] = (SPLIT == 1 ? steps : hf ? steps - mid : mid) - 1;
    dst[i] = base + hf * TL::STEP + (is_a ? 0 : TL::A_BYTES) + pc * 1024;
    const int row = pc * 8 + (lane >> 3), ch = lane & 7;
    if (!is_a) {
      src[i] = X + (size_t)min(row, l - 1) * Kc + first * 64 + ((ch ^ key8(row)) << 3);
    } else if (!TRANS) {       // 8 output rows of 64 elements
      src[i] = D + (size_t)min(n0 + row, N - 1) * in_d + first * 64 + ((ch ^ key8(row)) << 3);
    } else if (SPLIT == 1) {   // 4 contraction rows of 128 positions
      const int r4 = pc * 4 + (lane >> 4);
      src[i] = D + (size_t)r4 * in_d + min(n0 + (((lane & 15) ^ (r4 & 15)) << 3), N - 8);
    } else {                   // 8 contraction rows of 64 positions
      src[i] = D + (size_t)(first * 64 + row) * in_d + min(n0 + ((ch ^ key8(row)) << 3), N - 8);
    }
  }
  const long a_step = TRANS ? 64L * in_d : 64L;
  auto issue = [&](int st, int stage) {
#pragma unroll
    for (int i = 0; i < TL::PER; ++i) {
      const long k = SPLIT == 1 ? st : max(min(st, last[i]), 0);   // a shorter half repeats its last step, unused
      if (i < TL::PER_A)
        dma16_nt(src[i] + k * a_step, dst[i] + stage * TL::STAGE);
      else
        dma16(src[i] + k * 64, dst[i] + stage * TL::STAGE);
    }
  };
  float16v acc[NP], sum[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[p][v] = sum[p][v] = 0.f;
  // this wavefront's quarters end (exclusively) at step s0 + fold; with SPLIT = 2 and the upper half the two
  // quarters stay apart until the lower half's sum is there
  int quarter = half * 2, fold = (quarter + 1) * steps / 4 - s0;
  float16v third[SPLIT == 2 ? NP : 1];
  auto fold_quarter = [&] {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (SPLIT == 2 && half == 1 && quarter == 2) {
        third[SPLIT == 2 ? p : 0] = acc[p];
      } else if (SPLIT == 2 && half == 1) {
        sum[p] = acc[p];
      } else {
        sum[p] += acc[p];
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[p][v] = 0.f;
    }
    ++quarter;
    fold = (quarter + 1) * steps / 4 - s0;
  };
  const int quarters_end = SPLIT == 1 ? 4 : half * 2 + 2;
#pragma unroll
  for (int s = 0; s < TL::NS - 1; ++s)
    if (s < stages) issue(s, s);
  int stage = 0, nstage = TL::NS - 1;
  for (int st = 0; st < stages; ++st) {
    // stage st has landed (own loads), then everyone's; the stage refilled below was read in iteration
    // st - 1, which every wavefront has left with its reads completed
    if (st + TL::NS - 2 < stages) wait_vm<(TL::NS - 2) * TL::PER>(); else wait_vm<0>();
    wait_lds();
    __builtin_amdgcn_s_barrier();
    if (st + TL::NS - 1 < stages) issue(st + TL::NS - 1, nstage);
    if (st < mine) {
      while (st == fold && quarter < quarters_end) fold_quarter();
      const char* sa = smem + stage * TL::STAGE + half * TL::STEP;
      const char* sb = sa + TL::A_BYTES;
#pragma unroll
      for (int s = 0; s < 4; ++s) {   // 16 contraction elements
        half8 fa;
        if (!TRANS) {
          const int row = 32 * wn + fr;
          fa = *(const half8*)(sa + row * 128 + (((2 * s + h) ^ key8(row)) << 4));
        } else {
          half4 v[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int row = 16 * s + 8 * h + 4 * u + ((lane & 15) >> 2);
            const int ch = 4 * wn + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
            v[u] = lds_read_tr(sa + row * (TL::ROWS * 2) + ((ch ^ (SPLIT == 1 ? row & 15 : key8(row))) << 4) + 8 * (lane & 1));
          }
          fa = join8(v[0], v[1]);
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          const int row = 32 * p + fr < BR ? 32 * p + fr : 0;   // columns past the rows of X are not stored
          const half8 fb = *(const half8*)(sb + row * 128 + (((2 * s + h) ^ key8(row)) << 4));
          acc[p] = mfma16(fa, fb, acc[p]);
        }
      }
    }
    stage = stage + 1 == TL::NS ? 0 : stage + 1;
    nstage = nstage + 1 == TL::NS ? 0 : nstage + 1;
  }
  while (quarter < quarters_end) fold_quarter();
  if (SPLIT == 2) {   // ((first + second) + third) + fourth quarter
    __syncthreads();  // the stages have been read
    float* red = (float*)smem + (size_t)wn * 2 * NP * 1024 + lane;
    if (half == 1)
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          red[((2 * p) * 16 + v) * 64] = third[SPLIT == 2 ? p : 0][v];
          red[((2 * p + 1) * 16 + v) * 64] = sum[p][v];
        }
    __syncthreads();
    if (half == 1) return;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        sum[p][v] += red[((2 * p) * 16 + v) * 64];
        sum[p][v] += red[((2 * p + 1) * 16 + v) * 64];
      }
  }
  const int n = n0 + 32 * wn;
  if (n >= N) return;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int row = 32 * p + fr;
    if (row >= l) continue;
#pragma unroll
    for (int qd = 0; qd < 4; ++qd)
      *(half4*)(Y + ((size_t)e * l + row) * N + n + 8 * qd + 4 * h) = to_half4(sum[p], qd);
  }
}

// ---------------------------------------------------------------- small dense steps, one workgroup per expert
// The Gram partials of an expert summed (FP64, in chunk order, sixteen loads in flight) into the full matrix A.
// Called by the whole workgroup of NT threads; ends behind a barrier.
template <int NT, int LD>
__device__ __forceinline__ void gram_sum(const float* __restrict__ src, int n_chunks, int l, double (*A)[LD]) {
  const int tri = tri_size(l);
  for (int i = threadIdx.x; i < tri; i += NT) {
    double s = 0.0;
    int ch = 0;
    for (; ch + 16 <= n_chunks; ch += 16) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = src[(size_t)(ch + u) * tri + i];
#pragma unroll
      for (int u = 0; u < 16; ++u) s += (double)v[u];
    }
    for (; ch < n_chunks; ++ch) s += (double)src[(size_t)ch * tri + i];
    int a = (int)((sqrtf(8.f * i + 1.f) - 1.f) * 0.5f);
    while (tri_size(a) > i) --a;
    while (tri_size(a + 1) <= i) ++a;
    const int b = i - tri_size(a);
    A[a][b] = s;
    A[b][a] = s;
  }
  __syncthreads();
}

// coef = inverse of the Cholesky factor of the Gram matrix, so that coef X has orthonormal rows.
//   The sketch may be rank deficient (a residual of rank below l).  A pivot below tau, which is far
// above the rounding noise of the FP16 rows and their FP32 Gram sums, marks a row the earlier rows
// already span: it gets a huge pivot, so that its output row is (numerically) zero instead of amplified
// noise and the rows after it do not see it.
//   Behind the sums a single wavefront works, a chain of l pivots: lane t keeps row t of the factor, then
// column t of the inverse, in registers, and an element that all lanes need is broadcast from its
// lane; pivots come as reciprocal square roots: 9.6 us for 24 rows (with divisions and square roots 12, with the
// matrix in LDS and three barriers per column 35).
__device__ __forceinline__ double lane_bcast(double v, int lane) {
  typedef int int2v __attribute__((ext_vector_type(2)));
  const int2v b = __builtin_bit_cast(int2v, v);
  return __builtin_bit_cast(double, int2v{__builtin_amdgcn_readlane(b[0], lane), __builtin_amdgcn_readlane(b[1], lane)});
}
// 1 / sqrt(y) in FP64 to full precision: the instruction's value and a third-order step
__device__ __forceinline__ double rsqrt_full(double y) {
  const double c = __builtin_amdgcn_rsq(y), e = fma(-y * c, c, 1.0);
  return fma(c * e, fma(e, 0.375, 0.5), c);
}
constexpr int CF_THREADS = 512;
// LB: l rounded up to 8; the rows beyond l stay zero
template <int LB>
__global__ __launch_bounds__(CF_THREADS) void cmp_factor_kernel(const float* __restrict__ gpart, int n_chunks, int l,
                                                                float* __restrict__ coef) {
  __shared__ double A[CP_LMAX][CP_LMAX + 1];
  const int e = blockIdx.x, t = threadIdx.x;
  gram_sum<CF_THREADS>(gpart + (size_t)e * n_chunks * tri_size(l), n_chunks, l, A);
  if (t >= 64) return;
  double tau = 0.0;
  for (int i = 0; i < l; ++i) tau += A[i][i];
  tau = 1e-5 * tau / l + 1e-290;
  double row[LB], inv_diag = 1.0;   // row t of A, then of L; 1 / L[t][t]
#pragma unroll
  for (int k2 = 0; k2 < LB; ++k2) row[k2] = t < l && k2 <= t ? A[t][k2] : 0.0;
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    const double ajj = lane_bcast(row[j], j), inv = ajj > tau ? rsqrt_full(ajj) : 1e-150;
    if (t == j) inv_diag = inv;
    row[j] *= inv;
#pragma unroll
    for (int k2 = j + 1; k2 < LB; ++k2)   // rows t >= k2; the others' values are not read
      row[k2] -= row[j] * lane_bcast(row[j], k2);
  }
  // V = L^-1 by forward substitution, lane t: column t
  float* cf = coef + (size_t)e * CP_LMAX * CP_LMAX;
  double v[LB];
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    double s = i == t ? 1.0 : 0.0;
#pragma unroll
    for (int k2 = 0; k2 < i; ++k2) s -= lane_bcast(row[k2], i) * v[k2];
    v[i] = s * lane_bcast(inv_diag, i);
    if (i < l && t < CP_LMAX) cf[i * CP_LMAX + t] = t <= i ? (float)v[i] : 0.f;
  }
}

// Rayleigh-Ritz: Jacobi eigenvectors of the Gram matrix; coef rows = the r eigenvectors of largest
// eigenvalue (transposed), and lam[e] = the sum of those eigenvalues.  The sweeps use the round-robin
// ordering: a sweep is l - 1 rounds of l / 2 rotations on disjoint index pairs, which commute, so a
// round applies all of them at once, A <- J^T A J and V <- V J, every element by one thread.
// A chain of rounds, one workgroup per expert: what counts is a round's latency.  The rotation of a pair comes from the
// reciprocal instructions, the tangent as they give it (a rotation need not annihilate to the last bit), the cosine with a
// third-order step to full precision.  A thread takes the 2 x 2 elements of A where two pairs meet, or the two of a
// row of V in a pair, which it may overwrite, so that a round reads half of the LDS and has two barriers: 64 experts,
// 24 rows 164 us with divisions, square roots and an element a thread, 139 with the reciprocals alone, 98 so.
constexpr int CS_THREADS = 512;
template <int LB>   // l rounded up to 8
__global__ __launch_bounds__(CS_THREADS) void cmp_ritz_kernel(const float* __restrict__ gpart, int n_chunks, int l, int r,
                                                              float* __restrict__ coef, double* __restrict__ lam) {
  __shared__ double A[LB][LB + 1], V[LB][LB + 1];
  __shared__ double ev[LB];
  __shared__ int order[LB];
  const int e = blockIdx.x, t = threadIdx.x;
  gram_sum<CS_THREADS>(gpart + (size_t)e * n_chunks * tri_size(l), n_chunks, l, A);
  float* cf = coef + (size_t)e * CP_LMAX * CP_LMAX;
  __shared__ double cc[LB / 2], ss[LB / 2];   // of pair h: new column p = c column p - s column q, q = c column q + s column p
  __shared__ double red[2][CS_THREADS / 64];
  for (int idx = t; idx < l * l; idx += CS_THREADS) V[idx / l][idx % l] = (idx / l == idx % l) ? 1.0 : 0.0;
  const int np = (l + 1) / 2, m = 2 * np - 1;   // pairs of a round; an odd l plays with one idle index
  // pair h of round rr: p < q; q >= l: p has no partner
  auto pair = [&](int h, int rr, int& p, int& q) {
    int a = rr + h, b = rr - h;
    a -= a >= m ? m : 0;
    b += b < 0 ? m : 0;
    if (h == 0) a = m;
    p = min(a, b);
    q = max(a, b);
  };
  // this thread's items: pairs (h, g) of A, then rows and pairs of V
  constexpr int N_ITEM = LB / 2 * (LB / 2) + LB * (LB / 2), PER = (N_ITEM + CS_THREADS - 1) / CS_THREADS;
  int item_h[PER], item_g[PER];   // g: pair of the columns; h: pair of the rows, or -1 - row of V; g < 0: none
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = t + u * CS_THREADS, j = i - np * np;
    item_g[u] = j < 0 ? i % np : j < l * np ? j % np : -1;
    item_h[u] = j < 0 ? i / np : -1 - j / np;
  }
  __syncthreads();
  for (int sweep = 0; sweep < 12; ++sweep) {
    // converged when every off-diagonal element is negligible against the diagonal
    double offmax = 0.0, diagmax = 0.0;
    for (int idx = t; idx < l * l; idx += CS_THREADS) {
      const double a = fabs(A[idx / l][idx % l]);
      if (idx / l == idx % l) diagmax = fmax(diagmax, a); else offmax = fmax(offmax, a);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      offmax = fmax(offmax, __shfl_xor(offmax, off, 64));
      diagmax = fmax(diagmax, __shfl_xor(diagmax, off, 64));
    }
    if ((t & 63) == 0) {
      red[0][t >> 6] = offmax;
      red[1][t >> 6] = diagmax;
    }
    __syncthreads();
    offmax = 0.0;
    diagmax = 0.0;
    for (int w = 0; w < CS_THREADS / 64; ++w) {
      offmax = fmax(offmax, red[0][w]);
      diagmax = fmax(diagmax, red[1][w]);
    }
    if (offmax <= 1e-10 * diagmax) break;   // the same values in every thread
    for (int rr = 0; rr < m; ++rr) {
      if (t < np) {
        int p, q;
        pair(t, rr, p, q);
        double c = 1.0, sn = 0.0;
        if (q < l) {
          const double apq = A[p][q], app = A[p][p], aqq = A[q][q];
          if (fabs(apq) > 1e-300 && apq * apq > 1e-34 * fabs(app * aqq)) {
            // |tan| = |b| / (|d| + sqrt(d^2 + b^2)), d = aqq - app, b = 2 apq, scaled by the larger
            const double d0 = aqq - app, b0 = 2.0 * apq, sc = __builtin_amdgcn_rcp(fmax(fabs(d0), fabs(b0)));
            const double d = d0 * sc, b = b0 * sc, x = fma(d, d, b * b);
            const double at = fabs(b) * __builtin_amdgcn_rcp(fma(x, __builtin_amdgcn_rsq(x), fabs(d)));
            const double tt = d == 0.0 || (d > 0.0) == (b > 0.0) ? at : -at;
            c = rsqrt_full(fma(tt, tt, 1.0));
            sn = tt * c;
          }
        }
        cc[t] = c;
        ss[t] = sn;
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        if (item_g[u] < 0) continue;
        int p, q;
        pair(item_g[u], rr, p, q);
        const bool two = q < l;
        const int qc = two ? q : p;
        const double c = cc[item_g[u]], sn = ss[item_g[u]];
        if (item_h[u] < 0) {
          double* v = V[-1 - item_h[u]];
          const double x = v[p], y = v[qc];
          v[p] = c * x - sn * y;
          if (two) v[q] = c * y + sn * x;
        } else {
          int i, k;
          pair(item_h[u], rr, i, k);
          const bool rows = k < l;
          const int kc = rows ? k : i;
          const double ci = cc[item_h[u]], si = ss[item_h[u]];
          const double a00 = A[i][p], a01 = A[i][qc], a10 = A[kc][p], a11 = A[kc][qc];
          const double x00 = c * a00 - sn * a01, x01 = c * a01 + sn * a00, x10 = c * a10 - sn * a11, x11 = c * a11 + sn * a10;
          A[i][p] = ci * x00 - si * x10;
          if (two) A[i][q] = ci * x01 - si * x11;
          if (rows) A[k][p] = ci * x10 + si * x00;
          if (rows && two) A[k][q] = ci * x11 + si * x01;
        }
      }
      __syncthreads();
    }
  }
  if (t < l) ev[t] = A[t][t];
  __syncthreads();
  if (t < l) {   // rank of eigenvalue t in descending order, ties by index
    int rank = 0;
    for (int i = 0; i < l; ++i) rank += (ev[i] > ev[t]) || (ev[i] == ev[t] && i < t);
    order[rank] = t;
  }
  __syncthreads();
  for (int idx = t; idx < r * CP_LMAX; idx += CS_THREADS) {
    const int rho = idx / CP_LMAX, b = idx % CP_LMAX;
    cf[idx] = b < l ? (float)V[b][order[rho]] : 0.f;
  }
  if (t == 0) {
    double s = 0.0;
    for (int rho = 0; rho < r; ++rho) s += fmax(ev[order[rho]], 0.0);
    lam[e] = s;
  }
}

// ---------------------------------------------------------------- out[e][a][:] = sum_b coef[e][a][b] X[e l + b][:]
// A thread takes two columns and keeps their l <= 8 NB values; the coefficients are read from LDS (16 experts, 24 rows
// of 1024 to 4096: 11 and 17 us without and with the Gram part, as scalar loads row by row 15 and 20).  GRAM: also the workgroup's part of the Gram matrix of the rounded rows (ra = l).  Block (ceil(n / 512), E).
template <int NB, bool GRAM, class OutT>
__global__ __launch_bounds__(256) void cmp_apply_kernel(const float* __restrict__ coef, const half_t* __restrict__ X,
                                                        int l, int ra, int n, OutT* __restrict__ out,
                                                        float* __restrict__ gpart) {
  constexpr int LB = 8 * NB;
  typedef OutT out2 __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(16))) half_t xs[GRAM ? LB * GR_LD : 8];
  __shared__ __attribute__((aligned(16))) float cs[LB * LB];   // ra <= l
  const int e = blockIdx.y, tid = threadIdx.x;
  const int col = blockIdx.x * 512 + tid * 2;   // n is even
  const bool in = col < n;
  float x0[LB], x1[LB];
#pragma unroll
  for (int b = 0; b < LB; ++b) {
    half2v v = {0, 0};
    if (b < l && in) v = *(const half2v*)(X + ((size_t)e * l + b) * n + col);
    x0[b] = (float)v[0];
    x1[b] = (float)v[1];
  }
  for (int i = tid; i < ra * (LB / 4); i += 256)
    *(float4v*)(cs + i * 4) = *(const float4v*)(coef + ((size_t)e * CP_LMAX + i / (LB / 4)) * CP_LMAX + i % (LB / 4) * 4);
  __syncthreads();
  for (int a = 0; a < ra; ++a) {
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int b4 = 0; b4 < LB / 4; ++b4) {
      const float4v c = *(const float4v*)(cs + a * LB + b4 * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s0 = fmaf(c[i], x0[b4 * 4 + i], s0);
        s1 = fmaf(c[i], x1[b4 * 4 + i], s1);
      }
    }
    const out2 o = {(OutT)s0, (OutT)s1};
    if (in) *(out2*)(out + ((size_t)e * ra + a) * n + col) = o;
    if constexpr (GRAM) *(half2v*)(xs + a * GR_LD + tid * 2) = in ? half2v{o[0], o[1]} : half2v{0, 0};
  }
  if constexpr (GRAM) {
    __syncthreads();
    gram_tile(xs, l, gpart + ((size_t)e * gridDim.x + blockIdx.x) * tri_size(l));
  }
}

// ---------------------------------------------------------------- Sec. 3.4 quantiser
// Groups of q consecutive elements of a row: scale = f16(absmax / 7), code = clip(rint(w / scale), -7, 7), codes
// 0 when the scale rounds to 0 or the row's expert is gated off (gate != NULL and
// gate[row / rows_per_expert] != 0).
__device__ __forceinline__ half_t quant_scale(float absmax, bool off) { return off ? (half_t)0.f : (half_t)(absmax / 7.0f); }
__device__ __forceinline__ unsigned quant_code(float w, float sc) {   // sc > 0
  return (unsigned)(int)fminf(fmaxf(rintf(w / sc), -7.f), 7.f) & 0xFu;
}
// q = 8, 16, .. 512: a thread takes eight elements (32 contiguous bytes, one code word), q / 8 lanes a group.
// 33 MB of factors (64 experts, rank 16, 8192): 74 us with a thread per group of 64.
__global__ __launch_bounds__(256) void cmp_quantize8_kernel(const float* __restrict__ src, long words, int L, int q,
                                                            const int* __restrict__ gate, int rows_per_expert,
                                                            uint8_t* __restrict__ codes, half_t* __restrict__ scales) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  const bool in = i < words;   // a group's lanes lie in one wavefront and are in or out together
  float v[8];
  const float4v a = in ? *(const float4v*)(src + i * 8) : float4v{0.f, 0.f, 0.f, 0.f};
  const float4v b = in ? *(const float4v*)(src + i * 8 + 4) : float4v{0.f, 0.f, 0.f, 0.f};
  float absmax = 0.f;
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    v[u] = u < 4 ? a[u & 3] : b[u & 3];
    absmax = fmaxf(absmax, fabsf(v[u]));
  }
  for (int off = 1; off < q / 8; off <<= 1) absmax = fmaxf(absmax, __shfl_xor(absmax, off, 64));
  if (!in) return;
  const bool off = gate != nullptr && gate[i * 8 / L / rows_per_expert] != 0;
  const half_t sc = quant_scale(absmax, off);
  if (i * 8 % q == 0) scales[i * 8 / q] = sc;
  unsigned w = 0;
#pragma unroll
  for (int u = 0; u < 8; ++u) w |= sc > (half_t)0.f ? quant_code(v[u], (float)sc) << (4 * u) : 0u;
  *(unsigned*)(codes + i * 4) = w;
}
// Any even q: one thread per group.
__global__ __launch_bounds__(256) void cmp_quantize_kernel(const float* __restrict__ src, long rows, int L, int q,
                                                           const int* __restrict__ gate, int rows_per_expert,
                                                           uint8_t* __restrict__ codes, half_t* __restrict__ scales) {
  const long gidx = (long)blockIdx.x * 256 + threadIdx.x;
  const int gpr = L / q;
  if (gidx >= rows * gpr) return;
  const long row = gidx / gpr;
  const int g = (int)(gidx % gpr);
  const float* s = src + row * L + (long)g * q;
  const bool off = gate != nullptr && gate[row / rows_per_expert] != 0;
  float absmax = 0.f;
  for (int i = 0; i < q; ++i) absmax = fmaxf(absmax, fabsf(s[i]));
  const half_t sc = quant_scale(absmax, off);
  const float scf = (float)sc;
  scales[row * gpr + g] = sc;
  uint8_t* dst = codes + row * (L / 2) + (long)g * (q / 2);
  for (int i = 0; i < q; i += 2) {
    unsigned c = 0u;
    if (scf > 0.f) c = quant_code(s[i], scf) | quant_code(s[i + 1], scf) << 4;
    dst[i / 2] = (uint8_t)c;
  }
}
}  // namespace
// The word-wise kernel: its group lengths, and no more words than a launch has threads (a thread per group goes further).
bool quantize_by_words(long rows, int L, int q) {
  return q >= 8 && q <= 512 && (q & (q - 1)) == 0 && rows * (L / 8) <= (1L << 32) - 256;
}
namespace {
hipError_t launch_quantize(const float* src, long rows, int L, int q, const int* gate, int rows_per_expert, uint8_t* codes,
                           half_t* scales, hipStream_t st) {
  if (quantize_by_words(rows, L, q)) {
    const long words = rows * (L / 8);
    hipLaunchKernelGGL(cmp_quantize8_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, src, words, L, q, gate,
                       rows_per_expert, codes, scales);
  } else {
    const long groups = rows * (L / q);
    hipLaunchKernelGGL(cmp_quantize_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, st, src, rows, L, q, gate,
                       rows_per_expert, codes, scales);
  }
  return hipGetLastError();
}

// gate[e] = 1 when cos(vec Delta_e, vec base_c) < gamma (Sec. 3.4); report[e][2] = cosine,
// report[e][3] = gate, report[e][1] = rank-r error before quantisation
//   sqrt(max(||Delta||^2 - sum of the r largest Ritz values, 0)) / ||W_e||.
__global__ void cmp_gate_kernel(const double* __restrict__ stats, const double* __restrict__ lam, int E, int use_gate,
                                float gamma, int* __restrict__ gate, float* __restrict__ report) {
  const int e = blockIdx.x * 64 + threadIdx.x;
  if (e >= E) return;
  const double dd = stats[e * 4 + 0], db = stats[e * 4 + 1], bb = stats[e * 4 + 2], ww = stats[e * 4 + 3];
  const double den = sqrt(dd) * sqrt(bb);
  const double cosv = den > 0.0 ? db / den : 0.0;
  const int g = (use_gate && cosv < (double)gamma) ? 1 : 0;
  gate[e] = g;
  report[e * 4 + 1] = ww > 0.0 ? (float)(sqrt(fmax(dd - lam[e], 0.0)) / sqrt(ww)) : 0.f;
  report[e * 4 + 2] = (float)cosv;
  report[e * 4 + 3] = (float)g;
}

// ---------------------------------------------------------------- reconstruction error of a stored form
// epart[e][workgroup] = sum over its elements of (W - base - U V)^2 with U, V dequantised
// (Sec. 3.2's Frobenius error, for what the layer will actually compute); wpart = sum W^2.
__device__ __forceinline__ float cmp_nib(const uint8_t* row, int n) {
  const unsigned b = row[n >> 1];
  return (float)((int)((n & 1 ? b >> 4 : b & 0xF) ^ 8) - 8);
}
// A workgroup takes RT tiles of 64 rows and CE_CT consecutive 64-column tiles of one expert, the global loads of a
// row tile issued before the work on the one above it; epart has one entry per workgroup.  A one-dimensional grid of
// 8 * ceil(G * tiles / 8) * K workgroups.  U V takes r products per element (34 GFLOP for 64 experts of 8192 x 2048
// at r = 16) next to 2.4 GB of reads.  A factor value, FP16 scale x INT4 code, has at most 14 significant
// bits and splits exactly into two FP16 parts, so that four FP16 products are the exact product and the
// FP16 matrix instruction (FP32 sums) rebuilds U V in a quarter of the FP32 instruction's time, from panels
// of which those of all column tiles fit LDS at once: 778 -> 640 us.
// Columns are its rows (A = V), rows its columns (B = U); a wavefront owns 16 rows, and tile row
// 4 q + i of block a holds column 8 q + 4 a + i of 32, so that blocks 0 and 1 give lane (t, q) the
// eight consecutive columns 8 q .. 8 q + 7 of row t, as it loads them from W and base.
// CE_CT = 4, or as many as a narrower matrix has: 15 experts of 2112 x 64 28.5 us on the FP32 instruction, 29.9 with four
// tiles loaded of which one exists, 25.9 with one (each with its launches and the wait of the caller).
// A panel row (one column of V, one row of U): the upper parts of RB rank values, then the lower ones.
template <int RB, int CE_CT, int RT>
__global__ __launch_bounds__(256) void cmp_error_kernel(const half_t* __restrict__ W, const half_t* __restrict__ base,
                                                        const uint8_t* __restrict__ u_q,
                                                        const half_t* __restrict__ u_s,
                                                        const uint8_t* __restrict__ v_q,
                                                        const half_t* __restrict__ v_s, int G, int K, int out_d, int in_d,
                                                        int r, int q, int tiles_x, int tiles_y,
                                                        float* __restrict__ epart) {
  constexpr int LD = 2 * RB + 8, CE_COLS = 64 * CE_CT;
  __shared__ __attribute__((aligned(16))) half_t us[64 * RT][LD], vs[CE_COLS][LD];
  __shared__ float red[4][2];
  // Workgroups are dealt round-robin to the 8 XCDs; the K experts of one (cluster, tile) take
  // K consecutive workgroups of ONE XCD, so that the base tile they share is fetched from
  // memory once and found in that XCD's L2 by the others.
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
  const int tc = (local / K) * 8 + xcd, per_c = tiles_x * tiles_y;
  if (tc >= G * per_c) return;
  const int c = tc / per_c, e = c * K + local % K;
  const int tile_y = (tc % per_c) / tiles_x, tile_x = (tc % per_c) % tiles_x;
  const int o0 = tile_y * 64 * RT, c0 = tile_x * CE_COLS, tid = threadIdx.x;
  const int t16 = tid & 15, quad = (tid >> 4) & 3, row = (tid >> 6) * 16 + t16;
  const size_t me = (size_t)out_d * in_d;
  // Panels: a thread takes two rank rows (rho, rho + 1) and one word of eight codes of each, at a time
  // (one scale per word when q is a multiple of 8; other group lengths take the element-wise path).
  const bool words = (q % 8) == 0;
  constexpr int PAIRS = RB / 2, V_ITEMS = PAIRS * CE_COLS / 8, U_ITEMS = PAIRS * 8 * RT;
  constexpr int PER = (V_ITEMS + U_ITEMS + 255) / 256;
  unsigned pw[PER][2];
  float ps[PER][2];
  auto item = [&](int u, int& rho, int& word, bool& is_v) {   // of the panels; false: none
    int i = tid + u * 256;
    is_v = i < V_ITEMS;
    if (!is_v) i -= V_ITEMS;
    rho = 2 * (i % PAIRS);
    word = i / PAIRS;
    return is_v || i < U_ITEMS;
  };
  if (words)
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      int rho, word;
      bool is_v;
      const bool some = item(u, rho, word, is_v);
      const int L = is_v ? in_d : out_d, at = (is_v ? c0 : o0) + word * 8;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        pw[u][h] = 0u;
        ps[u][h] = 0.f;
        if (some && rho + h < r && at < L) {
          const size_t fr = (size_t)e * r + rho + h;
          pw[u][h] = *(const unsigned*)((is_v ? v_q : u_q) + fr * (L / 2) + at / 2);
          ps[u][h] = (float)(is_v ? v_s : u_s)[fr * (L / q) + at / q];
        }
      }
    }
  struct Elements {
    half8 w[CE_CT][2], b[CE_CT][2];
  } next;
  auto load = [&](Elements& v, int rt) {   // of row tile rt; past the last row the last tile's again
    const int o = min(o0 + 64 * rt, out_d - 64) + row;
#pragma unroll
    for (int ct = 0; ct < CE_CT; ++ct) {
      const int i0 = c0 + ct * 64;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const size_t off = (size_t)o * in_d + (i0 < in_d ? i0 : 0) + 32 * u + quad * 8;
        v.w[ct][u] = *(const half8*)(W + (size_t)e * me + off);
        v.b[ct][u] = *(const half8*)(base + (size_t)c * me + off);
      }
    }
  };
  load(next, 0);
  if (words) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      int rho, word;
      bool is_v;
      if (!item(u, rho, word, is_v)) continue;
      half_t* dst = (is_v ? &vs[word * 8][0] : &us[word * 8][0]) + rho;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        half2v hi, lo;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float v = ps[u][h] * (float)((int)((pw[u][h] >> (4 * i) & 0xFu) ^ 8u) - 8);
          hi[h] = (half_t)v;
          lo[h] = (half_t)(v - (float)hi[h]);
        }
        *(half2v*)(dst + i * LD) = hi;
        *(half2v*)(dst + i * LD + RB) = lo;
      }
    }
  } else {
    for (int idx = tid; idx < RB * (CE_COLS + 64 * RT); idx += 256) {
      const int rho = idx % RB, j = idx / RB;
      const bool is_v = j < CE_COLS;
      const int L = is_v ? in_d : out_d, at = is_v ? c0 + j : o0 + j - CE_COLS;
      float v = 0.f;
      if (rho < r && at < L) {
        const size_t fr = (size_t)e * r + rho;
        v = (float)(is_v ? v_s : u_s)[fr * (L / q) + at / q] * cmp_nib((is_v ? v_q : u_q) + fr * (L / 2), at);
      }
      half_t* dst = is_v ? &vs[j][rho] : &us[j - CE_COLS][rho];
      dst[0] = (half_t)v;
      dst[RB] = (half_t)(v - (float)(half_t)v);
    }
  }
  __syncthreads();
  float se = 0.f, sw = 0.f;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    if (o0 + 64 * rt >= out_d) break;   // uniform over the workgroup
    const Elements now = next;
    if (rt + 1 < RT) load(next, rt + 1);
    float et = 0.f, wt = 0.f;   // sums of this tile: chains of 64 values a lane, as with one tile a workgroup
    // U operands: with 16 rank values the matrix instruction's 32 contraction elements are both parts of V
    // against one part of U twice; with 32 one part of each
    half8 fu[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) fu[p] = *(const half8*)&us[64 * rt + row][p * RB + (RB == 16 ? 8 * (quad & 1) : 8 * quad)];
#pragma unroll
    for (int ct = 0; ct < CE_CT; ++ct) {
      if (c0 + ct * 64 >= in_d) break;   // uniform over the workgroup
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float4v uv[2] = {};
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const half_t* v = &vs[ct * 64 + 32 * u + 8 * (t16 >> 2) + 4 * a + (t16 & 3)][8 * quad];
#pragma unroll
          for (int pv = 0; pv < RB / 16; ++pv) {
            const half8 fv = *(const half8*)(v + pv * RB);
#pragma unroll
            for (int p = 0; p < 2; ++p) uv[a] = mfma32(fv, fu[p], uv[a]);
          }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float w = (float)now.w[ct][u][i];
          const float dv = w - (float)now.b[ct][u][i] - uv[i >> 2][i & 3];
          et = fmaf(dv, dv, et);
          wt = fmaf(w, w, wt);
        }
      }
    }
    se += et;
    sw += wt;
  }
  // a factor value beyond FP16 (a scale above 8188) leaves parts of infinity and an error that is not a number:
  // the lane's elements once more, product by product in FP32
  if (!(se < INFINITY)) {
    se = 0.f;
    for (int rc = 0; rc < RT * CE_CT; ++rc) {
      const int ct = rc % CE_CT, o0t = o0 + 64 * (rc / CE_CT);
      if (o0t >= out_d || c0 + ct * 64 >= in_d) continue;
      float et = 0.f;
      for (int u = 0; u < 2; ++u) {
        const int col = c0 + ct * 64 + 32 * u + quad * 8;
        const half8 wv = *(const half8*)(W + (size_t)e * me + (size_t)(o0t + row) * in_d + col);
        const half8 bv = *(const half8*)(base + (size_t)c * me + (size_t)(o0t + row) * in_d + col);
        for (int i = 0; i < 8; ++i) {
          float uv = 0.f;
          for (int rho = 0; rho < r; ++rho) {
            const size_t fr = (size_t)e * r + rho;
            uv = fmaf((float)u_s[fr * (out_d / q) + (o0t + row) / q] * cmp_nib(u_q + fr * (out_d / 2), o0t + row),
                      (float)v_s[fr * (in_d / q) + (col + i) / q] * cmp_nib(v_q + fr * (in_d / 2), col + i), uv);
          }
          const float dv = (float)wv[i] - (float)bv[i] - uv;
          et = fmaf(dv, dv, et);
        }
      }
      se += et;
    }
  }
  float v[2] = {se, sw};
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v[a] += __shfl_xor(v[a], off, 64);
  if ((tid & 63) == 0) {
    red[tid >> 6][0] = v[0];
    red[tid >> 6][1] = v[1];
  }
  __syncthreads();
  if (tid < 2)
    epart[((size_t)e * per_c + tc % per_c) * 2 + tid] = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
}
// err[e * stride] = sqrt(sum epart[..][0]) / sqrt(sum epart[..][1]), FP64, fixed order
__global__ __launch_bounds__(64) void cmp_error_finish_kernel(const float* __restrict__ epart, int n_tiles, int stride,
                                                              float* __restrict__ err) {
  const int e = blockIdx.x, lane = threadIdx.x;
  double se = 0.0, sw = 0.0;
  for (int t = lane; t < n_tiles; t += 64) {
    se += (double)epart[((size_t)e * n_tiles + t) * 2];
    sw += (double)epart[((size_t)e * n_tiles + t) * 2 + 1];
  }
  for (int off = 32; off > 0; off >>= 1) {
    se += __shfl_xor(se, off, 64);
    sw += __shfl_xor(sw, off, 64);
  }
  if (lane == 0) err[(size_t)e * stride] = sw > 0.0 ? (float)(sqrt(se) / sqrt(sw)) : 0.f;
}

// epart and then err[e * stride] of the stored form.
}  // namespace
// Row tiles of a workgroup of cmp_error_kernel: four share the panel of V and load the next tile's elements during the work on one,
// where that leaves four workgroups a CU and the last of a column has not too few of its four, on average 3.5 (3 at rank 17 on,
// where the panel is twice the work).  One and four: 64 experts of 8192 x 2048 644 -> 593 us at r = 16 and 923 -> 736 at r = 32,
// 16 of 4096 x 1024 63.9 -> 59.3 and 79.4 -> 65.7 (at r = 24 and groups of 2 codes 174 -> 108); of 64 experts, r = 16, 1472 x 1024
// (3.83) 78.3 -> 73.7, 1344 x 1024 (3.5) 74.2 -> 73.5, 832 x 2048 (3.25) 84.9 -> 87.0, 576 x 2048 (3) 67.3 -> 71.9, 320 x 2048
// (2.5) 49.6 -> 54.0; r = 32, 832 x 2048 109.3 -> 101.4, 576 x 2048 84.2 -> 81.0, 320 x 2048 59.4 -> 60.9.
int error_row_tiles(const cmoe_compress_config& c) {
  const int tiles = c.out_dim / 64, groups = (tiles + 3) / 4;
  const bool full = 2 * tiles >= (c.r > 16 ? 6 : 7) * groups;
  return c.in_dim > 128 && full && (long)c.G * c.K * ((c.in_dim / 64 + 3) / 4) * (c.out_dim / 256) >= 1024 ? 4 : 1;
}
namespace {
void launch_error(const cmoe_compress_config& c, const half_t* W, const half_t* base, const uint8_t* u_q, const half_t* u_s,
                  const uint8_t* v_q, const half_t* v_s, float* epart, int stride, float* err, hipStream_t st) {
  const int ct = c.in_dim <= 64 ? 1 : c.in_dim <= 128 ? 2 : 4;
  const int tx = (c.in_dim / 64 + ct - 1) / ct, rt = error_row_tiles(c), ty = (c.out_dim / 64 + rt - 1) / rt;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((c.G * tx * ty + 7) / 8 * 8 * c.K)), dim3(256), 0, st, W, base, u_q, u_s, v_q, v_s,
                       c.G, c.K, c.out_dim, c.in_dim, c.r, c.q_group, tx, ty, epart);
  };
  auto pick = [&](auto rb) {
    constexpr int RB = decltype(rb)::value;
    if (ct == 1) go(cmp_error_kernel<RB, 1, 1>);
    else if (ct == 2) go(cmp_error_kernel<RB, 2, 1>);
    else if (rt == 1) go(cmp_error_kernel<RB, 4, 1>);
    else go(cmp_error_kernel<RB, 4, 4>);
  };
  if (c.r <= 16) pick(std::integral_constant<int, 16>{}); else pick(std::integral_constant<int, 32>{});
  hipLaunchKernelGGL(cmp_error_finish_kernel, dim3(c.G * c.K), dim3(64), 0, st, (const float*)epart, tx * ty, stride, err);
}

struct CompressLayout {
  size_t D, XA, XB, part, stats, gpart, coef, lam, gate, UF, VF, epart, total;
};
CompressLayout compress_layout(const cmoe_compress_config& c) {
  CompressLayout L{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t at = off;
    off = (off + bytes + 255) & ~(size_t)255;
    return at;
  };
  const size_t E = (size_t)c.G * c.K, me = (size_t)c.out_dim * c.in_dim;
  const size_t nmax = c.out_dim > c.in_dim ? c.out_dim : c.in_dim;
  const size_t tiles = (size_t)(c.out_dim / 64) * (c.in_dim / 64);
  L.D = take(E * me * 2);
  L.XA = take(E * c.sketch * nmax * 2);
  L.XB = take(E * c.sketch * nmax * 2);
  L.part = take(E * tiles * 4 * 4 * 4);   // four quantities x four wavefront partials per tile
  L.stats = take(E * 4 * 8);
  L.gpart = take(E * ((nmax + GR_COLS - 1) / GR_COLS) * tri_size(c.sketch) * 4);
  L.coef = take(E * CP_LMAX * CP_LMAX * 4);
  L.lam = take(E * 8);
  L.gate = take(E * 4);
  L.UF = take(E * c.r * (size_t)c.out_dim * 4);
  L.VF = take(E * c.r * (size_t)c.in_dim * 4);
  L.epart = take(E * tiles * 2 * 4);
  L.total = off;
  return L;
}

bool compress_cfg_ok(const cmoe_compress_config* c) {
  if (c == nullptr) return false;
  if (c->out_dim <= 0 || c->in_dim <= 0 || c->out_dim % 64 || c->in_dim % 64) return false;
  if (c->G < 1 || c->K < 1 || c->K > 64 || (long)c->G * c->K > 4096) return false;
  if (c->r < 1 || c->r > 32 || c->sketch < c->r || c->sketch > CP_LMAX) return false;
  if (c->q_group < 2 || c->q_group % 2 || c->out_dim % c->q_group || c->in_dim % c->q_group) return false;
  if (c->n_iter < 0 || c->n_iter > 16) return false;
  return true;
}
bool cptr_ok(const void* p) { return p != nullptr && (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

#define CP_CHECK()                         \
  do {                                     \
    hipError_t e_ = hipGetLastError();     \
    if (e_ != hipSuccess) return CMOE_ERR_HIP; \
  } while (0)

// f(kernel<LR>) for l rounded up to LR, a multiple of 8.
template <class F>
void for_rows(int l, F f) {
  switch ((l + 7) / 8) {
    case 1: f(std::integral_constant<int, 8>{}); break;
    case 2: f(std::integral_constant<int, 16>{}); break;
    case 3: f(std::integral_constant<int, 24>{}); break;
    case 4: f(std::integral_constant<int, 32>{}); break;
    case 5: f(std::integral_constant<int, 40>{}); break;
    default: f(std::integral_constant<int, 48>{}); break;
  }
}

// The product of every residual (TRANS: transposed) with the sketch rows X -> Y, and the Gram partials of Y.
// Workgroups of 128 output positions when they fill the CUs at two each, else of 64.
template <bool TRANS>
void stream_product(const cmoe_compress_config& c, const half_t* D, const half_t* X, half_t* Y, float* gpart, hipStream_t st) {
  const int E = c.G * c.K, l = c.sketch, N = TRANS ? c.in_dim : c.out_dim;
  const bool wide = (long)E * ((N + 127) / 128) >= 512;
  const int blocks = wide ? (N + 127) / 128 : N / 64;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)(E * blocks)), dim3(256), 0, st, D, X, c.out_dim, c.in_dim, l, blocks, Y);
  };
  if (wide) {
    if (l <= 16) go(cmp_stream_kernel<16, 1, TRANS>);
    else if (l <= 24) go(cmp_stream_kernel<24, 1, TRANS>);
    else if (l <= 32) go(cmp_stream_kernel<32, 1, TRANS>);
    else go(cmp_stream_kernel<48, 1, TRANS>);
  } else {
    if (l <= 16) go(cmp_stream_kernel<16, 2, TRANS>);
    else if (l <= 24) go(cmp_stream_kernel<24, 2, TRANS>);
    else if (l <= 32) go(cmp_stream_kernel<32, 2, TRANS>);
    else go(cmp_stream_kernel<48, 2, TRANS>);
  }
  for_rows(l, [&](auto lr) {
    hipLaunchKernelGGL((cmp_gram_kernel<decltype(lr)::value>), dim3((N + GR_COLS - 1) / GR_COLS, E), dim3(256), 0, st, Y, l, N,
                       gpart);
  });
}

template <bool GRAM, class OutT>
void apply_coef(const cmoe_compress_config& c, const float* coef, const half_t* X, int ra, int n, OutT* out, float* gpart,
                hipStream_t st) {
  for_rows(c.sketch, [&](auto lr) {
    hipLaunchKernelGGL((cmp_apply_kernel<decltype(lr)::value / 8, GRAM, OutT>), dim3((n + GR_COLS - 1) / GR_COLS, c.G * c.K),
                       dim3(256), 0, st, coef, X, c.sketch, ra, n, out, gpart);
  });
}

// Rows of X [E l][n] with their Gram partials -> orthonormal rows, in place (tmp: another buffer of the
// size), by Cholesky QR applied twice: the second pass takes the rows from a few per cent off to FP16 rounding.
void orth_rows(const cmoe_compress_config& c, int n, half_t* X, half_t* tmp, char* ws, const CompressLayout& L,
               hipStream_t st) {
  float *gpart = (float*)(ws + L.gpart), *coef = (float*)(ws + L.coef);
  auto factor = [&] {
    for_rows(c.sketch, [&](auto lr) {
      hipLaunchKernelGGL((cmp_factor_kernel<decltype(lr)::value>), dim3(c.G * c.K), dim3(CF_THREADS), 0, st,
                         (const float*)gpart, (n + GR_COLS - 1) / GR_COLS, c.sketch, coef);
    });
  };
  factor();
  apply_coef<true>(c, coef, X, c.sketch, n, tmp, gpart, st);
  factor();
  apply_coef<false>(c, coef, tmp, c.sketch, n, X, (float*)nullptr, st);
}

}  // namespace

extern "C" size_t cmoe_compress_workspace_bytes(const cmoe_compress_config* cfg) {
  return compress_cfg_ok(cfg) ? compress_layout(*cfg).total : 0;
}

extern "C" int cmoe_quantize_int4(const float* src, int64_t rows, int32_t L, int32_t q_group, uint8_t* codes,
                                  cmoe_f16* scales, void* stream) {
  if (rows < 0 || L <= 0 || q_group < 2 || q_group % 2 || L % q_group) return CMOE_ERR_INVALID_ARG;
  if (rows == 0) return CMOE_OK;
  if (!cptr_ok(src) || !cptr_ok(codes) || !cptr_ok(scales)) return CMOE_ERR_INVALID_ARG;
  (void)launch_quantize(src, (long)rows, L, q_group, nullptr, 1, codes, (half_t*)scales, (hipStream_t)stream);
  CP_CHECK();
  return CMOE_OK;
}

extern "C" int cmoe_reconstruction_error(const cmoe_compress_config* cfg, const cmoe_f16* W, const cmoe_f16* base,
                                         const uint8_t* u_q, const cmoe_f16* u_s, const uint8_t* v_q,
                                         const cmoe_f16* v_s, float* err, void* workspace, size_t workspace_bytes,
                                         void* stream) {
  if (!compress_cfg_ok(cfg)) return CMOE_ERR_UNSUPPORTED;
  if (!cptr_ok(W) || !cptr_ok(base) || !cptr_ok(u_q) || !cptr_ok(u_s) || !cptr_ok(v_q) || !cptr_ok(v_s) ||
      !cptr_ok(err) || !cptr_ok(workspace))
    return CMOE_ERR_INVALID_ARG;
  const CompressLayout L = compress_layout(*cfg);
  if (workspace_bytes < L.total) return CMOE_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  launch_error(*cfg, (const half_t*)W, (const half_t*)base, u_q, (const half_t*)u_s, v_q, (const half_t*)v_s,
               (float*)(ws + L.epart), 1, err, st);
  CP_CHECK();
  return CMOE_OK;
}

extern "C" int cmoe_compress(const cmoe_compress_config* cfg, const cmoe_f16* W, const cmoe_f16* omega,
                             cmoe_f16* base, uint8_t* u_q, cmoe_f16* u_s, uint8_t* v_q, cmoe_f16* v_s, float* report,
                             void* workspace, size_t workspace_bytes, void* stream) {
  if (!compress_cfg_ok(cfg)) return CMOE_ERR_UNSUPPORTED;
  if (!cptr_ok(W) || !cptr_ok(omega) || !cptr_ok(base) || !cptr_ok(u_q) || !cptr_ok(u_s) || !cptr_ok(v_q) ||
      !cptr_ok(v_s) || !cptr_ok(report) || !cptr_ok(workspace))
    return CMOE_ERR_INVALID_ARG;
  const cmoe_compress_config& c = *cfg;
  const CompressLayout L = compress_layout(c);
  if (workspace_bytes < L.total) return CMOE_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  const int E = c.G * c.K, l = c.sketch, out_d = c.out_dim, in_d = c.in_dim;
  const int tx = in_d / 64, ty = out_d / 64;
  half_t* D = (half_t*)(ws + L.D);
  half_t* XA = (half_t*)(ws + L.XA);
  half_t* XB = (half_t*)(ws + L.XB);
  float* coef = (float*)(ws + L.coef);
  double* stats = (double*)(ws + L.stats);
  double* lam = (double*)(ws + L.lam);
  int* gate = (int*)(ws + L.gate);
  float* UF = (float*)(ws + L.UF);
  float* VF = (float*)(ws + L.VF);

  // Eq. 6 and the residuals against the stored base
  hipLaunchKernelGGL(cmp_residual_kernel, dim3(tx, ty, c.G), dim3(256), 0, st, (const half_t*)W, c.K, out_d, in_d,
                     (half_t*)base, D, (float*)(ws + L.part));
  hipLaunchKernelGGL(cmp_stats_kernel, dim3(E), dim3(256), 0, st, (const float*)(ws + L.part), tx * ty * 4, stats);
  hipLaunchKernelGGL(cmp_tile_rows_kernel, dim3((in_d / 8 + 255) / 256, E * l), dim3(256), 0, st, (const half_t*)omega,
                     l, in_d, XA);
  CP_CHECK();
  float* gpart = (float*)(ws + L.gpart);
  // Q^T [l][out]: orthonormal rows spanning Delta Omega, refined by n_iter rounds of
  // Z = orth(Delta^T Q), Q = orth(Delta Z)
  half_t *cur = XA, *other = XB;   // rows of the last step, the other buffer
  auto step = [&](auto trans) {
    constexpr bool TRANS = decltype(trans)::value;
    stream_product<TRANS>(c, D, cur, other, gpart, st);
    orth_rows(c, TRANS ? in_d : out_d, other, cur, ws, L, st);
    half_t* o = cur;
    cur = other;
    other = o;
  };
  step(std::false_type{});
  for (int it = 0; it < c.n_iter; ++it) {
    step(std::true_type{});
    step(std::false_type{});
  }
  CP_CHECK();
  // B = Q^T Delta [l][in]; Rayleigh-Ritz: eigenvectors of B B^T pick the best rank-r pair inside the
  // sketch: U^T = C Q^T, V = C B with C = the r leading eigenvectors
  stream_product<true>(c, D, cur, other, gpart, st);
  for_rows(l, [&](auto lr) {
    hipLaunchKernelGGL((cmp_ritz_kernel<decltype(lr)::value>), dim3(E), dim3(CS_THREADS), 0, st, (const float*)gpart,
                       (in_d + GR_COLS - 1) / GR_COLS, l, c.r, coef, lam);
  });
  apply_coef<false>(c, coef, cur, c.r, out_d, UF, (float*)nullptr, st);
  apply_coef<false>(c, coef, other, c.r, in_d, VF, (float*)nullptr, st);
  // gate, quantisation (Sec. 3.4), and the error of the stored form
  hipLaunchKernelGGL(cmp_gate_kernel, dim3((E + 63) / 64), dim3(64), 0, st, (const double*)stats, (const double*)lam,
                     E, c.use_gate, c.gate_gamma, gate, report);
  (void)launch_quantize(UF, (long)E * c.r, out_d, c.q_group, gate, c.r, u_q, (half_t*)u_s, st);
  (void)launch_quantize(VF, (long)E * c.r, in_d, c.q_group, gate, c.r, v_q, (half_t*)v_s, st);
  launch_error(c, (const half_t*)W, (const half_t*)base, u_q, (const half_t*)u_s, v_q, (const half_t*)v_s,
               (float*)(ws + L.epart), 4, report, st);
  CP_CHECK();
  return CMOE_OK;
}
