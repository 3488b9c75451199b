// The middle of the backward pass (training step of Sec. 3.5): everything between the base products that
// enter the hidden layer (hb = B1 x, dab = B2^T dy, once per token) and those that leave it.  Per
// selected expert j of a token, with the rank parts added on the matrix cores:
//   h_j = hb + U1 t1_j, da_j = dab + V2^T uy_j               t1 = V1 x, uy = U2^T dy
//   a_j = GELU(h_j), dh_j = g_j da_j GELU'(h_j)              never written to memory
//   dhsum = sum_j dh_j (rows and transposed), agsum = sum_j g_j a_j (transposed): operands of the base products
//   q_j = U1^T dh_j, g_j s_j = V2 (g_j a_j), dg_j = da_j . a_j      partial sums per MD_N hidden units
//   dU1 += dh_j t1_j^T, dV2 += (g_j a_j) uy_j^T              accumulators over a run of tokens
// Written out as kernels of their own (ways back from rank space, activations, products into rank
// space, transposing copies, factor gradients) these steps moved 17 GB for 32768 tokens, two experts
// each, 8192 hidden units; here they read 1.1 and write 1.6 GB and the partial sums.
#include <type_traits>

#include "cmoe_device.h"

namespace {

constexpr int MD_N = 128;         // hidden units of a workgroup
constexpr int MD_M = 32;          // tokens of a tile
constexpr int MD_THREADS = 512;   // eight wavefronts: 4 x 2 of 32 hidden units x 16 tokens

// Phi(u) and exp(-u^2 / 2): the upper tail Phi(-|u|) = exp(-u^2 / 2) P(t), t = 1 / (1 + 0.32 |u|), P of degree 5
// fitted to 0.5 erfc(x / sqrt 2) exp(x^2 / 2) with weight (1 + x) exp(-x^2 / 2) on 0 <= x <= 7 (least
// squares, reweighted towards the largest error).  In FP32, with the reciprocal and the exponential up to an ulp off,
// |dPhi| < 3.2e-7 (2.2e-7 with both rounded correctly) and |d GELU'| < 3.4e-7; |d GELU| < 3.9e-7 where
// an erff leaves 4.5e-7 (|u| <= 9).  One reciprocal, one exponential and six FMAs serve the function and
// its derivative.
__device__ __forceinline__ void phi_exp(float u, float& phi, float& ex) {
  const float t = __builtin_amdgcn_rcpf(fmaf(0.32f, fabsf(u), 1.f));
  ex = __builtin_amdgcn_exp2f(u * u * -0.72134752044f);
  float p = fmaf(t, -0.129180768f, 0.493095306f);
  p = fmaf(t, p, -0.261299534f);
  p = fmaf(t, p, 0.311606895f);
  p = fmaf(t, p, 0.0808944892f);
  p = fmaf(t, p, 0.00488357156f);
  const float tail = ex * p;
  phi = u < 0.f ? tail : 1.f - tail;
}

// Or over the 16 lanes of a row (every lane gets it).
__device__ __forceinline__ unsigned row_or(unsigned v) {
  v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false);   // row_ror:8
  v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false);
  v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false);
  v |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false);
  return v;
}
// Per 16-bit element of 8: all ones where byte i of w equals e (e < 128), else zero.
__device__ __forceinline__ void match8(uint2 w, unsigned e, unsigned (&m)[4]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const unsigned v = (h ? w.y : w.x) ^ (e * 0x01010101u);
    const unsigned z = ~(((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u;   // 0x80 in the matching bytes
    const unsigned f = (z - (z >> 7)) | z;
    m[2 * h] = __builtin_amdgcn_perm(f, f, 0x01010000u);
    m[2 * h + 1] = __builtin_amdgcn_perm(f, f, 0x03030202u);
  }
}
__device__ __forceinline__ half8 and8(const half8& v, const unsigned (&m)[4]) {
  typedef unsigned uint4v __attribute__((ext_vector_type(4)));
  const uint4v x = __builtin_bit_cast(uint4v, v);
  return __builtin_bit_cast(half8, uint4v{x[0] & m[0], x[1] & m[1], x[2] & m[2], x[3] & m[3]});
}

// One workgroup: MD_N hidden units of one cluster and a run of its tokens in tiles of MD_M.  Phase 1 of a
// tile: a wavefront computes h, da, a, dh of its 32 units x 16 tokens (a lane owns a token and eight
// consecutive units, as in the forward epilogue) and leaves dh_j and g_j a_j as FP16 in LDS.  Phase 2: the
// products that contract over the units (q, s) and over the tokens (factor gradients) read them from
// there, the latter by transposing LDS reads.  The factor panels of the workgroup's units stay in LDS, the
// factor gradients in accumulators.
//   Phase 1 is bound by the vector ALUs (about 30 operations per unit and pair), phase 2 by chains of LDS
// reads and matrix instructions.  In one step of the loop every wavefront does phase 1 of a tile and
// phase 2 of the tile before it (staging twice, tables three times, one barrier), and the two wavefronts of
// a SIMD do them in opposite order, so that the one fills the gaps of the other.  32768 tokens, two of
// 8 x 8 experts of rank 16, 8192 units: 1.21-1.27 ms (1.38 with both in the same order; phase 1 alone 0.93), where
// the kernels it replaces took 3.4; vector ALUs issue in 0.67 of the cycles.
//   A rank part takes the 32 rank rows of a chunk at once, with zeros where a row is not of the token's expert. Where a
// panel holds an infinity or a NaN, 0 * Inf would reach the other experts' tokens: it is then taken expert by expert.
//   U panel [n][kr] and V panel [kr][n], staging [tensor][token][n]: 16-byte chunks at chunk ^ key of the
// row, keys such that both plain and transposing fragment reads spread over the banks.
template <int R, int K, int KRP>
__global__ __launch_bounds__(MD_THREADS) void bw_mid_kernel(bw_mid_args a, int G, int Ke, int KRp, int f, int run,
                                                           int n_chunks) {
  using FU = FusedUp<R, K>;
  constexpr int NSP = FU::NSP, PB = KRP / 16;             // passes of 16 rank rows per expert; passes
  constexpr int PER_CHUNK = 32 / R;                       // experts of a chunk of 32 rank rows
  constexpr int PER_GROUP = R >= 16 ? 1 : 16 / R;         // experts of a group of NSP passes
  constexpr int KR = K * R, PIECE = KR >= 8 ? 8 : 4, PIECES = MD_M * KR / PIECE;   // of t1, and as many of uy
  constexpr int U_BYTES = MD_N * KRP * 2, V_BYTES = KRP * MD_N * 2, S_BYTES = MD_M * MD_N * 2;
  static_assert(2 * PIECES <= MD_THREADS, "one piece per thread");
  __shared__ __attribute__((aligned(1024))) char smem[U_BYTES + V_BYTES + 2 * 2 * K * S_BYTES];
  __shared__ __attribute__((aligned(16))) half_t sT[3][2][MD_M][KR];
  __shared__ int sE[3][MD_M][K];
  __shared__ float sG[3][MD_M][K];
  __shared__ __attribute__((aligned(8))) unsigned char sB[3][K][MD_M];   // the experts, 255 for rows past the run
  __shared__ float sD[2][4][MD_M][K];
  __shared__ unsigned sM[2][2][K];   // experts of a 16-token block
  __shared__ int sApart[MD_THREADS / 64];   // a panel value that the wavefront loaded is not finite
  char *sU = smem, *sV = smem + U_BYTES, *sS = sV + V_BYTES;
  const int tid = threadIdx.x, lane = tid & 63, t16 = lane & 15, q = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), cg = wave & 3, hi = wave >> 2;
  const int chunk = blockIdx.x % n_chunks, slot = blockIdx.x / n_chunks;
  int c, m0, m_end;
  if (!find_tile(a.offsets, G, run, slot, c, m0, m_end)) return;
  m_end = min(m_end, m0 + run);
  const int T = a.T, n0 = chunk * MD_N, nblk = min(MD_N / 32, (f - n0) / 32);
  const int col0 = a.krange[2 * c] + (m0 - a.offsets[c]);   // of the transposed copies
  auto key_u = [](int n) { const int i = (n & 3) | ((n >> 1) & 12); return KRP == 128 ? i : i >> 1; };

  // factor panels, zero rows for experts without a token
  {
    bool bad = false;
    const int cpr = KRp / 8;
    for (int i = tid; i < nblk * 32 * cpr; i += MD_THREADS) {
      const int n = i / cpr, ch = i % cpr;
      half8 v = *(const half8*)(a.u1t + ((size_t)c * f + n0 + n) * KRp + ch * 8);
#pragma unroll
      for (int h = 0; h < 8; h += 4) {
        const int e = c * Ke + min((ch * 8 + h) / R, Ke - 1);
        if (a.offe[e + 1] == a.offe[e]) v[h] = v[h + 1] = v[h + 2] = v[h + 3] = (half_t)0.f;
      }
      bad |= not_finite(v);
      *(half8*)(sU + n * (KRP * 2) + ((ch ^ key_u(n)) << 4)) = v;
    }
    for (int i = tid; i < KRp * nblk * 4; i += MD_THREADS) {
      const int kr = i / (nblk * 4), ch = i % (nblk * 4), e = c * Ke + min(kr / R, Ke - 1);
      half8 v = *(const half8*)(a.v2p + ((size_t)c * KRp + kr) * f + n0 + ch * 8);
      if (a.offe[e + 1] == a.offe[e]) v = half8{0, 0, 0, 0, 0, 0, 0, 0};
      bad |= not_finite(v);
      *(half8*)(sV + kr * (MD_N * 2) + ((ch ^ (kr & 15)) << 4)) = v;
    }
    const bool any = __ballot(bad) != 0ull;
    if (lane == 0) sApart[wave] = any;
  }

  const size_t block = (size_t)((n0 >> 5) + min(cg, nblk - 1)) * T * 32;   // this wavefront's 32 units in [f / 32][T][32]

  // A tile's rank-space rows, experts and gates (one piece per thread) and base parts, loaded a tile ahead
  // (rows past the end repeat the last).
  typedef _Float16 piece_t __attribute__((ext_vector_type(PIECE)));
  piece_t tp;
  int te;
  float tg;
  half8 hv, dv;
  auto load_tile = [&](int mt) {
    {
      const int g = tid / PIECES & 1, w = tid % PIECES;
      const unsigned p = min(mt + w / (KR / PIECE), T - 1);
      tp = *(const piece_t*)((g ? a.uy : a.t1) + (size_t)(p * KR + w % (KR / PIECE) * PIECE));
    }
    const unsigned i = min(mt + tid % (MD_M * K) / K, m_end - 1) * K + tid % K;
    te = a.es[i];
    tg = a.gs[i];
    const unsigned at = (unsigned)min(mt + 16 * hi + t16, m_end - 1) * 32u + 8u * q;
    hv = *(const half8*)(a.hb + block + at);
    dv = *(const half8*)(a.dab + block + at);
  };
  auto store_table = [&](int mt, int buf) {
    if (tid < 2 * PIECES) *(piece_t*)(&sT[buf][0][0][0] + tid * PIECE) = tp;
    if (tid < MD_M * K) {
      sE[buf][tid / K][tid % K] = te;
      sB[buf][tid % K][tid / K] = mt + tid / K < m_end ? (unsigned char)te : 255;
      sG[buf][tid / K][tid % K] = tg;
    }
  };
  const half8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};

  // ---------------------------------------------------------------- phase 1
  // apart: the experts of a chunk of rank rows one by one
  auto phase1 = [&](int mt, int buf, int par, auto apart) __attribute__((always_inline)) {
    const half8 h8 = hv, d8 = dv;
    load_tile(mt + MD_M);
    if (cg < nblk) {
      char* stage = sS + par * (2 * K * S_BYTES);   // dh_0, g_0 a_0, dh_1, g_1 a_1
      const int tl = 16 * hi + t16;
      const int own = tl * (MD_N * 2) + (((4 * cg + q) ^ t16) << 4);   // this lane's 16 bytes of a staging tensor
      const bool valid = mt + tl < m_end;
      float dhs[8], ags[8];
      half8 dh_last, ga_last;
#pragma unroll
      for (int j = 0; j < K; ++j) {
        const int e = sE[buf][tl][j];
        const float g = sG[buf][tl][j];
        const unsigned em = __builtin_amdgcn_readfirstlane(row_or(valid ? 1u << e : 0u));
        if (cg == 0 && lane == 0) sM[par][hi][j] = em;
        half8 ft = zero8, fu = zero8;   // this lane's slices of t1_j and uy_j
        if constexpr (R == 4) {
          const half4 x = *(const half4*)&sT[buf][0][tl][j * R], y = *(const half4*)&sT[buf][1][tl][j * R];
          ft = join8(x, x);
          fu = join8(y, y);
        } else {
          const int at = j * R + (R == 32 ? 8 * q : R == 16 ? 8 * (q & 1) : 0);
          ft = *(const half8*)&sT[buf][0][tl][at];
          fu = *(const half8*)&sT[buf][1][tl][at];
        }
        float4v h[2], z[2];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          h[0][v] = (float)h8[v];
          h[1][v] = (float)h8[4 + v];
          z[0][v] = (float)d8[v];
          z[1][v] = (float)d8[4 + v];
        }
        auto frag_u = [&](int ch, int hh) {
          const int n = 32 * cg + ((t16 & 12) << 1) + 4 * hh + (t16 & 3);
          return *(const half8*)(sU + n * (KRP * 2) + (((4 * ch + q) ^ key_u(n)) << 4));
        };
        auto frag_v = [&](int ch, int hh) {
          const int kr = 32 * ch + 8 * q + (t16 >> 2);
          const char* v0 = sV + kr * (MD_N * 2) + (((4 * cg + (t16 & 3)) ^ (kr & 15)) << 4) + 8 * hh;
          const char* v1 = sV + (kr + 4) * (MD_N * 2) + (((4 * cg + (t16 & 3)) ^ ((kr + 4) & 15)) << 4) + 8 * hh;
          return join8(lds_read_tr(v0), lds_read_tr(v1));
        };
        if constexpr (!decltype(apart)::value) {
          for (unsigned m = em; m != 0u;) {
            const int ch = __builtin_ctz(m) / PER_CHUNK;
            m &= ~(((1u << PER_CHUNK) - 1u) << (ch * PER_CHUNK));
            const half8 ft1 = FU::t1_frag(e, ch, q, ft), fu1 = FU::t1_frag(e, ch, q, fu);
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
              h[hh] = mfma32(frag_u(ch, hh), ft1, h[hh]);
              z[hh] = mfma32(frag_v(ch, hh), fu1, z[hh]);
            }
          }
        } else {
          for (unsigned m = em; m != 0u; m &= m - 1u) {
            const int x = __builtin_ctz(m), ch = x / PER_CHUNK, kr = 32 * ch + 8 * q;
            const half8 ft1 = FU::t1_frag(e, ch, q, ft), fu1 = FU::t1_frag(e, ch, q, fu);
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
              const float4v hx = mfma32(rows_of_expert(frag_u(ch, hh), kr, R, x), ft1, h[hh]);
              const float4v zx = mfma32(rows_of_expert(frag_v(ch, hh), kr, R, x), fu1, z[hh]);
              if (e == x) h[hh] = hx, z[hh] = zx;
            }
          }
        }
        float dot = 0.f;
        half8 dh8, ga8;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float u = h[i >> 2][i & 3], y = z[i >> 2][i & 3];
          float phi, ex;
          phi_exp(u, phi, ex);
          const float av = u * phi, dg = fmaf(u * 0.3989422804014327f, ex, phi);
          const float dh = g * y * dg, ga = g * av;
          dot = fmaf(y, av, dot);
          dhs[i] = j == 0 ? dh : dhs[i] + dh;
          ags[i] = j == 0 ? ga : ags[i] + ga;
          dh8[i] = (half_t)dh;
          ga8[i] = (half_t)ga;
        }
        dot += __shfl_xor(dot, 16, 64);
        dot += __shfl_xor(dot, 32, 64);
        if (q == 0) sD[par][cg][tl][j] = dot;
        if (!valid) dh8 = ga8 = zero8;
        if (j + 1 < K) {
          *(half8*)(stage + 2 * j * S_BYTES + own) = dh8;
          *(half8*)(stage + (2 * j + 1) * S_BYTES + own) = ga8;
        } else {
          dh_last = dh8;
          ga_last = ga8;
        }
        __builtin_amdgcn_sched_barrier(0);   // one pair's values live at a time
      }
      half8 dhs8, ags8;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        dhs8[i] = (half_t)dhs[i];
        ags8[i] = (half_t)ags[i];
      }
      if (!valid) dhs8 = ags8 = zero8;
      // the sums leave transposed, through this wavefront's part of the last expert's tensors: lane (t16, q)
      // takes unit 16 (q / 2) + t16 and tokens 8 (q % 2) ..
      char* last = stage + (2 * K - 2) * S_BYTES;
      *(half8*)(last + own) = dhs8;
      *(half8*)(last + S_BYTES + own) = ags8;
      wave_lds_order();
      half4 tr[2][2];
#pragma unroll
      for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int t2 = 16 * hi + 8 * (q & 1) + 4 * u + (t16 >> 2);
          tr[w][u] = lds_read_tr(last + w * S_BYTES + t2 * (MD_N * 2) +
                                 (((4 * cg + (q & 2) + ((t16 & 3) >> 1)) ^ (t2 & 15)) << 4) + 8 * (t16 & 1));
        }
      wave_lds_order();
      *(half8*)(last + own) = dh_last;
      *(half8*)(last + S_BYTES + own) = ga_last;
      if (valid) *(half8*)(a.dhsum + block + ((unsigned)(mt + tl) * 32u + 8u * q)) = dhs8;
      const size_t at = ((size_t)((col0 + (mt - m0)) >> 5) * f + n0 + 32 * cg) * 32 +
                        (unsigned)((16 * (q >> 1) + t16) * 32 + 16 * hi + 8 * (q & 1));
      *(half8*)(a.dhst + at) = join8(tr[0][0], tr[0][1]);
      *(half8*)(a.agt + at) = join8(tr[1][0], tr[1][1]);
    }
  };

  // ---------------------------------------------------------------- phase 2
  float4v acc[PB][2];
#pragma unroll
  for (int i = 0; i < PB; ++i) acc[i][0] = acc[i][1] = float4v{0.f, 0.f, 0.f, 0.f};
  auto phase2 = [&](int mt, int buf, int par) __attribute__((always_inline)) {
    const char* stage = sS + par * (2 * K * S_BYTES);
    // over the hidden units: token block wave % 2, q or s by the next bit, expert hi
    if (hi < K) {
      const int tb = wave & 1, which = (wave >> 1) & 1, j = hi;
      const int tl = 16 * tb + t16, p = mt + tl;
      const int e = sE[buf][tl][j];
      half8 fb[MD_N / 32];
#pragma unroll
      for (int nb = 0; nb < MD_N / 32; ++nb)
        if (nb < nblk)
          fb[nb] = *(const half8*)(stage + (2 * j + which) * S_BYTES + tl * (MD_N * 2) + (((4 * nb + q) ^ t16) << 4));
      float4v sel[NSP];
#pragma unroll
      for (int s = 0; s < NSP; ++s) sel[s] = float4v{0.f, 0.f, 0.f, 0.f};
      for (unsigned m = __builtin_amdgcn_readfirstlane(sM[par][tb][j]); m != 0u;) {
        const int pg = __builtin_ctz(m) / PER_GROUP;
        m &= ~(((1u << PER_GROUP) - 1u) << (pg * PER_GROUP));
#pragma unroll
        for (int s = 0; s < NSP; ++s) {
          const int pp = pg * NSP + s;
          half8 fa[MD_N / 32];
#pragma unroll
          for (int nb = 0; nb < MD_N / 32; ++nb) {
            if (nb >= nblk) continue;
            if (which == 0) {
              half4 v[2];
#pragma unroll
              for (int u = 0; u < 2; ++u) {
                const int n = 32 * nb + 8 * q + 4 * u + (t16 >> 2);
                v[u] = lds_read_tr(sU + n * (KRP * 2) + (((2 * pp + ((t16 & 3) >> 1)) ^ key_u(n)) << 4) + 8 * (t16 & 1));
              }
              fa[nb] = join8(v[0], v[1]);
            } else {
              fa[nb] = *(const half8*)(sV + (16 * pp + t16) * (MD_N * 2) + (((4 * nb + q) ^ t16) << 4));
            }
          }
          float4v d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int nb = 0; nb < MD_N / 32; ++nb)
            if (nb < nblk) d = mfma32(fa[nb], fb[nb], d);
          // a token keeps the rows of its own expert's passes
          const bool mine = pg == e / PER_GROUP;
#pragma unroll
          for (int v = 0; v < 4; ++v) sel[s][v] = mine ? d[v] : sel[s][v];
        }
      }
      const int be = (e * R) & 15, row0 = 4 * q;   // first row of the expert inside its pass; this lane's rows
      if (p < m_end && row0 >= be && row0 < be + (R < 16 ? R : 16)) {
        float* dst = (which ? a.spart : a.qpart) + (size_t)chunk * T * KR + ((unsigned)p * KR + (unsigned)(j * R + row0 - be));
#pragma unroll
        for (int s = 0; s < NSP; ++s) *(float4v*)(dst + 16 * s) = sel[s];
      }
    }
    if (tid < MD_M * K && mt + tid / K < m_end) {
      const float* d = &sD[par][0][tid / K][tid % K];
      float sum = d[0];
      for (int w = 1; w < nblk; ++w) sum += d[w * MD_M * K];
      a.dotp[(size_t)chunk * T * K + (unsigned)(mt * K + tid)] = sum;
    }
    // over the tokens, units 32 cg ..: hi == 0 dU1 from dh_j and t1_j, hi == 1 dV2 from g_j a_j and uy_j.  Expert by
    // expert, both operands cut to the expert's tokens: a value that is not finite stays with its expert.
    if (cg < nblk) {
#pragma unroll 1
      for (int j = 0; j < K; ++j) {
        const unsigned em = __builtin_amdgcn_readfirstlane(sM[par][0][j] | sM[par][1][j]);
        const uint2 ew = *(const uint2*)&sB[buf][j][8 * q];
        half8 fa[2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          half4 v[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int tl = 8 * q + 4 * u + (t16 >> 2);
            v[u] = lds_read_tr(stage + (2 * j + hi) * S_BYTES + tl * (MD_N * 2) +
                               (((4 * cg + (t16 & 3)) ^ (tl & 15)) << 4) + 8 * hh);
          }
          fa[hh] = join8(v[0], v[1]);
        }
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
          constexpr unsigned few = (1u << PER_GROUP) - 1u;
          const int e0 = pb / NSP * PER_GROUP;
          for (unsigned m = (em >> e0) & few; m != 0u; m &= m - 1u) {
            const int sub = __builtin_ctz(m);
            unsigned keep[4];
            match8(ew, (unsigned)(e0 + sub), keep);
            const half8 a0 = and8(fa[0], keep), a1 = and8(fa[1], keep);
            const int rho = (R == 32 ? 16 * (pb & 1) : 0) + ((4 * (t16 & 3)) & (R - 1) & 15);
            half4 v[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) v[u] = lds_read_tr(&sT[buf][hi][8 * q + 4 * u + (t16 >> 2)][j * R + rho]);
            const half8 fb = and8(join8(v[0], v[1]), keep);
            if constexpr (R >= 16) {
              acc[pb][0] = mfma32(a0, fb, acc[pb][0]);
              acc[pb][1] = mfma32(a1, fb, acc[pb][1]);
            } else {   // only the columns of the pass that are the expert's
              const float4v zero = {0.f, 0.f, 0.f, 0.f}, d0 = mfma32(a0, fb, zero), d1 = mfma32(a1, fb, zero);
              if (t16 / R == sub) acc[pb][0] += d0, acc[pb][1] += d1;
            }
          }
        }
      }
    }
  };

  load_tile(m0);
  store_table(m0, 0);
  __syncthreads();
  const int tiles = (m_end - m0 + MD_M - 1) / MD_M;
  // tables: tile i in buffer i % 3
  auto steps = [&](auto first, auto apart) __attribute__((always_inline)) {
    for (int i = 0, buf = 0, prev = 0; i < tiles; ++i) {
      const int mt = m0 + i * MD_M, next = buf == 2 ? 0 : buf + 1;
      if (decltype(first)::value) phase1(mt, buf, i & 1, apart);
      if (i > 0) phase2(mt - MD_M, prev, (i - 1) & 1);
      if (!decltype(first)::value) phase1(mt, buf, i & 1, apart);
      store_table(mt + MD_M, next);
      prev = buf;
      buf = next;
      __syncthreads();
    }
  };
  // (a branch inside the loop made the kernel 3 % slower)
  if (__ballot(lane < MD_THREADS / 64 && sApart[lane % (MD_THREADS / 64)] != 0) != 0ull) steps(std::false_type{}, std::true_type{});
  else if (hi == 0) steps(std::true_type{}, std::false_type{});
  else steps(std::false_type{}, std::false_type{});
  phase2(m0 + (tiles - 1) * MD_M, (tiles - 1) % 3, (tiles - 1) & 1);
  if (cg >= nblk) return;
  float* out = (hi ? a.dv : a.du) + (size_t)slot * KRp * f + n0 + 32 * cg + 8 * q;
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const int kr = 16 * pb + t16;
    if (kr >= KRp) continue;
    *(float4v*)(out + (size_t)kr * f) = acc[pb][0];
    *(float4v*)(out + (size_t)kr * f + 4) = acc[pb][1];
  }
}

// The partial q and g s of the pairs summed over the chunks of hidden units, in order: q16 [p][j][rho] (tile
// order, operand of the input gradient), qq / ss (32 columns per pair, pair rows sorted by expert), and the softmax
// backward over the selected logits (Eq. 10) from the summed dg: dl_j = g_j (dg_j - sum_i g_i dg_i).  A
// workgroup owns 256 consecutive values (four per lane); its four wavefronts take every fourth chunk.
constexpr int MS_WAVES = 4;
template <int K>
__global__ __launch_bounds__(64 * MS_WAVES) void bw_mid_sum_kernel(bw_mid_args a, int n_chunks, int r,
                                                                   const int* __restrict__ perm2,
                                                                   const int* __restrict__ invm, half_t* __restrict__ q16,
                                                                   half_t* __restrict__ qq, half_t* __restrict__ ss,
                                                                   float* __restrict__ dl) {
  __shared__ float4v part[2][MS_WAVES][64];
  __shared__ float dpart[MS_WAVES][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, kr = K * r;
  const size_t total = (size_t)a.T * kr, idx = ((size_t)blockIdx.x * 64 + lane) * 4;
  const size_t p0 = (size_t)blockIdx.x * 256 / kr;   // first token: 256 is a multiple of k r
  const int toks = 256 / kr;
  float4v sq = {0.f, 0.f, 0.f, 0.f}, sv = sq;
  float sd = 0.f;
  const bool in = idx < total, dots = lane < toks * K && p0 + lane / K < (size_t)a.T;
#pragma unroll 4
  for (int ch = wave; ch < n_chunks; ch += MS_WAVES) {
    if (in) {
      sq += *(const float4v*)(a.qpart + (size_t)ch * total + idx);
      sv += *(const float4v*)(a.spart + (size_t)ch * total + idx);
    }
    if (dots) sd += a.dotp[((size_t)ch * a.T + p0) * K + lane];
  }
  part[0][wave][lane] = sq;
  part[1][wave][lane] = sv;
  dpart[wave][lane] = sd;
  __syncthreads();
  if (wave < 2 && in) {
    float4v s = part[wave][0][lane];
#pragma unroll
    for (int w = 1; w < MS_WAVES; ++w) s += part[wave][w][lane];
    const half4 h = {(half_t)s[0], (half_t)s[1], (half_t)s[2], (half_t)s[3]};
    const size_t p = idx / kr;
    const int w = (int)(idx % kr), j = w / r, rho = w % r;
    const size_t m = invm[(size_t)perm2[p] * K + j];
    *(half4*)((wave ? ss : qq) + m * 32 + rho) = h;
    if (wave == 0) *(half4*)(q16 + idx) = h;
  } else if (wave == 2 && dots) {
    const size_t p = p0 + lane / K;
    float dg[K], mean = 0.f, g[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const int l = lane / K * K + j;
      dg[j] = ((dpart[0][l] + dpart[1][l]) + dpart[2][l]) + dpart[3][l];
      g[j] = a.gs[p * K + j];
      mean += g[j] * dg[j];
    }
#pragma unroll
    for (int j = 0; j < K; ++j)
      if (lane % K == j) dl[(size_t)perm2[p] * K + j] = g[j] * (dg[j] - mean);
  }
}

// out[e][rho][n] = sum over the runs of the expert's cluster, in order, of part[run][j r + rho][n].
// Block (ceil(f / 1024), G K r, 2): dU1, dV2.
__global__ __launch_bounds__(256) void bw_mid_grad_kernel(bw_mid_args a, int G, int Ke, int r, int KRp, int f, int run,
                                                          float* __restrict__ du1, float* __restrict__ dv2) {
  const int er = blockIdx.y, e = er / r, c = e / Ke, n = (blockIdx.x * 256 + threadIdx.x) * 4;
  const RowTiles rt(a.offsets, G, run);
  const int s0 = rt.first_tile(c), s1 = rt.end_tile(c);
  if (n >= f) return;
  const float* src = (blockIdx.z ? a.dv : a.du) + ((size_t)s0 * KRp + (e % Ke) * r + er % r) * f + n;
  const size_t step = (size_t)KRp * f;
  float4v s = {0.f, 0.f, 0.f, 0.f};
  for (int i = 0; i < s1 - s0; i += 8) {
    float4v v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i + u < s1 - s0) v[u] = *(const float4v*)(src + (i + u) * step);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i + u < s1 - s0) s += v[u];
  }
  *(float4v*)((blockIdx.z ? dv2 : du1) + (size_t)er * f + n) = s;
}

template <int R, int K, int KRP>
void go_mid(const cmoe_dims& dm, const bw_mid_args& a, hipStream_t st) {
  hipLaunchKernelGGL((bw_mid_kernel<R, K, KRP>), dim3((unsigned)(bw_mid_chunks(dm) * bw_mid_slots(dm, a.T))),
                     dim3(MD_THREADS), 0, st, a, dm.G, dm.K, dm.KRp, dm.d_ff, bw_mid_run(dm, a.T), bw_mid_chunks(dm));
}
template <int R>
void go_mid_r(const cmoe_dims& dm, const bw_mid_args& a, hipStream_t st) {
  if (dm.k == 1) {
    if (dm.KRp <= 64) go_mid<R, 1, 64>(dm, a, st); else go_mid<R, 1, 128>(dm, a, st);
  } else {
    if (dm.KRp <= 64) go_mid<R, 2, 64>(dm, a, st); else go_mid<R, 2, 128>(dm, a, st);
  }
}

}  // namespace

int bw_mid_chunks(const cmoe_dims& dm) { return (dm.d_ff + MD_N - 1) / MD_N; }
// Runs such that about 1024 workgroups share the tokens, in whole tiles.
constexpr int MD_WORKGROUPS = 1024;
int bw_mid_run(const cmoe_dims& dm, int T) {
  const long want = (long)T * bw_mid_chunks(dm) / MD_WORKGROUPS;
  return (int)((want < 1 ? 1 : want) + MD_M - 1) / MD_M * MD_M;
}
int bw_mid_slots(const cmoe_dims& dm, int T) {
  const int run = bw_mid_run(dm, T);
  return (T + run - 1) / run + dm.G;
}
// Runs to reserve space for: no T up to this one has more.  A run of m tiles holds want < 32 m + 1, so T / run is
// below 33 / 32 of 1024 / chunks, and it is never more than the tiles.
int bw_mid_slots_room(const cmoe_dims& dm, int T) {
  const int chunks = bw_mid_chunks(dm), tiles = (T + MD_M - 1) / MD_M;
  const int most = (MD_WORKGROUPS + MD_WORKGROUPS / MD_M + chunks - 1) / chunks;
  return (tiles < most ? tiles : most) + dm.G;
}

hipError_t launch_bw_mid(const cmoe_dims& dm, const bw_mid_args& a, hipStream_t st) {
  switch (dm.r) {
    case 4: go_mid_r<4>(dm, a, st); break;
    case 8: go_mid_r<8>(dm, a, st); break;
    case 16: go_mid_r<16>(dm, a, st); break;
    default: go_mid_r<32>(dm, a, st); break;
  }
  return hipGetLastError();
}

// What remains of the partial sums of launch_bw_mid: q, s and the gate path, and the factor gradients.
hipError_t launch_bw_mid_sums(const cmoe_dims& dm, const bw_mid_args& a, const int* perm2, const int* invm, half_t* q16,
                              half_t* qq, half_t* ss, float* dl, float* du1, float* dv2, hipStream_t st) {
  const int chunks = bw_mid_chunks(dm), kr = dm.k * dm.r;
  const dim3 grid((unsigned)(((size_t)a.T * kr + 255) / 256)), block(64 * MS_WAVES);
  if (dm.k == 1)
    hipLaunchKernelGGL(bw_mid_sum_kernel<1>, grid, block, 0, st, a, chunks, dm.r, perm2, invm, q16, qq, ss, dl);
  else
    hipLaunchKernelGGL(bw_mid_sum_kernel<2>, grid, block, 0, st, a, chunks, dm.r, perm2, invm, q16, qq, ss, dl);
  hipLaunchKernelGGL(bw_mid_grad_kernel, dim3((dm.d_ff + 1023) / 1024, dm.G * dm.K * dm.r, 2), dim3(256), 0, st, a, dm.G,
                     dm.K, dm.r, dm.KRp, dm.d_ff, bw_mid_run(dm, a.T), du1, dv2);
  return hipGetLastError();
}
