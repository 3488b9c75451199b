// Device-side building blocks shared by the matrix-core kernels.
#pragma once

#include "cmoe_internal.h"

namespace {

__device__ __forceinline__ float16v mfma16(half8 a, half8 b, float16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// GELU(u) = u Phi(u) in the erf form = max(u, 0) - a Q(a), a = |u|, Q(a) = 1 - Phi(a): a polynomial of degree 8 in a on
// [0, 4], zero to the bit at 4 (the constant is -4 times what is added to it), and a held at 4 beyond.  The minimum keeps a NaN.
// Eleven full-rate operations per element.
//   Error against 64 bits, of this / of u Phi by seven coefficients in u^2 with u clamped to 3.75 (twelve operations) / of the
// same with Phi saturated instead of u (ten): largest for |u| < 3 8.6e-5 / 1.7e-4 / 1.4e-4, for any |u| 1.3e-4 (at 3.8) /
// 3.3e-4 and growing with u / 3.7e-4 (at 3.72); RMS under a Gaussian of deviation 0.25 7.6e-6 / 1.2e-5 / 1.3e-5, of 1 2.0e-5 /
// 4.0e-5 / 2.9e-5, of 2 3.7e-5 / 7.6e-5 / 6.9e-5; the RMS of no quarter of a unit of |u| is above 1.004 of the smaller
// of theirs.
// Fitted to a Q(a) with each quarter weighted by the smaller of their two errors.  Against the ten operations the layer's forward
// pass takes 64.8 -> 65.9 us (777 tokens of 4 clusters of 1024 x 4096), 392 -> 398 (16384 Zipf tokens of those), 2419 -> 2434
// (32768 of 8 of 2048 x 8192).
__device__ __forceinline__ float gelu_erf(float u) {
  const float a = __builtin_elementwise_minimum(fabsf(u), 4.f);
  float p = fmaf(a, 6.229498831e-05f, -1.057959977e-03f);
  p = fmaf(a, p, 6.718921941e-03f);
  p = fmaf(a, p, -1.702310517e-02f);
  p = fmaf(a, p, -2.335787285e-03f);
  p = fmaf(a, p, 7.805491239e-02f);
  p = fmaf(a, p, -9.440604597e-03f);
  p = fmaf(a, p, -3.960606754e-01f);
  p = fmaf(a, p, 4.997466803e-01f);
  return fmaf(-a, p, __builtin_elementwise_maximum(u, 0.f));
}
// One value each from here on: a conversion to FP16 would otherwise become a second form of the last operation, with all three
// operands of every element kept for the first (up to 52 registers spilled, 1 % of the whole forward pass).
__device__ __forceinline__ void settle(float (&a)[8]) {
  asm("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]));
}

__device__ __forceinline__ half4 to_half4(const float16v& a, int qd) {
  half4 o;
  o[0] = (half_t)a[4 * qd + 0];
  o[1] = (half_t)a[4 * qd + 1];
  o[2] = (half_t)a[4 * qd + 2];
  o[3] = (half_t)a[4 * qd + 3];
  return o;
}


// ---------------------------------------------------------------- 16 x 16 x 32 blocks
// The grouped products run on v_mfma_f32_16x16x32_f16: D (16 rows x 16 tokens, FP32) +=
// A (16 weight rows x 32 contraction elements) * B (32 x 16 tokens).  Lane l supplies row
// (or token) l % 16 and the eight contraction elements 8q .. 8q + 7, q = l / 16, and holds of
// D the token l % 16 and the rows 4q .. 4q + 3.  Measured on this part, the instruction
// sustains about 14 % more flops than the 32 x 32 x 16 form at the same board power (it moves
// half the accumulator bytes per flop), and board power is what limits the products.
//
// Weight rows are taken in "pair blocks" of 32 consecutive rows = two MFMA blocks.  Row i of
// block hh (0 or 1) of a pair block is the weight row 8 (i / 4) + 4 hh + i % 4 of the pair
// block, so that a lane's 4 + 4 accumulators of the two blocks are the EIGHT CONSECUTIVE rows
// 8q .. 8q + 7: a lane stores 16 contiguous bytes of FP16 output per token, four lanes a
// token's 64-byte line, and an accumulator pair is a ready-made B operand (contraction
// positions in natural order) for a further product.
__device__ __forceinline__ float4v mfma32(half8 a, half8 b, float4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// Weight row (offset inside its 32-row pair block kept in the upper bits) held by tile row rho
// of an LDS operand tile whose rows are stored in MFMA order: rho = 32 P + 16 hh + i.
__device__ __forceinline__ int pi_row(int rho) {
  return (rho & ~31) | ((rho & 12) << 1) | ((rho & 16) >> 2) | (rho & 3);
}

// Position (XOR mask over the four 16-byte chunks of a 64-byte operand-tile row) at which
// tile row `row` keeps its chunks.  A 16x16x32 fragment read has lane l fetch 16 bytes of row
// l % 16, chunk l / 16; the LDS serves such a read in groups of sixteen lanes
// {0-3, 12-15, 20-23, 24-27} and {4-7, 8-11, 16-19, 28-31} (and the same plus 32), so the
// four row quads of one group need four different chunk positions: quads 0,1,2,3 use
// masks 0,3,2,1.  Measured on gfx950: the plain mask (row >> 2) & 3 serves a 32-row fragment
// read without conflicts but gives two-way conflicts on every 16-row read.
__device__ __forceinline__ int swz(int row) { return ((row >> 2) & 3) ^ ((row >> 1) & 2); }

// One 1-KiB direct-to-LDS load: lane l's 16 bytes land at lds_byte + 16 l.  The hardware asks for
// one wait state between a scalar write of M0 and a load that goes to LDS through it, and the
// compiler adds none inside an asm block: without the s_nop a load may still use the old M0.
__device__ __forceinline__ void dma16(const void* g, unsigned lds_byte) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(lds_byte) : "memory");
}
// 256 bytes: lane l's 4 bytes land at lds_byte + 4 l.
__device__ __forceinline__ void dma4(const void* g, unsigned lds_byte) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(g), "s"(lds_byte) : "memory");
}
// dma16 with the non-temporal hint: the line is not kept in the caches behind the load.
// For a matrix that is read once per call and is larger than the last-level cache this is
// worth 9 % of the whole weight-streaming path (the two base streams go from 6.0 to 6.5-6.7
// TB/s, and the router, whose rows and tokens are no longer evicted, gets faster too).
__device__ __forceinline__ void dma16_nt(const void* g, unsigned lds_byte) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(g), "s"(lds_byte) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// LDS reads and writes of this wavefront completed.  A bare barrier does not imply it: before a
// stage that was read is refilled by loads that go to LDS, or what was written is read by others.
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Transposing LDS read of 16-bit elements: the 16 lanes of a group (l / 16) read a 4 x 16 matrix, lane i
// the four consecutive elements 4 (i % 4) .. of matrix row i / 4 at its own address p, and lane i
// gets column i, element u of the result being row u.  Two of them make a matrix-core operand of a
// tile stored with the contraction index along its rows.
__device__ __forceinline__ half4 lds_read_tr(const void* p) {
  typedef short s4 __attribute__((__vector_size__(4 * sizeof(short))));
  return __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                       (__attribute__((address_space(3))) s4*)(__attribute__((address_space(3))) void*)p));
}
__device__ __forceinline__ half8 join8(const half4& a, const half4& b) {
  return half8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
}
// Does an element hold an infinity or a NaN?
__device__ __forceinline__ bool not_finite(const half8& v) {
  typedef unsigned uint4v __attribute__((ext_vector_type(4)));
  const uint4v x = __builtin_bit_cast(uint4v, v);
  unsigned m = 0u;
#pragma unroll
  for (int i = 0; i < 4; ++i) m |= (x[i] & 0x7c007c00u) + 0x04000400u;
  return (m & 0x80008000u) != 0u;
}
// Of the rank rows kr .. kr + 7 of a cluster (kr a multiple of 8) those of expert e; zero for the others.
__device__ __forceinline__ half8 rows_of_expert(const half8& v, int kr, int r, int e) {
  const half4 z = {0, 0, 0, 0};
  return join8(kr / r == e ? half4{v[0], v[1], v[2], v[3]} : z, (kr + 4) / r == e ? half4{v[4], v[5], v[6], v[7]} : z);
}
// What this wavefront wrote to LDS is read by its own lanes behind this (no barrier needed).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Ranking key of a logit: a NaN ranks below every number (as -inf), so that the selections of the
// router always return distinct, valid slots whatever the input holds.
__device__ __forceinline__ float rank_key(float v) { return v == v ? v : -INFINITY; }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
// The two INT4 codes of a byte (even element in the low nibble), and the dot product of eight codes (a
// word) with eight values, in element order.
__device__ __forceinline__ float nib_lo(unsigned b) { return (float)((int)(b << 28) >> 28); }
__device__ __forceinline__ float nib_hi(unsigned b) { return (float)((int)(b << 24) >> 28); }
__device__ __forceinline__ float code_dot8(unsigned word, const half8& x) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned b = (word >> (8 * i)) & 0xffu;
    s = fmaf(nib_lo(b), (float)x[2 * i], s);
    s = fmaf(nib_hi(b), (float)x[2 * i + 1], s);
  }
  return s;
}

// Inclusive sum over the lanes of a wavefront by data-parallel-primitive moves (no LDS round
// trips): rows of 16 lanes by shifts, then the row totals broadcast upwards.
__device__ __forceinline__ int wave_inclusive_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

// Row tiles of bm rows that never straddle a group, dealt group after group.  offsets
// [n_groups + 1], at most MAX_GROUPS groups: lane g looks at group g, so that the search for a tile
// costs one round trip to memory instead of one per group.  A group beyond would be passed over.
struct RowTiles {
  static constexpr int MAX_GROUPS = 64;
  int lo, hi, tiles, incl;   // per lane: rows and tiles of group `lane`, tiles up to and including it
  // rows_each != 0: every group has that many rows and offsets is not read
  __device__ __forceinline__ RowTiles(const int* offsets, int n_groups, int bm, int rows_each = 0) : lo(0), hi(0) {
    const int lane = threadIdx.x & 63;
    if (lane < n_groups) {
      lo = rows_each ? lane * rows_each : offsets[lane];
      hi = rows_each ? lo + rows_each : offsets[lane + 1];
    }
    tiles = (hi - lo + bm - 1) / bm;
    incl = wave_inclusive_sum(tiles);
  }
  __device__ __forceinline__ int total() const { return __builtin_amdgcn_readlane(incl, 63); }
  // the tiles of group c are [first_tile(c), end_tile(c))
  __device__ __forceinline__ int first_tile(int c) const { return __builtin_amdgcn_readlane(incl - tiles, c); }
  __device__ __forceinline__ int end_tile(int c) const { return __builtin_amdgcn_readlane(incl, c); }
  // group c of tile `slot`, its first row m0 and the end m_end of the group's rows; false: past the last tile
  __device__ __forceinline__ bool find(int slot, int bm, int& c, int& m0, int& m_end) const {
    const unsigned long long past = __ballot(incl > slot);
    if (past == 0ull) return false;
    c = __builtin_ctzll(past);
    m0 = __builtin_amdgcn_readlane(lo, c) + (slot - __builtin_amdgcn_readlane(incl - tiles, c)) * bm;
    m_end = __builtin_amdgcn_readlane(hi, c);
    return true;
  }
};
__device__ __forceinline__ bool find_tile(const int* offsets, int n_groups, int bm, int slot, int& c, int& m0, int& m_end) {
  return RowTiles(offsets, n_groups, bm).find(slot, bm, c, m0, m_end);
}

__device__ __forceinline__ half8 pack_half8(const float4v& lo, const float4v& hi) {
  half8 o;
  o[0] = (half_t)lo[0]; o[1] = (half_t)lo[1]; o[2] = (half_t)lo[2]; o[3] = (half_t)lo[3];
  o[4] = (half_t)hi[0]; o[5] = (half_t)hi[1]; o[6] = (half_t)hi[2]; o[7] = (half_t)hi[3];
  return o;
}

// The per-(token, selected expert) part of the fused up-projection (Sec. 3.2) on one pair
// block of the accumulators hb = (W1_base x)^T: 32 rows n of d_ff x 16 tokens; a lane owns
// one token (l % 16) and the eight rows 8q .. 8q + 7.
//   h_j = hb + U1cat^T t1ext_j   t1ext_j = the token's t1_j at the rank rows of expert
//                                e_j, zero elsewhere; contraction over the cluster's
//                                K*r rank rows in chunks of 32, chunks no token of the
//                                block needs are skipped
//   a_j = GELU(h_j),  o = sum_j g_j a_j
//   s_j += V2 a_j                the a_j pair block is fed back as B operand (contraction
//                                over its 32 rows n); the product runs over "passes" of
//                                16 rank rows, a lane contributes to a pass only if its
//                                expert's rows lie in it
template <int R, int KMAX>
struct FusedUp {
  static constexpr int NSP = (R == 32) ? 2 : 1;  // 16-row passes per expert

  struct Tok {
    int e[KMAX];      // selected experts, local to the cluster
    float g[KMAX];    // gates (0 for a padding column)
    half8 f[KMAX];    // this lane's slice of t1_j (see t1_frag)
    int p;            // sorted row
    bool valid;
  };

  __device__ static __forceinline__ void load_tok(Tok& t, int p, int m_end, int c, int K, int k, const int* perm,
                                                  const int* expert_idx, const float* gate, const half_t* t1,
                                                  int q) {
    t.p = p;
    t.valid = p < m_end;
    const int pc = t.valid ? p : m_end - 1;
    const int tok = perm[pc];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      t.e[j] = 0;
      t.g[j] = 0.f;
      t.f[j] = half8{0, 0, 0, 0, 0, 0, 0, 0};
      if (j < k) {
        t.e[j] = min(max(expert_idx[(size_t)tok * k + j] - c * K, 0), K - 1);
        t.g[j] = t.valid ? gate[(size_t)tok * k + j] : 0.f;
        load_t1(t.f[j], t1 + ((size_t)pc * k + j) * R, q);
      }
    }
  }
  __device__ static __forceinline__ void load_t1(half8& f, const half_t* tr, int q) {
    if (R == 32) {
      f = *(const half8*)(tr + 8 * q);
    } else if (R == 16) {
      f = *(const half8*)(tr + 8 * (q & 1));
    } else if (R == 8) {
      f = *(const half8*)(tr);
    } else {
      const half4 q4 = *(const half4*)(tr);
      f[0] = q4[0]; f[1] = q4[1]; f[2] = q4[2]; f[3] = q4[3];
    }
  }

  // chunk of 32 rank rows that holds expert e
  __device__ static __forceinline__ int chunk_of(int e) { return (e * R) >> 5; }
  // group of passes that holds expert e
  __device__ static __forceinline__ int pass_group(int e) { return (e * R) / (16 * NSP); }
  // B operand of chunk c for a lane (contraction elements 32 c + 8 q ..) whose token selected
  // expert e and keeps the slice f of its t1
  __device__ static __forceinline__ half8 t1_frag(int e, int c, int q, const half8& f) {
    const half8 z = {0, 0, 0, 0, 0, 0, 0, 0};
    if (R == 32) return (e == c) ? f : z;
    if (R == 16) return (e == 2 * c + (q >> 1)) ? f : z;
    if (R == 8) return (e == 4 * c + q) ? f : z;
    half8 o = z;  // R == 4: elements 0..3 belong to expert 8c + 2q, elements 4..7 to expert 8c + 2q + 1
    if (e == 8 * c + 2 * q) {
      o[0] = f[0]; o[1] = f[1]; o[2] = f[2]; o[3] = f[3];
    } else if (e == 8 * c + 2 * q + 1) {
      o[4] = f[0]; o[5] = f[1]; o[6] = f[2]; o[7] = f[3];
    }
    return o;
  }

  // Chunks of 32 rank rows and groups of NSP passes of 16 rank rows that at least one valid token
  // of the 16-token block needs for its j-th expert (wavefront-uniform bit masks, taken once
  // per token block).
  struct Need {
    unsigned chunks[KMAX], passes[KMAX];
  };
  __device__ static __forceinline__ void need_of(const Tok& t, int k, int n_chunks, int n_pass, Need& nd) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      nd.chunks[j] = 0u;
      nd.passes[j] = 0u;
      if (j >= k) continue;
      for (int c = 0; c < n_chunks; ++c)
        if (__ballot(t.valid && chunk_of(t.e[j]) == c) != 0ull) nd.chunks[j] |= 1u << c;
      for (int pg = 0; pg < n_pass / NSP; ++pg)
        if (__ballot(t.valid && pg == pass_group(t.e[j])) != 0ull) nd.passes[j] |= 1u << pg;
    }
  }

  // uf(c, hh): A operand of U1cat^T for rank chunk c and block hh of the pair block;
  // vf(pp): A operand of V2 for pass pp (rank rows 16 pp + l % 16, the pair block's rows
  // 8q .. 8q + 7 as contraction elements).
  template <class UF, class VF>
  __device__ static __forceinline__ void pair_block(const float4v& hb0, const float4v& hb1, const Tok& t,
                                                    const Need& nd, int k, int q, UF uf, VF vf, float (&o)[8],
                                                    float4v (&sacc)[KMAX][NSP]) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      if (j >= k) {
        if (j == 0) {   // k >= 1 always; keeps o defined for the compiler
#pragma unroll
          for (int i = 0; i < 8; ++i) o[i] = 0.f;
        }
        continue;
      }
      const int ej = t.e[j];
      float4v h0 = hb0, h1 = hb1;
      for (unsigned m = nd.chunks[j]; m != 0u; m &= m - 1u) {
        const int c = __builtin_ctz(m);
        const half8 fb = t1_frag(ej, c, q, t.f[j]);
        h0 = mfma32(uf(c, 0), fb, h0);
        h1 = mfma32(uf(c, 1), fb, h1);
      }
      float a[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = gelu_erf(h0[i]);
        a[4 + i] = gelu_erf(h1[i]);
      }
      settle(a);
      half8 ab;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        o[i] = j == 0 ? t.g[0] * a[i] : fmaf(t.g[j], a[i], o[i]);
        ab[i] = (half_t)a[i];
      }
      for (unsigned m = nd.passes[j]; m != 0u; m &= m - 1u) {
        const int pg = __builtin_ctz(m);
        const half8 z = {0, 0, 0, 0, 0, 0, 0, 0};
        const half8 fb = t.valid && pg == pass_group(ej) ? ab : z;
#pragma unroll
        for (int s = 0; s < NSP; ++s) sacc[j][s] = mfma32(vf(pg * NSP + s), fb, sacc[j][s]);
      }
    }
  }

  // The same for up to two experts per token (KMAX = k of them), with every operand under way before it is wanted: u
  // holds the first chunk's U1 operands of this pair block and leaves with the next one's (next: uf of it, if more), fb the
  // first chunk's B operands of the 16 tokens, the V2 operands come during the GELUs.  Rows are ordered by expert, so
  // most blocks of 16 tokens need one chunk and one group of passes.
  struct Ahead {
    half8 u[KMAX][2], fb[KMAX];
  };
  template <class UF>
  __device__ static __forceinline__ void start(Ahead& w, const Tok& t, const Need& nd, int q, UF uf) {
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      const int c = __builtin_ctz(nd.chunks[j]);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) w.u[j][hh] = uf(c, hh);
      w.fb[j] = t1_frag(t.e[j], c, q, t.f[j]);
    }
  }
  template <class UF, class VF, class Next>
  __device__ static __forceinline__ void pair_block_ahead(const float4v& hb0, const float4v& hb1, const Tok& t, const Need& nd,
                                                          int q, Ahead& w, bool more, UF uf, VF vf, Next next, float (&o)[8],
                                                          float4v (&sacc)[KMAX][NSP]) {
    float4v h[KMAX][2];
    half8 v[KMAX][NSP];
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      h[j][0] = mfma32(w.u[j][0], w.fb[j], hb0);
      h[j][1] = mfma32(w.u[j][1], w.fb[j], hb1);
    }
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      for (unsigned m = nd.chunks[j] & (nd.chunks[j] - 1u); m != 0u; m &= m - 1u) {
        const int c = __builtin_ctz(m);
        const half8 fb = t1_frag(t.e[j], c, q, t.f[j]);
        h[j][0] = mfma32(uf(c, 0), fb, h[j][0]);
        h[j][1] = mfma32(uf(c, 1), fb, h[j][1]);
      }
    }
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      const int pg = __builtin_ctz(nd.passes[j]), c = __builtin_ctz(nd.chunks[j]);
#pragma unroll
      for (int s = 0; s < NSP; ++s) v[j][s] = vf(pg * NSP + s);
      if (more) {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) w.u[j][hh] = next(c, hh);
      }
    }
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      float a[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] = gelu_erf(h[j][i / 4][i % 4]);
      settle(a);
      half8 ab;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        o[i] = j == 0 ? t.g[0] * a[i] : fmaf(t.g[j], a[i], o[i]);
        ab[i] = (half_t)a[i];
      }
      const unsigned rest = nd.passes[j] & (nd.passes[j] - 1u);
      const half8 z = {0, 0, 0, 0, 0, 0, 0, 0};
      if (rest == 0u) {   // all of the block's tokens; the columns of others are not stored
#pragma unroll
        for (int s = 0; s < NSP; ++s) sacc[j][s] = mfma32(v[j][s], ab, sacc[j][s]);
      } else {
        for (unsigned m = nd.passes[j]; m != 0u; m &= m - 1u) {
          const int pg = __builtin_ctz(m);
          const half8 fb = t.valid && pg == pass_group(t.e[j]) ? ab : z;
#pragma unroll
          for (int s = 0; s < NSP; ++s) sacc[j][s] = mfma32(vf(pg * NSP + s), fb, sacc[j][s]);
        }
      }
    }
  }

  // The lane holds rank rows 4q .. 4q + 3 of each pass accumulator; those inside the expert's
  // rows are the token's s_j.  dst_tile: [T][k][R] FP32 partial of this row tile.
  __device__ static __forceinline__ void store_s(const Tok& t, const float4v (&sacc)[KMAX][NSP], float* dst_tile,
                                                 int k, int q) {
    if (!t.valid) return;
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      if (j >= k) continue;
      const int be = (t.e[j] * R) & 15;   // first row of the expert inside its pass
      float* dst = dst_tile + ((size_t)t.p * k + j) * R;
      const int row0 = 4 * q;
      if (row0 >= be && row0 < be + (R < 16 ? R : 16)) {
#pragma unroll
        for (int s = 0; s < NSP; ++s) *(float4v*)(dst + 16 * s + row0 - be) = sacc[j][s];
      }
    }
  }
};

}  // namespace
