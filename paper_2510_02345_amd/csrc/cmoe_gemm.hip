// Grouped matrix-core kernels of the expert computation (Sec. 3.2):
//   Hb   = W1_base(c) x  -> fused: + U1 t1, GELU, gated sum A, s = V2 a
//   Yb   = W2_base(c) A
//   y    = Yb + sum_j g_j U2 s_j, back in token order
//
// All products are computed "weights x tokens^T": the weight rows are the A operand of
// v_mfma_f32_16x16x32_f16 (rows of the 16x16 block), the tokens are the B operand (columns).
// A lane of an accumulator block then holds ONE token (column lane % 16) and four output
// rows; with the row order of the pair blocks (cmoe_device.h) two blocks give it eight
// consecutive rows.  That is what lets the per-token quantities (experts, gates, t1) live in
// per-lane registers, and lets an accumulator pair be fed back as the B operand of the next
// product without leaving registers (its rows become the contraction index).
#include <type_traits>

#include "cmoe_device.h"

namespace {

// Tile of one workgroup: BN weight rows x BM tokens, WAVES_N x WAVES_M wavefronts, each
// owning (BN/WAVES_N) x (BM/WAVES_M) outputs as 16x16 accumulator blocks (as the epilogue sees
// it).  Operand tiles move global -> LDS with direct-to-LDS loads (no register staging) into NS
// stages; tile rows are 64 B (32 contraction elements), their four 16-B chunks XOR-swizzled with
// swz(row) so that the 16 lanes the LDS serves per cycle hit 64 distinct banks.  The weight rows
// of a tile are stored in MFMA order: tile row rho holds weight row pi_row(rho).
template <int BN_, int BM_, int WAVES_N_, int WAVES_M_, int NS_>
struct Tile {
  static constexpr int BN = BN_, BM = BM_, WAVES_N = WAVES_N_, WAVES_M = WAVES_M_, NS = NS_;
  static constexpr int NWAVES = WAVES_N * WAVES_M, NT = NWAVES * 64;
  static constexpr int WN = BN / WAVES_N, WM = BM / WAVES_M;
  static constexpr int NA = WN / 16, MT = WM / 16;   // 16-row blocks and 16-token blocks of a wavefront
  static constexpr int NP = WN / 32;                 // pair blocks of a wavefront
  static constexpr int BK = 32, ROWB = BK * 2;
  static constexpr int STAGE_BYTES = (BN + BM) * ROWB;
  static constexpr int SMEM_BYTES = NS * STAGE_BYTES;
  static constexpr int PER_WAVE = (BN + BM) / 16 / NWAVES;  // 1-KiB load instructions per wavefront and 32 elements
  static_assert(BN % (32 * WAVES_N) == 0 && BM % (16 * WAVES_M) == 0, "wave tile");
};
// 256 x 256: half the operand bytes per flop of 128 x 128; eight wavefronts in ping-pong.
using TileBig = Tile<256, 256, 2, 4, 4>;
// Half and a quarter of it, for what does not fill a round of the CUs (tile_small).  The quarter is
// 128 x 128, or 256 x 64 where the epilogue wants all 256 rows of the big tile in one workgroup.
// A stage is 64 contraction elements, hence NS = 8 blocks of 32 are four stages.
using TileHalf = Tile<256, 128, 2, 4, 6>;
using TileQuad = Tile<128, 128, 2, 4, 8>;
using TileSlab = Tile<256, 64, 4, 2, 6>;

struct GemmArgs {
  const half_t* W;   // weights of cluster c: W + c * w_cstride, [N][ldw] row-major
  long w_cstride;
  int ldw, N;
  const half_t* X;   // token-side operand, row for sorted row p: X + (gather ? gather[p] : p) * ldx
  int ldx;
  const int* gather;
  int Kc;            // contraction length, multiple of 32
  const int* offsets;
  int G, n_tiles;    // groups (at most 64); column tiles of TileBig::BN weight rows
  int x_div;         // row of X = gather[p] / x_div (several sorted rows may share one row of X); 0 = 1
  // optional per-group contraction range: group c contracts columns krange[2c] ..
  // krange[2c] + krange[2c+1] (both multiples of 32) of W and X instead of 0 .. Kc
  const int* krange;
  // elements between consecutive 32-element contraction blocks of a row of W / X; 0 = 32
  // (plain row-major rows).  An operand stored as [K / 32][rows][32] has ld = 32 and a
  // step of rows * 32: the 16 rows of one load instruction are then 1 KiB of contiguous memory.
  long kstep_w, kstep_x;
  // rows_each != 0: every group has that many rows (offsets is not read) and row p of group c reads
  // row p - c * rows_each of X, which all groups share
  int rows_each;
  // scratch for parts of the contraction (gemm_kernel), NULL: none.  [GEMM_PARTS] tiles of accumulators, and as
  // many arrival counts, zero before the launch
  float4v* parts;
  int* arrivals;
  // Kc2 != 0: the contraction goes on over Kc2 more elements of a second pair of operands (epilogues with EXTENDS): row n
  // of cluster c at W2 + c * w2_cstride + n * ldw2, row p of [Kc2 / 32][..][32] with X's row and block strides at X2
  const half_t* W2;
  long w2_cstride;
  int ldw2, Kc2;
  const half_t* X2;
};
constexpr int EXT_BLOCKS = 8;   // blocks of the first pair, at least, for a second one

struct TileCtx {
  int c, n_tile, n0, m0, m_end, wn, wm, lane, tid;
  half_t* smem;
  bool ext;        // the sums hold the second pair of operands
  int first_slot;  // epilogues with PANELS: portion i of them lies in slot (first_slot + i) % 4 of smem
};
// Factor panels of an epilogue with PANELS: up to four portions of 32 KiB, each 32 pieces of 1 KiB that one direct-to-LDS
// load fetches.
constexpr int PANEL_BYTES = 32768, PANEL_SLOTS = 4;
// Source of a wavefront's four pieces of the first portion, and the way from one portion to the next.
struct PanelSrc {
  const half_t* at[4];
  size_t step;
  template <class Epi>
  __device__ __forceinline__ PanelSrc(const Epi& epi, int c, int n0, int wave, int lane) : step(epi.panel_step(wave * 4)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) at[i] = epi.panel_src(c, n0, wave * 4 + i, lane);
  }
  __device__ __forceinline__ void issue(int portion, unsigned smem_base, int slot, int wave) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) dma16(at[i] + portion * step, smem_base + slot * PANEL_BYTES + (wave * 4 + i) * 1024);
  }
};

// Where a tile of a group comes from.
struct TileSrc {
  const GemmArgs& g;
  int c, n0, m0, m_end;
  int k_lo, KT;           // first 32-element block and number of blocks
  int ext_at;             // block from which on the second pair of operands is read (the KT count them)
  long kstep_w, kstep_x;
  // s, split: part s of 2^split of the contraction
  __device__ __forceinline__ TileSrc(const GemmArgs& g_, int c_, int n0_, int m0_, int m_end_, int s = 0, int split = 0)
      : g(g_), c(c_), n0(n0_), m0(m0_), m_end(m_end_) {
    k_lo = g.krange ? g.krange[2 * c] / 32 : 0;
    KT = (g.krange ? g.krange[2 * c + 1] : g.Kc) / 32;
    ext_at = KT;
    KT += g.Kc2 / 32;
    const int from = (s * KT) >> split;
    KT = (((s + 1) * KT) >> split) - from;
    ext_at -= from;
    k_lo += from;
    kstep_w = g.kstep_w ? g.kstep_w : 32;
    kstep_x = g.kstep_x ? g.kstep_x : 32;
  }
  // source of the 16-byte chunk at position `pos` of tile row `row` (BN weight rows, then the
  // tokens) in the tile's first block; rows past the end of the matrix / group repeat the last one
  __device__ __forceinline__ const half_t* chunk(int row, int pos, int bn) const {
    const half_t* base;
    if (row < bn) {
      base = g.W + (size_t)c * g.w_cstride + (size_t)min(n0 + pi_row(row), g.N - 1) * g.ldw + (size_t)k_lo * kstep_w;
    } else {
      const int p = min(m0 + row - bn, m_end - 1);
      base = g.X + (size_t)(g.gather ? (g.x_div > 1 ? g.gather[p] / g.x_div : g.gather[p]) : p - c * g.rows_each) * g.ldx +
             (size_t)k_lo * kstep_x;
    }
    return base + ((pos ^ swz(row)) << 3);
  }
  // the same of the second pair of operands, in what would be its block -ext_at
  __device__ __forceinline__ const half_t* chunk2(int row, int pos, int bn) const {
    const half_t* base = row < bn ? g.W2 + (size_t)c * g.w2_cstride + (size_t)min(n0 + pi_row(row), g.N - 1) * g.ldw2 - (long)ext_at * 32
                                  : g.X2 + (size_t)min(m0 + row - bn, m_end - 1) * g.ldx - (long)ext_at * kstep_x;
    return base + ((pos ^ swz(row)) << 3);
  }
};
// For a tile whose epilogue can do without the second pair of operands: each wavefront leaves in LDS whether it has seen a
// reason for that, and behind the next barrier everyone sees them all.
__device__ __forceinline__ void put_flag(int* flags, bool mine) {
  const bool any = __ballot(mine) != 0ull;
  if ((threadIdx.x & 63) == 0) flags[threadIdx.x >> 6] = any;
}
__device__ __forceinline__ bool any_flag(const int* flags) {
  int v = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) v |= flags[i];
  return __builtin_amdgcn_readfirstlane(v) != 0;
}

// ---------------------------------------------------------------- 256 x 256 tile
// Ping-pong: the two wavefronts of a SIMD (w, w + 4) run one barrier interval apart, so in every
// interval one of them issues its MFMAs while the other reads fragments from LDS and issues the
// next loads.  (Issuing the loads from inside the MFMA phase instead, between the 16-cycle
// MFMAs, measured 5 % slower on the whole layer.)
template <class Epi>
__device__ __forceinline__ void tile_big(const GemmArgs& g, const Epi& epi, char* smem, int* flags, int c, int n_tile, int m0,
                                         int m_end) {
  using TL = TileBig;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = wave % TL::WAVES_N, wm = wave / TL::WAVES_N;
  const int n0 = n_tile * TL::BN;
  const TileSrc src(g, c, n0, m0, m_end);
  const unsigned smem_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
  int tok = 0;
  if constexpr (Epi::PANELS) tok = epi.template token<TL>(tid, m0, m_end);
  const half_t* gsrc[TL::PER_WAVE];
#pragma unroll
  for (int i = 0; i < TL::PER_WAVE; ++i)
    gsrc[i] = src.chunk((wave * TL::PER_WAVE + i) * 16 + (lane >> 2), lane & 3, TL::BN);
  auto issue_from = [&](const half_t* const (&from)[TL::PER_WAVE], long kstep_w, int kt, int stage) {
#pragma unroll
    for (int i = 0; i < TL::PER_WAVE; ++i)
      dma16(from[i] + (size_t)kt * (((wave * TL::PER_WAVE + i) * 16 < TL::BN) ? kstep_w : src.kstep_x),
            smem_base + stage * TL::STAGE_BYTES + (wave * TL::PER_WAVE + i) * 1024);
  };
  auto issue = [&](int kt, int stage) { issue_from(gsrc, src.kstep_w, kt, stage); };

  float4v acc[TL::NA][TL::MT];
#pragma unroll
  for (int a = 0; a < TL::NA; ++a)
#pragma unroll
    for (int b = 0; b < TL::MT; ++b) acc[a][b] = float4v{0.f, 0.f, 0.f, 0.f};

  // fragment addresses: lane l reads row (or token) l % 16, 16-byte chunk l / 16 of the 64-byte row
  const int t16 = lane & 15, q = lane >> 4;
  int offa[TL::NA], offb[TL::MT];
#pragma unroll
  for (int a = 0; a < TL::NA; ++a) {
    const int row = wn * TL::WN + a * 16 + t16;
    offa[a] = row * TL::ROWB + ((q ^ swz(row)) << 4);
  }
#pragma unroll
  for (int b = 0; b < TL::MT; ++b) {
    const int row = TL::BN + wm * TL::WM + b * 16 + t16;
    offb[b] = row * TL::ROWB + ((q ^ swz(row)) << 4);
  }
  // 16-token blocks of this wavefront that hold at least one real token (a ragged last
  // row tile of a cluster skips the matrix-core work of the others)
  bool bv[TL::MT];
#pragma unroll
  for (int b = 0; b < TL::MT; ++b) bv[b] = m0 + wm * TL::WM + b * 16 < m_end;

  int KT = src.KT;
#pragma unroll
  for (int s = 0; s < TL::NS - 1; ++s)
    if (s < KT) issue(s, s);
  if constexpr (Epi::PANELS) epi.template put_tokens<TL>(tok, tid, m0, smem_base);
  bool ext = false;
  if constexpr (Epi::EXTENDS) {
    put_flag(flags, epi.apart(c, n0, TL::BN, tid, TL::NT));
    wait_lds();
  }
  int stage = 0, nstage = TL::NS - 1;
  const bool set_b = wave >= 4;
  if (KT > 1) wait_vm<(TL::NS - 2) * TL::PER_WAVE>(); else wait_vm<0>();
  if (KT <= TL::NS - 2) wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  if constexpr (Epi::EXTENDS) {
    ext = g.Kc2 != 0 && !any_flag(flags);
    if (!ext) KT = min(KT, src.ext_at);
  }
  if (set_b) __builtin_amdgcn_s_barrier();
  // next(): issues what comes next and waits until block kt + 1 (own loads) has landed
  constexpr int KEEP = (TL::NS - 2) * TL::PER_WAVE;   // younger loads then in flight
  auto step = [&](auto next) {
    const char* sb = smem + stage * TL::STAGE_BYTES;
    half8 fa[TL::NA], fb[TL::MT];
#pragma unroll
    for (int a = 0; a < TL::NA; ++a) fa[a] = *(const half8*)(sb + offa[a]);
#pragma unroll
    for (int b = 0; b < TL::MT; ++b)
      if (bv[b]) fb[b] = *(const half8*)(sb + offb[b]);
    // the stage refilled here held block kt - 1, which both sets read before the
    // barrier that opened this interval
    next();
    wait_lds();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int b = 0; b < TL::MT; ++b)
      if (bv[b]) {
#pragma unroll
        for (int a = 0; a < TL::NA; ++a) acc[a][b] = mfma32(fa[a], fb[b], acc[a][b]);
      }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    stage = (stage + 1 == TL::NS) ? 0 : stage + 1;
    nstage = (nstage + 1 == TL::NS) ? 0 : nstage + 1;
  };
  // The blocks behind which more of the first pair are to be loaded, and the rest: the change of operands in one loop
  // with the others cost registers and a fifth of its rate.
  const int plain = max(0, min(KT, Epi::EXTENDS ? src.ext_at : KT) - (TL::NS - 1));
  int kt = 0;
  for (; kt < plain; ++kt)
    step([&] {
      issue(kt + TL::NS - 1, nstage);
      wait_vm<KEEP>();
    });
  if constexpr (Epi::EXTENDS) {
    if (ext && KT > src.ext_at) {
      const half_t* gsrc2[TL::PER_WAVE];
#pragma unroll
      for (int i = 0; i < TL::PER_WAVE; ++i)
        gsrc2[i] = src.chunk2((wave * TL::PER_WAVE + i) * 16 + (lane >> 2), lane & 3, TL::BN);
      for (; kt + TL::NS - 1 < KT; ++kt)
        step([&] {
          issue_from(gsrc2, 32, kt + TL::NS - 1, nstage);
          wait_vm<KEEP>();
        });
    }
  }
  int first_slot = 0;
  if constexpr (Epi::PANELS) {
    // The epilogue's panels follow the last blocks through the stages: a portion into each one that is done with
    static_assert(TL::NS == 4 && TL::PER_WAVE == 4 && TL::STAGE_BYTES == PANEL_BYTES, "a portion is like a block");
    const PanelSrc panel(epi, c, n0, wave, lane);
    const int n = epi.portions(), early = KT >= TL::NS - 1 ? min(n, TL::NS - 1) : 0;
    first_slot = KT & 3;
    for (; kt < KT; ++kt)
      step([&] {
        const int i = kt + TL::NS - 1 - KT;
        if (i < early) {
          panel.issue(i, smem_base, (first_slot + i) & 3, wave);
          wait_vm<KEEP>();
        } else if (early == 0) {
          wait_vm<0>();
        } else if (i < TL::NS - 2) {   // only the portion behind the last block may be in flight
          wait_vm<TL::PER_WAVE>();
        }
      });
    if (!set_b) __builtin_amdgcn_s_barrier();
    // behind that barrier every wavefront has read the last block
    for (int i = early; i < n; ++i) panel.issue(i, smem_base, (first_slot + i) & 3, wave);
  } else {
    for (; kt < KT; ++kt) step([] { wait_vm<0>(); });
    if (!set_b) __builtin_amdgcn_s_barrier();
  }
  TileCtx ctx{c, n_tile, n0, m0, m_end, wn, wm, lane, tid, (half_t*)smem, ext, first_slot};
  epi.template run<TL>(ctx, acc);
}

// ---------------------------------------------------------------- half or a quarter of it
// What bounds a small tile is the LDS: 64 x 64 outputs per wavefront need 8 KiB of fragments per
// 32 contraction elements, half of what 64 x 32 need per flop.  So that eight wavefronts fit the
// tile at that size (128 x 64 for the half), it is computed by TWO sets of four, one on the even
// and one on the odd 32-element blocks, whose accumulators are added at the end (set 1 hands
// token blocks 0, 1 of a wavefront to set 0 and gets 2, 3 in return), which leaves every
// wavefront with 32 tokens for the epilogue.  A stage holds a block for each set; the fragments
// of the next stage are read while the matrix cores work on the current one.  Measured on
// 128 x 128 (204 workgroups, contraction 3072): 32 us, of which 0.42 us per 64 elements; with one
// set of eight wavefronts of 64 x 32 in ping-pong 40 us.
// With split > 0 the workgroup computes part s of 2^split of the contraction, and the last to arrive of the parts
// (number `first` on of g.parts) adds them, in their order, and runs the epilogue; nobody waits.
template <class TL, class Epi>
__device__ __forceinline__ void tile_small(const GemmArgs& g, const Epi& epi, char* smem, int* flags, int c, int n_tile, int n0, int m0,
                                           int m_end, int s = 0, int split = 0, int first = 0) {
  constexpr int NSTG = TL::NS / 2, HALF = TL::STAGE_BYTES, STAGE = 2 * HALF;
  constexpr int PIECES = (TL::BN + TL::BM) / 16, PER = PIECES / 4;   // 16-row pieces of a block, per wavefront of a set
  constexpr int NA = TL::NA, NB = 4;   // 16-row and 16-token blocks of a wavefront in the main loop
  static_assert(TL::WM == 32 && TL::NWAVES == 8 && PIECES % 4 == 0, "two sets of four wavefronts");
  static_assert(8 * NA * 2 * 1024 <= TL::SMEM_BYTES, "exchange area");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int set = wave >> 2, w4 = wave & 3, wn = w4 % TL::WAVES_N, wmh = w4 / TL::WAVES_N;
  const TileSrc src(g, c, n0, m0, m_end, s, split);
  const unsigned smem_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
  int KT = src.KT, steps = (KT + 1) / 2;   // an odd last block is set 0's; set 1 loads it too and ignores it
  int tok = 0;
  if constexpr (Epi::PANELS) tok = epi.template token<TL>(tid, m0, m_end);
  const half_t* gsrc[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) gsrc[i] = src.chunk((w4 * PER + i) * 16 + (lane >> 2), lane & 3, TL::BN);
  bool ext = false;
  auto issue_from = [&](const half_t* const (&from)[PER], long kstep_w, int st, int stage) {
    const int blk = min(2 * st + set, KT - 1);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      dma16(from[i] + (size_t)blk * (((w4 * PER + i) * 16 < TL::BN) ? kstep_w : src.kstep_x),
            smem_base + stage * STAGE + set * HALF + (w4 * PER + i) * 1024);
  };
  auto issue = [&](int st, int stage) { issue_from(gsrc, src.kstep_w, st, stage); };
  float4v acc[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = float4v{0.f, 0.f, 0.f, 0.f};
  const int t16 = lane & 15, q = lane >> 4;
  const int frag = set * HALF + t16 * 64 + ((q ^ swz(t16)) << 4);   // tile rows of a fragment start at multiples of 16
  const int offa = frag + wn * TL::WN * 64, offb = frag + (TL::BN + wmh * 64) * 64;
  const int nb = min(NB, (m_end - m0 - wmh * 64 + 15) / 16);   // token blocks that hold a token
  struct Frag {
    half8 a[NA], b[NB];
  };
  auto read = [&](Frag& f, int stage) {
    const char* sb = smem + stage * STAGE;
#pragma unroll
    for (int a = 0; a < NA; ++a) f.a[a] = *(const half8*)(sb + offa + a * 1024);
#pragma unroll
    for (int b = 0; b < NB; ++b) f.b[b] = *(const half8*)(sb + offb + b * 1024);
  };
  auto use = [&](const Frag& f) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (b < nb) {
#pragma unroll
        for (int a = 0; a < NA; ++a) acc[a][b] = mfma32(f.a[a], f.b[b], acc[a][b]);
      }
  };
  if (steps > 0) {
#pragma unroll
    for (int s = 0; s < NSTG - 1; ++s)
      if (s < steps) issue(s, s);
    if constexpr (Epi::PANELS) epi.template put_tokens<TL>(tok, tid, m0, smem_base);
    if constexpr (Epi::EXTENDS) {
      put_flag(flags, epi.apart(c, n0, TL::BN, tid, TL::NT));
      wait_lds();
    }
    if (NSTG - 2 < steps) wait_vm<(NSTG - 2) * PER>(); else wait_vm<0>();   // stage 0, for the first fragments
    __builtin_amdgcn_s_barrier();
    if constexpr (Epi::EXTENDS) {
      ext = g.Kc2 != 0 && !any_flag(flags);
      if (!ext) KT = min(KT, src.ext_at);
      steps = (KT + 1) / 2;
    }
    Frag f0, f1;
    read(f0, 0);
    int rd = 1, wr = NSTG - 1;   // stage of step st + 1; stage refilled in step st (it held step st - 1)
    auto step = [&](int st, const Frag& cur, Frag& nxt, auto next) {
      if (st + 1 < steps) {
        // step st + 1 has landed (own loads), then everyone's; every wavefront has left step st - 1
        if (st + NSTG - 2 < steps) wait_vm<(NSTG - 3) * PER>(); else wait_vm<0>();
        wait_lds();
        __builtin_amdgcn_s_barrier();
        read(nxt, rd);
        if (st + NSTG - 1 < steps) next(st + NSTG - 1, wr);
      }
      if (2 * st + set < KT) use(cur);
      rd = rd + 1 == NSTG ? 0 : rd + 1;
      wr = wr + 1 == NSTG ? 0 : wr + 1;
    };
    int st = 0;
    auto two = [&](auto next) {
      step(st, f0, f1, next);
      if (st + 1 < steps) step(st + 1, f1, f0, next);
    };
    if constexpr (Epi::EXTENDS) {
      // pairs of steps behind which only blocks of the first pair of operands are loaded, then the others
      const int plain = ext ? min(steps, src.ext_at / 2 - NSTG) : steps;
      for (; st < plain; st += 2) two(issue);
      if (st < steps) {
        const half_t* gsrc2[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) gsrc2[i] = src.chunk2((w4 * PER + i) * 16 + (lane >> 2), lane & 3, TL::BN);
        for (; st < steps; st += 2)
          two([&](int s, int stage) {
            if (min(2 * s + set, KT - 1) < src.ext_at) issue(s, stage); else issue_from(gsrc2, 32, s, stage);
          });
      }
    } else {
      for (; st < steps; st += 2) two(issue);
    }
  }
  float4v out[NA][2];
  __syncthreads();   // the stages have been read
  // panels: what fits behind the exchange area before it, the rest after
  constexpr int XSLOTS = 8 * NA * 2 * 1024 / PANEL_BYTES;
  const int first_slot = XSLOTS & 3;
  int n_panel = 0;
  if constexpr (Epi::PANELS) {
    for (; n_panel < min(epi.portions(), PANEL_SLOTS - XSLOTS); ++n_panel)
      PanelSrc(epi, c, n0, wave, lane).issue(n_panel, smem_base, XSLOTS + n_panel, wave);
  }
  {
    float4v* xs = (float4v*)smem + (size_t)w4 * NA * 2 * 64 + lane;
    float4v* send = xs + (set ? 0 : 4 * NA * 2 * 64);
    const float4v* recv = xs + (set ? 4 * NA * 2 * 64 : 0);
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        send[(a * 2 + b) * 64] = set ? acc[a][b] : acc[a][b + 2];
        out[a][b] = set ? acc[a][b + 2] : acc[a][b];
      }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) out[a][b] += recv[(a * 2 + b) * 64];
  }
  if constexpr (Epi::PANELS) {
    wait_lds();
    __builtin_amdgcn_s_barrier();
    for (; n_panel < epi.portions(); ++n_panel)
      PanelSrc(epi, c, n0, wave, lane).issue(n_panel, smem_base, (XSLOTS + n_panel) & 3, wave);
  } else {
    __syncthreads();   // the epilogue may use the space
  }
  if constexpr (Epi::SPLITS && TL::BN * TL::BM == GEMM_PART) {
    if (split > 0) {
      // The parts go through memory that all CUs see: stores and loads at device scope, completed before the
      // arrival is counted.  (With ordinary stores and a fence every workgroup writes back its whole L2.)
      constexpr int PART = GEMM_PART / 2;   // pairs of values
      typedef unsigned long long u64;
      u64* mine = (u64*)g.parts + (size_t)(first + s) * PART + tid;
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const u64* v = (const u64*)&out[a][b];
#pragma unroll
          for (int h = 0; h < 2; ++h)
            __hip_atomic_store(mine + ((a * 2 + b) * 2 + h) * TL::NT, v[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      wait_vm<0>();
      __syncthreads();
      int* last = (int*)smem;
      if (tid == 0)
        *last = __hip_atomic_fetch_add(g.arrivals + first, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (1 << split) - 1;
      __syncthreads();
      if (!*last) return;
      const u64* all = (const u64*)g.parts + (size_t)first * PART + tid;
      for (int i = 0; i < 1 << split; ++i) {
        u64 v[NA * 4];
#pragma unroll
        for (int n = 0; n < NA * 4; ++n)
          v[n] = __hip_atomic_load(all + (size_t)i * PART + n * TL::NT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int n = 0; n < NA * 4; ++n) {
          float4v& o = out[n / 4][n / 2 % 2];
          const int h = n % 2 * 2;
          const float lo = __uint_as_float((unsigned)v[n]), hi = __uint_as_float((unsigned)(v[n] >> 32));
          o[h] = i == 0 ? lo : o[h] + lo;
          o[h + 1] = i == 0 ? hi : o[h + 1] + hi;
        }
      }
      __syncthreads();   // *last has been read
    }
  }
  TileCtx ctx{c, n_tile, n0, m0, m_end, wn, wmh * 2 + set, lane, tid, (half_t*)smem, ext, first_slot};
  epi.template run<TL>(ctx, out);
}

// ---------------------------------------------------------------- grouped product
// Workgroups are dealt round-robin to the 8 XCDs.  Each XCD takes an equal run of the 256 x 256
// tiles, walked in super-tiles of 4 row tiles x 8 column tiles, so that the workgroups resident on
// one XCD share both operands through its L2.  Which tiles there are follows from the group
// offsets on the device, so no host round trip sits between routing and the products.  An XCD's
// 32 CUs take its tiles in rounds of 32; what is left after the full rounds is cut into halves or
// quarters when these fit one round (a half takes about 0.4 and a quarter 0.25 of a big
// tile's time), which is also how a launch with few tiles fills the machine.  Up-projection of
// 777 tokens (64 tiles, contraction 1024): 50 -> 29 us in 220 quarters; 16384 tokens with Zipf
// loads (132 tiles per XCD): 282 -> 250 us, its down-projection (33 tiles) 190 -> 168 us.
// Where the quarters of the leftover still leave CUs idle, the down-projection also cuts their contraction, into as many
// parts as there are CUs (and 10 blocks of it in a part): one more exchange of the sums, through memory,
// costs about 8 us (with ordinary stores and a device fence in each workgroup 30), a step of 64 elements takes 0.42.
// So a contraction below 50 blocks stays whole.  Whole forward with parts and without, 777 tokens of 4 clusters of width 1024
// and contraction 1024 63.4 and 59.4, 1536 63.7 and 64.0, 1728 64.8 and 66.0, 2560 67.1 and 72.1; of 2 of width 768 and 1408
// 60.2 and 58.7, 1600 60.2 and 60.5.  Of 4 of width 512 and 2048 in four parts 57.4, in eight of 8 blocks 60.7, whole 60.8.
// Groups of at most a quarter's tokens are bound by their weights where there are several of them on an XCD: four
// tiles (300 tokens of 16 of width 512) 1728 60.2 and 58.7, 2048 60.3 and 60.4, eight (width 1024) 1728 69.8 and 67.2,
// 3072 81.1 and 80.5, 777 tokens 89.2 and 91.8; so they are cut from 64 blocks on with four tiles, from 96 with eight.
// 4 clusters of 1024 x 4096: 777 tokens (2 tiles per XCD) 41 -> 29 us, 1200 (3) 43 -> 35; 2 of 768 x 3072,
// 300 tokens 30 -> 23; 8 of 2048 x 8192, 300 tokens (8, upper quarters only) 73 -> 63; 16384 Zipf tokens, whole
// forward 429 -> 422.
constexpr int XSM = 4, XSN = 8, XCD_CUS = 32;
constexpr int MAX_SPLIT = 3;   // log2 of the parts of the contraction of a quarter, at most
constexpr int SPLIT_BLOCKS = 50, PART_BLOCKS = 10;   // 32-element blocks of a contraction that is cut and of a part, at least
static_assert(8 * XCD_CUS == GEMM_PARTS, "a part per CU");
template <class Epi>
__global__ __launch_bounds__(512, 1) void gemm_kernel(GemmArgs g, Epi epi) {
  using Quarter = typename Epi::Quarter;
  constexpr int SB = Epi::template smem_bytes<TileBig>(), SH = Epi::template smem_bytes<TileHalf>(),
                SQ = Epi::template smem_bytes<Quarter>();
  constexpr int SMEM = SB > SH ? (SB > SQ ? SB : SQ) : (SH > SQ ? SH : SQ);
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  __shared__ int flags[8];
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
  const RowTiles rt(g.offsets, g.G, TileBig::BM, g.rows_each);
  const int slots = rt.total(), tiles = slots * g.n_tiles;
  const int lo = (int)((long)tiles * xcd >> 3), mine = (int)((long)tiles * (xcd + 1) >> 3) - lo;
  int full = mine / XCD_CUS * XCD_CUS, cut = 0;   // log2 of the parts a leftover tile is cut into
  if (mine - full > XCD_CUS / 2) full = mine; else cut = mine - full > XCD_CUS / 4 ? 1 : 2;
  int pieces = cut, split = 0;   // log2 of a leftover tile's pieces and of the parts of the contraction of each
  if constexpr (Epi::SPLITS) {
    const int left = mine - full;
    if (g.parts != nullptr && cut == 2 && left > 0) {
      // no group with more tokens than a quarter: its lower quarters are empty
      if (__ballot(rt.hi - rt.lo > Quarter::BM) == 0ull) pieces = TileBig::BN / Quarter::BN == 2 ? 1 : 0;
      const int blocks = g.Kc / 32, least = pieces == cut ? SPLIT_BLOCKS : max(SPLIT_BLOCKS, 32 + 8 * left);
      if (blocks >= least)
        while (split < MAX_SPLIT && left << (pieces + split + 1) <= XCD_CUS && blocks >= PART_BLOCKS << (split + 1)) ++split;
    }
  }
  const bool big = local < full;
  const int v = local - full, t = big ? lo + local : lo + full + (v >> (pieces + split)),
            part = (v >> split) & ((1 << pieces) - 1);
  if (t >= lo + mine) return;
  const int per_group = XSM * g.n_tiles, vg = t / per_group, rem = t % per_group;
  const int sm = min(XSM, slots - vg * XSM);                      // row tiles of the super-tile
  const int nblk = rem / (sm * XSN), r2 = rem % (sm * XSN);
  const int sn = min(XSN, g.n_tiles - nblk * XSN);                // column tiles of the super-tile
  const int slot = vg * XSM + r2 / sn, n_tile = nblk * XSN + r2 % sn;
  int c, m0, m_end;
  if (!rt.find(slot, TileBig::BM, c, m0, m_end)) return;
  int n0 = n_tile * TileBig::BN;
  if (big) {
    tile_big<Epi>(g, epi, smem, flags, c, n_tile, m0, m_end);
  } else if (cut == 1) {
    m0 += part * TileHalf::BM;
    if (m0 < m_end) tile_small<TileHalf, Epi>(g, epi, smem, flags, c, n_tile, n0, m0, m_end);
  } else {
    constexpr int ACROSS = TileBig::BN / Quarter::BN;
    n0 += part % ACROSS * Quarter::BN;
    m0 += part / ACROSS * Quarter::BM;
    if (n0 < g.N && m0 < m_end)
      tile_small<Quarter, Epi>(g, epi, smem, flags, c, n_tile, n0, m0, m_end, v & ((1 << split) - 1), split,
                                xcd * XCD_CUS + (v & -(1 << split)));
  }
}

template <class Epi>
hipError_t launch_gemm(const GemmArgs& g, int T, const Epi& epi, hipStream_t st) {
  const int tiles = ((T + TileBig::BM - 1) / TileBig::BM + g.G) * g.n_tiles;   // at most
  // the leftover tiles of an XCD, one at least, become up to XCD_CUS workgroups
  const int extra = g.parts != nullptr ? XCD_CUS - 1 : 3 * XCD_CUS / 4;
  hipLaunchKernelGGL((gemm_kernel<Epi>), dim3((unsigned)(8 * ((tiles + 7) / 8 + extra))), dim3(512), 0, st, g, epi);
  return hipGetLastError();
}

// ---------------------------------------------------------------- few weight rows
// At most 64 weight rows (products into rank space): one 64-row weight tile against 128 tokens,
// four wavefronts side by side along the tokens; bound by the stream of X rows.  Token blocks past
// a group's end are multiplied and not stored, and tiles are not placed by XCD: with both, in
// the tiled kernel that these products ran on before, the four products of a training step took
// 27 us for 128 tokens of width 128, here 22; for 32768 tokens, 64 experts and width 2048 724 and 722.
template <class Epi>
__global__ __launch_bounds__(256, 3) void gemm_thin_kernel(GemmArgs g, Epi epi) {
  using TL = Tile<64, 128, 1, 4, 4>;
  __shared__ __attribute__((aligned(1024))) char smem[TL::SMEM_BYTES];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int c, m0, m_end;
  if (!find_tile(g.offsets, g.G, TL::BM, blockIdx.x, c, m0, m_end)) return;
  const TileSrc src(g, c, 0, m0, m_end);
  const unsigned smem_base = (unsigned)(size_t)(__attribute__((address_space(3))) char*)smem;
  const half_t* gsrc[TL::PER_WAVE];
#pragma unroll
  for (int i = 0; i < TL::PER_WAVE; ++i)
    gsrc[i] = src.chunk((wave * TL::PER_WAVE + i) * 16 + (lane >> 2), lane & 3, TL::BN);
  auto issue = [&](int kt, int stage) {
#pragma unroll
    for (int i = 0; i < TL::PER_WAVE; ++i)
      dma16(gsrc[i] + (size_t)kt * (((wave * TL::PER_WAVE + i) * 16 < TL::BN) ? src.kstep_w : src.kstep_x),
            smem_base + stage * TL::STAGE_BYTES + (wave * TL::PER_WAVE + i) * 1024);
  };
  float4v acc[TL::NA][TL::MT];
#pragma unroll
  for (int a = 0; a < TL::NA; ++a)
#pragma unroll
    for (int b = 0; b < TL::MT; ++b) acc[a][b] = float4v{0.f, 0.f, 0.f, 0.f};
  const int t16 = lane & 15, q = lane >> 4, frag = t16 * 64 + ((q ^ swz(t16)) << 4);
  const int KT = src.KT;
#pragma unroll
  for (int s = 0; s < TL::NS - 1; ++s)
    if (s < KT) issue(s, s);
  int stage = 0, nstage = TL::NS - 1;
  for (int kt = 0; kt < KT; ++kt) {
    // block kt has landed (own loads), then everyone's; the stage refilled below was
    // read during iteration kt - 1, which every wavefront has left with its reads completed
    if (kt + TL::NS - 2 < KT) wait_vm<(TL::NS - 2) * TL::PER_WAVE>(); else wait_vm<0>();
    wait_lds();
    __builtin_amdgcn_s_barrier();
    if (kt + TL::NS - 1 < KT) issue(kt + TL::NS - 1, nstage);
    const char* sb = smem + stage * TL::STAGE_BYTES + frag;
    half8 fa[TL::NA], fb[TL::MT];
#pragma unroll
    for (int a = 0; a < TL::NA; ++a) fa[a] = *(const half8*)(sb + a * 1024);
#pragma unroll
    for (int b = 0; b < TL::MT; ++b) fb[b] = *(const half8*)(sb + (TL::BN + wave * TL::WM + b * 16) * 64);
#pragma unroll
    for (int b = 0; b < TL::MT; ++b)
#pragma unroll
      for (int a = 0; a < TL::NA; ++a) acc[a][b] = mfma32(fa[a], fb[b], acc[a][b]);
    stage = (stage + 1 == TL::NS) ? 0 : stage + 1;
    nstage = (nstage + 1 == TL::NS) ? 0 : nstage + 1;
  }
  TileCtx ctx{c, 0, 0, m0, m_end, 0, wave, lane, tid, (half_t*)smem, false, 0};
  epi.template run<TL>(ctx, acc);
}

// ---------------------------------------------------------------- epilogue: plain store
// out[p][n] = acc (f16 or f32), rows p in cluster-sorted order.  A lane writes the eight
// consecutive outputs of a pair block for its token in one piece.
template <class OutT>
struct EpiStoreT {
  static constexpr bool SPLITS = false, EXTENDS = false, PANELS = false;
  using Quarter = TileQuad;
  OutT* out;
  const int* rowmap;  // row p of the tile order is written to out[rowmap[p]] (NULL: identity)
  int ldo, N;
  template <class TL>
  static constexpr int smem_bytes() { return TL::SMEM_BYTES; }
  template <class TL>
  __device__ void run(const TileCtx& t, float4v (&acc)[TL::NA][TL::MT]) const {
    const int t16 = t.lane & 15, q = t.lane >> 4;
#pragma unroll
    for (int b = 0; b < TL::MT; ++b) {
      const int p = t.m0 + t.wm * TL::WM + b * 16 + t16;
      if (p >= t.m_end) continue;
      const size_t orow = rowmap ? rowmap[p] : p;
#pragma unroll
      for (int P = 0; P < TL::NP; ++P) {
        const int nb = t.n0 + t.wn * TL::WN + 32 * P + 8 * q;
        if (nb >= N) continue;   // N is a multiple of 8
        if constexpr (sizeof(OutT) == 2) {
          *(half8*)(out + orow * ldo + nb) = pack_half8(acc[2 * P][b], acc[2 * P + 1][b]);
        } else {
          *(float4v*)(out + orow * ldo + nb) = acc[2 * P][b];
          *(float4v*)(out + orow * ldo + nb + 4) = acc[2 * P + 1][b];
        }
      }
    }
  }
};
using EpiStore = EpiStoreT<half_t>;

// The same in 32-column blocks, out[n / 32][p][n % 32] (rows p in tile order): the layout in which the
// middle of the backward pass and a further product read whole KiBs.
struct EpiStoreBlocked {
  static constexpr bool SPLITS = false, EXTENDS = false, PANELS = false;
  using Quarter = TileQuad;
  half_t* out;
  int T, N;
  template <class TL>
  static constexpr int smem_bytes() { return TL::SMEM_BYTES; }
  template <class TL>
  __device__ void run(const TileCtx& t, float4v (&acc)[TL::NA][TL::MT]) const {
    const int t16 = t.lane & 15, q = t.lane >> 4;
#pragma unroll
    for (int b = 0; b < TL::MT; ++b) {
      const int p = t.m0 + t.wm * TL::WM + b * 16 + t16;
      if (p >= t.m_end) continue;
#pragma unroll
      for (int P = 0; P < TL::NP; ++P) {
        const int nb = t.n0 + t.wn * TL::WN + 32 * P;
        if (nb >= N) continue;   // N is a multiple of 32
        *(half8*)(out + ((size_t)(nb >> 5) * T + p) * 32 + 8 * q) = pack_half8(acc[2 * P][b], acc[2 * P + 1][b]);
      }
    }
  }
};

// ---------------------------------------------------------------- epilogue: input gradient
// acc = (B1^T sum_j dh_j) blocks (rows n of d).  Adds the rank part of the pairs as one more contraction
// over the cluster's rank rows, V1cat^T qext (qext[m][e_j r + rho] = q_j[rho], as EpiDownCombine does
// for the second matrix), and the gate path sum_j dl_j v_{e_j} in FP32, and writes FP32 rows in
// token order.  The panel V1cat is stored with the contraction index along its rows, so its
// fragments are transposing LDS reads.  K*r <= 128, k <= 2.  A panel value that is not finite stays with its expert's
// tokens as in the middle kernel (cmoe_backward_mid.hip).
struct EpiInputGrad {
  static constexpr bool SPLITS = false, EXTENDS = false, PANELS = false;
  using Quarter = TileQuad;
  const half_t* v1cat;          // [G][KRp][d]
  const int* offe;              // [G K + 1] pair rows of the experts: the panel rows of an expert without any are zero
  const half_t* q;              // [T][k][r], tile order
  const int* es;                // [T][k] experts local to the cluster, tile order
  const int* rperm;             // token of tile row p
  const float* dl;              // [T][k], token order
  const half_t* router_expert;  // [G K][d]
  float* dx;                    // [T][d], token order
  int k, K, r, KRp, d;
  template <class TL>
  static constexpr int panel_bytes() { return 128 * (TL::BN + 8) * 2; }
  template <class TL>
  static constexpr int smem_bytes() {
    constexpr int need = panel_bytes<TL>() + TL::BM * (128 + 8) * 2 + 16;
    return need > TL::SMEM_BYTES ? need : TL::SMEM_BYTES;
  }
  template <class TL>
  __device__ void run(const TileCtx& t, float4v (&acc)[TL::NA][TL::MT]) const {
    const int t16 = t.lane & 15, q4 = t.lane >> 4;
    constexpr int LDV = TL::BN + 8;
    const int lds = KRp + 8, n_chunks = KRp / 32;
    half_t* sV = t.smem;                                // [KRp][LDV]
    half_t* sS = t.smem + panel_bytes<TL>() / 2;        // [BM][lds]
    int* s_apart = (int*)(sS + TL::BM * (128 + 8));     // a panel value is not finite
    const half_t* vc = v1cat + (size_t)t.c * KRp * d;
    bool bad = false;
    __syncthreads();  // the stage buffers are free
    if (t.tid == 0) *s_apart = 0;
    constexpr int CPR = TL::BN / 8;
    for (int idx = t.tid; idx < KRp * CPR; idx += TL::NT) {
      const int row = idx / CPR, ch = idx % CPR;
      const int e = t.c * K + min(row / r, K - 1);
      half8 v = *(const half8*)(vc + (size_t)row * d + min(t.n0 + ch * 8, d - 8));
      if (offe[e + 1] == offe[e]) v = half8{0, 0, 0, 0, 0, 0, 0, 0};
      bad |= not_finite(v);
      *(half8*)(sV + row * LDV + ch * 8) = v;
    }
    for (int i = t.tid; i < TL::BM * lds / 8; i += TL::NT) ((half8*)sS)[i] = half8{0, 0, 0, 0, 0, 0, 0, 0};
    __syncthreads();
    if (bad) *s_apart = 1;
    const int r4 = r / 4;
    for (int idx = t.tid; idx < TL::BM * k * r4; idx += TL::NT) {
      const int rho = idx % r4 * 4, j = (idx / r4) % k, m = idx / (r4 * k), p = t.m0 + m;
      if (p >= t.m_end) continue;
      const int* ep = es + (size_t)p * k;
      const half_t* qp = q + (size_t)p * k * r + rho;
      half4 v = *(const half4*)(qp + j * r);
      // a token that names its expert twice: the sum of both, which both of its pairs write (k <= 2)
      if (k == 2 && ep[0] == ep[1]) {
        const half4 o = *(const half4*)(qp + (1 - j) * r);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (half_t)((float)v[i] + (float)o[i]);
      }
      *(half4*)(sS + m * lds + ep[j] * r + rho) = v;
    }
    __syncthreads();
    const bool apart = __builtin_amdgcn_readfirstlane(*s_apart) != 0;
#pragma unroll
    for (int b = 0; b < TL::MT; ++b) {
      const int m = t.wm * TL::WM + b * 16 + t16, p = t.m0 + m;
      const bool valid = p < t.m_end;
      const size_t pc = valid ? p : t.m_end - 1;
      const size_t tok = rperm[pc];
      unsigned mine = 0;
      for (int j = 0; j < k; ++j) {
        const int e = es[pc * k + j];
        mine |= (0xffffffffu >> (31 - ((e * r + r - 1) >> 5))) & (0xffffffffu << ((e * r) >> 5));
      }
      if (!valid) mine = 0;
      unsigned cmask = 0;
      for (int kc = 0; kc < n_chunks; ++kc)
        if (__ballot((mine >> kc) & 1u) != 0ull) cmask |= 1u << kc;
#pragma unroll
      for (int P = 0; P < TL::NP; ++P) {
        const int nl = t.wn * TL::WN + 32 * P;
        if (t.n0 + nl >= d) continue;
        // rows n = 8 (i / 4) + 4 hh + i % 4 of the pair block, contraction elements 32 kc + 8 q4 ..
        auto frag_v = [&](int kc, int hh) {
          const half_t* a0 = sV + (kc * 32 + 8 * q4 + (t16 >> 2)) * LDV + nl + 8 * (t16 & 3) + 4 * hh;
          return join8(lds_read_tr(a0), lds_read_tr(a0 + 4 * LDV));
        };
        if (__builtin_expect(!apart, 1)) {
          for (unsigned mm = cmask; mm != 0u; mm &= mm - 1u) {
            const int kc = __builtin_ctz(mm);
            const half8 fb = *(const half8*)(sS + m * lds + kc * 32 + 8 * q4);
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) acc[2 * P + hh][b] = mfma32(frag_v(kc, hh), fb, acc[2 * P + hh][b]);
          }
        } else {
          for (int e = 0; e < K; ++e) {
            bool own = false;
            for (int j = 0; j < k; ++j) own |= valid && es[pc * k + j] == e;
            if (__ballot(own) == 0ull) continue;
            const int kc = (e * r) >> 5;
            const half8 fb = *(const half8*)(sS + m * lds + kc * 32 + 8 * q4);
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
              const float4v x = mfma32(rows_of_expert(frag_v(kc, hh), kc * 32 + 8 * q4, r, e), fb, acc[2 * P + hh][b]);
              if (own) acc[2 * P + hh][b] = x;
            }
          }
        }
        if (!valid) continue;
        float4v o0 = acc[2 * P][b], o1 = acc[2 * P + 1][b];
        for (int j = 0; j < k; ++j) {
          const float c = dl[tok * k + j];
          const half8 v = *(const half8*)(router_expert + ((size_t)t.c * K + es[pc * k + j]) * d + t.n0 + nl + 8 * q4);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            o0[i] = fmaf(c, (float)v[i], o0[i]);
            o1[i] = fmaf(c, (float)v[4 + i], o1[i]);
          }
        }
        float* dst = dx + tok * d + t.n0 + nl + 8 * q4;
        *(float4v*)dst = o0;
        *(float4v*)(dst + 4) = o1;
      }
    }
  }
};

// ---------------------------------------------------------------- epilogue: down-projection + combine
// acc = (W2_base A)^T blocks.  The residual of the second matrix is a contraction over the cluster's rank rows,
// y^T += U2cat^T sext^T with sext[p][e_j*r + rho] = g_j s_j[rho] (zero elsewhere, sext_kernel), so it is the second
// pair of operands of the main loop: KRp / 32 more blocks, and all that is left to do here is to write the rows straight to
// token order, 16 bytes per lane.  As a step of the epilogue, chains of loads by token behind the main loop, it cost 20 to
// 26 us of a 256 x 256 tile and 6 to 7 of a quarter, now 4 and 1; whole kernel, 777 tokens of 4 clusters of 1024 x 4096
// 29.5 -> 23.2 us, 4096 of 2 of 768 x 3072 33.7 -> 32.0, 16384 Zipf tokens of the former 149 -> 133, 32768 of 8 of
// 2048 x 8192 939 -> 880.
// A factor value that is not finite would reach the other tokens of the tile as 0 * inf; a tile with one (by its
// scales: apart) leaves the second pair out and adds the residual here, chunks of 32 rank rows that no token of a
// 16-token block needs skipped.  So does a contraction of less than EXT_BLOCKS blocks.  K*r <= 128.
struct EpiDownCombine {
  static constexpr bool SPLITS = true, EXTENDS = true, PANELS = false;
  using Quarter = TileQuad;
  const half_t* u2t;     // [G][d][KRp]
  const half_t* u2_s;    // [G K][r][d / qg]
  const half_t* sext;    // [KRp / 32][T][32], sorted rows
  const int* rperm;      // token of tile row p
  const int* expert_idx;
  half_t* y;             // [T][d], token order
  int k, K, r, KRp, d, qg, T;
  // Is a value of the tile's columns of U2 not finite?  |code| <= 8, so a scale up to 8188 keeps them in FP16.
  __device__ __forceinline__ bool apart(int c, int n0, int bn, int tid, int nt) const {
    const int g0 = n0 / qg, ng = (min(n0 + bn, d) - 1) / qg + 1 - g0, n = K * r * ng;
    bool bad = false;
    for (int i = tid; i < n; i += nt) {
      const int row = i / ng;
      bad |= !(fabsf((float)u2_s[((size_t)c * K * r + row) * (d / qg) + g0 + (i - row * ng)]) <= 8188.f);
    }
    return bad;
  }
  template <class TL>
  static constexpr int smem_bytes() {
    return 2 * (TL::BN + TL::BM) * (128 + 8) > TL::SMEM_BYTES ? 2 * (TL::BN + TL::BM) * (128 + 8) : TL::SMEM_BYTES;
  }
  template <class TL>
  __device__ void run(const TileCtx& t, float4v (&acc)[TL::NA][TL::MT]) const {
    const int t16 = t.lane & 15, q = t.lane >> 4;
    if (t.ext) {
      int tok[TL::MT];
#pragma unroll
      for (int b = 0; b < TL::MT; ++b) tok[b] = rperm[min(t.m0 + t.wm * TL::WM + b * 16 + t16, t.m_end - 1)];
#pragma unroll
      for (int b = 0; b < TL::MT; ++b) {
        if (t.m0 + t.wm * TL::WM + b * 16 + t16 >= t.m_end) continue;
#pragma unroll
        for (int P = 0; P < TL::NP; ++P) {
          const int n = t.n0 + t.wn * TL::WN + 32 * P;
          if (n < d) *(half8*)(y + (size_t)tok[b] * d + n + 8 * q) = pack_half8(acc[2 * P][b], acc[2 * P + 1][b]);
        }
      }
      return;
    }
    const int ldu = KRp + 8, n_chunks = KRp / 32;
    half_t* sU = t.smem;                 // [BN][ldu]  U2 rows of the tile, in MFMA order
    half_t* sS = t.smem + TL::BN * ldu;  // [BM][ldu]  expanded gated s of the tile's tokens
    const half_t* u2c = u2t + (size_t)t.c * d * KRp;
    __syncthreads();  // the stage buffers are free
    {
      constexpr int UB = 4;
      const int u_chunks = TL::BN * (KRp / 8), ucpr = KRp / 8;
      for (int base = t.tid; base < u_chunks; base += UB * TL::NT) {
        half8 tmp[UB];
#pragma unroll
        for (int i = 0; i < UB; ++i) {
          int idx = base + i * TL::NT;
          if (idx < u_chunks)
            tmp[i] = *(const half8*)(u2c + (size_t)min(t.n0 + pi_row(idx / ucpr), d - 1) * KRp + (idx % ucpr) * 8);
        }
#pragma unroll
        for (int i = 0; i < UB; ++i) {
          int idx = base + i * TL::NT;
          if (idx < u_chunks) *(half8*)(sU + (idx / ucpr) * ldu + (idx % ucpr) * 8) = tmp[i];
        }
      }
      for (int i = t.tid; i < TL::BM * ucpr; i += TL::NT) {
        const int m = i / ucpr, kk = i % ucpr * 8, p = min(t.m0 + m, t.m_end - 1);
        *(half8*)(sS + m * ldu + kk) = *(const half8*)(sext + ((size_t)(kk >> 5) * T + p) * 32 + (kk & 31));
      }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < TL::MT; ++b) {
      const int ml_t = t.wm * TL::WM + b * 16 + t16;
      const int p = t.m0 + ml_t;
      const bool valid = p < t.m_end;
      const int tok = rperm[valid ? p : t.m_end - 1];
      unsigned mine = 0;
      for (int j = 0; j < k; ++j) {
        const int e = min(max(expert_idx[(size_t)tok * k + j] - t.c * K, 0), K - 1);
        const int lo = (e * r) >> 5, hi = (e * r + r - 1) >> 5;
        mine |= (0xffffffffu >> (31 - hi)) & (0xffffffffu << lo);
      }
      if (!valid) mine = 0;
      unsigned cmask = 0;
      for (int kc = 0; kc < n_chunks; ++kc)
        if (__ballot((mine >> kc) & 1u) != 0ull) cmask |= 1u << kc;
#pragma unroll
      for (int P = 0; P < TL::NP; ++P) {
        const int nl = t.wn * TL::WN + 32 * P;
        if (t.n0 + nl >= d) continue;
        for (int kc = 0; kc < n_chunks; ++kc) {
          if (!((cmask >> kc) & 1u)) continue;
          const half8 fb = *(const half8*)(sS + ml_t * ldu + kc * 32 + 8 * q);
          const half8 fa0 = *(const half8*)(sU + (nl + t16) * ldu + kc * 32 + 8 * q);
          const half8 fa1 = *(const half8*)(sU + (nl + 16 + t16) * ldu + kc * 32 + 8 * q);
          acc[2 * P][b] = mfma32(fa0, fb, acc[2 * P][b]);
          acc[2 * P + 1][b] = mfma32(fa1, fb, acc[2 * P + 1][b]);
        }
        if (valid) *(half8*)(y + (size_t)tok * d + t.n0 + nl + 8 * q) = pack_half8(acc[2 * P][b], acc[2 * P + 1][b]);
      }
    }
  }
};

// ---------------------------------------------------------------- epilogue: fused up-projection
// acc = Hb^T blocks (rows n of d_ff, columns = tokens).  Per token column and selected
// expert j:  h_j = Hb + U1cat^T t1ext_j with t1ext_j the token's t1_j placed at the rank rows
// of expert e_j and zero elsewhere (matrix core, contraction over the cluster's K*r rank
// rows in chunks of 32; a chunk no token of the 16-token block needs is skipped);
// a_j = GELU(h_j); A += g_j a_j; s_j += V2 a_j by feeding the a_j pair block back as B operand
// (contraction over its 32 rows n).  The V2 product runs over "passes" of 16 rank rows; a
// lane contributes to a pass only if its token's expert lies in it.
// With STAGE the U1 / V2 panels of the tile are staged through LDS (K*r <= 128), in portions of 32 rank rows that the
// tile has under way while it works on its last blocks (PANELS); otherwise they are read from global memory.  Panels and
// token state loaded behind the main loop, through registers, cost 4 us of a 256 x 256 tile for 32 rank rows and 9 for
// 128, now 0.6 and 1.5; whole kernel, with a GELU of ten operations (of eleven, as it is now, 1 to 3 % more), 4096 tokens of 2
// clusters of 768 x 3072 46.6 -> 42.7 us, 16384 Zipf tokens of 4 of 1024 x 4096 246 -> 222, 32768 of 8 of 2048 x 8192 1450 -> 1390.
template <int R, int KMAX, bool STAGE>
struct EpiFusedUp {
  static constexpr bool SPLITS = false, EXTENDS = false, PANELS = STAGE;
  using Quarter = TileSlab;   // one s partial per 256 rows of d_ff whatever the tile
  const half_t* u1t;  // [G][d_ff][KRp]
  const half_t* v2p;  // [G][KRp][d_ff]
  const half_t* t1;   // [T][k][r], sorted rows
  const int* perm;
  const int* expert_idx;
  const float* gate;
  half_t* A;          // [d_ff / 32][T][32]
  float* spart;       // [n_tiles][T][k][r] partials of V2 a over the tile's rows of d_ff, FP32
  int T, k, K, KRp, d_ff;
  bool t1_by_token;   // t1 is in token order (TOK_T1 and rows of whole 16 bytes only)
  using FU = FusedUp<R, KMAX>;

  __device__ __forceinline__ int portions() const { return KRp / 32; }
  // A portion: 256 rows of U1 (tile order) x 32 rank rows, then for each of the tile's 8 pair blocks 32 rank rows of V2 x its 32
  // columns; rows of 64 bytes, chunks at swz(row) as in the operand stages.  Source of the lane's 16 bytes of a piece of the
  // first portion, and elements from there to the next.
  __device__ __forceinline__ const half_t* panel_src(int c, int n0, int piece, int lane) const {
    const int row = piece * 16 + (lane >> 2), pos = lane & 3;
    if (piece < 16) return u1t + ((size_t)c * d_ff + min(n0 + pi_row(row), d_ff - 1)) * KRp + ((pos ^ swz(row)) << 3);
    const int rank = row & 31;
    return v2p + ((size_t)c * KRp + rank) * d_ff + min(n0 + ((row - 256) & ~31), d_ff - 32) + ((pos ^ swz(rank)) << 3);
  }
  __device__ __forceinline__ size_t panel_step(int piece) const { return piece < 16 ? 32 : (size_t)32 * d_ff; }
  template <class TL>
  static constexpr int panel_bytes() {
    return STAGE && PANEL_SLOTS * PANEL_BYTES > TL::SMEM_BYTES ? PANEL_SLOTS * PANEL_BYTES : TL::SMEM_BYTES;
  }
  // With STAGE and up to two experts per token, the tokens' experts, gates and (up to 32 halfs each) t1 rows are brought to
  // LDS while the tile's first blocks are under way: behind the main loop the chain of loads rows, experts and gates
  // costs 3 to 5 us of a tile.
  static constexpr bool TOK = STAGE && KMAX <= 2, TOK_T1 = TOK && KMAX * R <= 32;
  template <class TL>   // experts and gates, then t1 in whole KiBs as the loads bring it (64 rows of 8 bytes are half of one)
  static constexpr int tok_bytes() { return TOK ? TL::BM * KMAX * 8 + (TOK_T1 ? (TL::BM * KMAX * R * 2 + 1023) / 1024 * 1024 : 0) : 0; }
  // The last BM threads take a token each: their wavefronts wait for rows of perm anyway.
  template <class TL>
  __device__ __forceinline__ int token(int tid, int m0, int m_end) const {
    return TOK && tid >= TL::NT - TL::BM ? perm[min(m0 + tid - (TL::NT - TL::BM), m_end - 1)] : 0;
  }
  template <class TL>
  __device__ __forceinline__ void put_tokens(int tok, int tid, int m0, unsigned smem_base) const {
    if constexpr (TOK) {
      static_assert(!TOK_T1 || (tok_bytes<TL>() - TL::BM * KMAX * 8) % 1024 == 0, "a piece of t1 is a KiB");
      const int kr = k * R, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
      const unsigned at = smem_base + panel_bytes<TL>();
      constexpr int FIRST = (TL::NT - TL::BM) / 64;
      if (TOK_T1 && t1_by_token) {
        if (wave >= FIRST) {
          const int lane = tid & 63, per = kr >> 3;   // 16-byte pieces of a row, a power of two
          for (int i = 0; i < per; ++i) {
            const int piece = i * 64 + lane, from = __shfl(tok, piece / per, 64);
            dma16(t1 + (size_t)from * kr + (piece & (per - 1)) * 8,
                  at + TL::BM * KMAX * 8 + (wave - FIRST) * 128 * kr + i * 1024);
          }
        }
      } else if constexpr (TOK_T1) {
        // Rows past the last are read from there and not used.  A piece of 16 bytes is one row or part of one, or two rows of
        // four halfs: then the very last may reach 8 bytes past the rows, into what follows them in the workspace, and its
        // address is a multiple of 8 bytes only, where the load asks for 4.
        const long last = (long)T * kr - min(kr, 8);
        for (int i = wave; i * 512 < TL::BM * kr; i += TL::NWAVES)
          dma16(t1 + min((long)m0 * kr + i * 512 + (tid & 63) * 8, last), at + TL::BM * KMAX * 8 + i * 1024);
      }
      if (wave >= FIRST) {
#pragma unroll
        for (int j = 0; j < KMAX; ++j)
          if (j < k) {
            dma4(expert_idx + (size_t)tok * k + j, at + (j * TL::BM + (wave - FIRST) * 64) * 4);
            dma4(gate + (size_t)tok * k + j, at + ((KMAX + j) * TL::BM + (wave - FIRST) * 64) * 4);
          }
      }
    }
  }
  // the state of the token of tile row m
  template <class TL>
  __device__ __forceinline__ void get_token(typename FU::Tok& t, int m, int c, int m0, int m_end, int q, const char* smem) const {
    t.p = m0 + m;
    t.valid = t.p < m_end;
    const int* es = (const int*)(smem + panel_bytes<TL>());
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      t.e[j] = 0;
      t.g[j] = 0.f;
      t.f[j] = half8{0, 0, 0, 0, 0, 0, 0, 0};
      if (j < k) {
        t.e[j] = min(max(es[j * TL::BM + m] - c * K, 0), K - 1);
        t.g[j] = t.valid ? ((const float*)es)[(KMAX + j) * TL::BM + m] : 0.f;
        if constexpr (TOK_T1)
          FU::load_t1(t.f[j], (const half_t*)(es + 2 * KMAX * TL::BM) + ((size_t)m * k + j) * R, q);
        else
          FU::load_t1(t.f[j], t1 + ((size_t)min(t.p, m_end - 1) * k + j) * R, q);
      }
    }
  }
  // The WAVES_N wavefronts that share a token block add their s partials through LDS.  With up
  // to two experts per token the partials of all token blocks are exchanged at the end, in
  // the space of the panels (no longer needed then); otherwise block by block through an
  // area of its own behind the panels.
  static constexpr bool BATCH = KMAX <= 2;
  template <class TL>
  static constexpr int xs_floats() { return (BATCH ? TL::MT * KMAX * FU::NSP : 1) * 4 * 64; }   // per wavefront
  template <class TL>
  static constexpr int xs_bytes() { return TL::WAVES_M * (BATCH ? TL::WAVES_N : TL::WAVES_N - 1) * xs_floats<TL>() * 4; }
  template <class TL>
  static constexpr int smem_bytes() {
    static_assert(!BATCH || xs_bytes<TL>() <= TL::SMEM_BYTES, "exchange area");
    return panel_bytes<TL>() + tok_bytes<TL>() + (BATCH ? 0 : xs_bytes<TL>());
  }

  template <class TL>
  __device__ void run(const TileCtx& t, float4v (&acc)[TL::NA][TL::MT]) const {
    static_assert(TL::BN == TileBig::BN, "one s partial per tile, summed over its wavefront columns");
    const int t16 = t.lane & 15, q = t.lane >> 4;
    const half_t* u1c = u1t + (size_t)t.c * d_ff * KRp;
    const half_t* v2c = v2p + (size_t)t.c * KRp * d_ff;
    const int n_chunks = KRp / 32, n_pass = KRp / 16;
    if (STAGE) {
      wait_vm<0>();
      __builtin_amdgcn_s_barrier();   // the panels and tokens are there
    }
    // per-lane token state of a 16-token block: from LDS, or of all blocks up front while it fits the registers, or block
    // by block
    constexpr bool PRELOAD = KMAX <= 2 && !TOK;
    typename FU::Tok pre[PRELOAD ? TL::MT : 1];
    auto token_of = [&](typename FU::Tok& tk, int b) {
      const int m = t.wm * TL::WM + b * 16 + t16;
      if constexpr (TOK)
        get_token<TL>(tk, m, t.c, t.m0, t.m_end, q, (const char*)t.smem);
      else
        FU::load_tok(tk, t.m0 + m, t.m_end, t.c, K, k, perm, expert_idx, gate, t1, q);
    };
    if constexpr (PRELOAD) {
#pragma unroll
      for (int b = 0; b < TL::MT; ++b) token_of(pre[b], b);
    }

    // LDS bytes of portion `c` of the panels
    auto portion = [&](int c) { return (const char*)t.smem + ((t.first_slot + c) & 3) * PANEL_BYTES; };
    const int in_row = t16 * 64 + ((q ^ swz(t16)) << 4);   // of row t16 of 16 rows of a portion

    // with few experts per token the s partials of all token blocks are kept and exchanged
    // at the end in one go; otherwise block by block
    constexpr int NSB = BATCH ? TL::MT : 1;
    float4v sacc[NSB][KMAX][FU::NSP];
    // block by block: partials of wavefront column wn >= 1 of token column wm
    auto xs = [&](int wn) {
      return (float*)((char*)t.smem + panel_bytes<TL>()) + ((wn - 1) * TL::WAVES_M + t.wm) * xs_floats<TL>() + t.lane;
    };
#pragma unroll
    for (int b = 0; b < TL::MT; ++b) {
      const int sb = BATCH ? b : 0;
#pragma unroll
      for (int j = 0; j < KMAX; ++j)
#pragma unroll
        for (int s2 = 0; s2 < FU::NSP; ++s2) sacc[sb][j][s2] = float4v{0.f, 0.f, 0.f, 0.f};
      const int p = t.m0 + t.wm * TL::WM + b * 16 + t16;
      typename FU::Tok own;
      if constexpr (!PRELOAD) token_of(own, b);
      const typename FU::Tok& tkb = PRELOAD ? pre[PRELOAD ? b : 0] : own;
      typename FU::Need nd;
      FU::need_of(tkb, k, n_chunks, n_pass, nd);
      if (BATCH && nd.chunks[0] == 0u) continue;   // no token of the group
      // With the operands in LDS only: as loads from memory they wait in registers, 12 to 28 more than there are.  4096 tokens of
      // 8 clusters of 4096 x 14336, rank 32, 892 -> 879 us (kernel) without, 2500 of 4 of 1024 x 4096 96.9 -> 93.4, 1024 of
      // those with 16 experts of rank 16 87.3 -> 84.0.
      constexpr bool AHEAD = STAGE && KMAX <= 2;
      typename FU::Ahead ahead;
#pragma unroll
      for (int P = 0; P < TL::NP; ++P) {
        const int nl = t.wn * TL::WN + 32 * P;  // first row of the pair block inside the tile
        const int nb = t.n0 + nl;
        if (nb >= d_ff) continue;
        auto uf_at = [&](int nl) {
          return [&, nl](int c, int hh) {
            return STAGE ? *(const half8*)(portion(c) + (nl + 16 * hh) * 64 + in_row)
                         : *(const half8*)(u1c + (size_t)(t.n0 + nl + pi_row(16 * hh + t16)) * KRp + c * 32 + 8 * q);
          };
        };
        auto vf = [&](int pp) {
          return STAGE ? *(const half8*)(portion(pp >> 1) + (256 + nl + 16 * (pp & 1)) * 64 + in_row)
                       : *(const half8*)(v2c + (size_t)(pp * 16 + t16) * d_ff + nb + 8 * q);
        };
        float o[8];
        if constexpr (AHEAD) {
          if (P == 0) FU::start(ahead, tkb, nd, q, uf_at(nl));
          FU::pair_block_ahead(acc[2 * P][b], acc[2 * P + 1][b], tkb, nd, q, ahead, P + 1 < TL::NP && nb + 32 < d_ff, uf_at(nl),
                               vf, uf_at(nl + 32), o, sacc[sb]);
        } else {
          FU::pair_block(acc[2 * P][b], acc[2 * P + 1][b], tkb, nd, k, q, uf_at(nl), vf, o, sacc[sb]);
        }
        // A[p][nb + 8q .. nb + 8q + 8) in 32-column blocks ([d_ff / 32][T][32], the operand
        // layout of the down-projection): 16 bytes per lane, four lanes a token's 64 bytes,
        // the block's 16 tokens 1 KiB of contiguous memory
        if (p < t.m_end) {
          half8 o8;
#pragma unroll
          for (int i = 0; i < 8; ++i) o8[i] = (half_t)o[i];
          *(half8*)(A + ((size_t)(nb >> 5) * T + p) * 32 + 8 * q) = o8;
        }
      }
      if (!BATCH) {
        // the wavefronts that share these tokens add their partial s through LDS, one
        // accumulator at a time; wn = 0 stores the tile's partial
        __syncthreads();
#pragma unroll
        for (int j = 0; j < KMAX; ++j) {
          if (j >= k) continue;
#pragma unroll
          for (int s2 = 0; s2 < FU::NSP; ++s2) {
            if (t.wn != 0) {
              float* x = xs(t.wn);
#pragma unroll
              for (int v = 0; v < 4; ++v) x[v * 64] = sacc[0][j][s2][v];
            }
            __syncthreads();
            if (t.wn == 0) {
#pragma unroll
              for (int w = 1; w < TL::WAVES_N; ++w) {
                const float* x = xs(w);
#pragma unroll
                for (int v = 0; v < 4; ++v) sacc[0][j][s2][v] += x[v * 64];
              }
            }
            __syncthreads();
          }
        }
        if (t.wn == 0) FU::store_s(tkb, sacc[0], spart + (size_t)t.n_tile * T * k * R, k, q);
      }
    }
    if (BATCH) {
      // all token blocks at once: the WAVES_N wavefronts of a token column share them out, each adds up its own
      // over the wavefronts in order and stores them
      constexpr int OWN = TL::MT / TL::WAVES_N > 0 ? TL::MT / TL::WAVES_N : 1;
      auto owner = [&](int b) { return b / OWN; };
      __syncthreads();
      float* xb = (float*)t.smem + (size_t)t.wm * TL::WAVES_N * xs_floats<TL>() + t.lane;   // of this token column
#pragma unroll
      for (int b = 0; b < NSB; ++b)
        if (owner(b) != t.wn) {
#pragma unroll
          for (int j = 0; j < KMAX; ++j)
#pragma unroll
            for (int s2 = 0; s2 < FU::NSP; ++s2)
#pragma unroll
              for (int v = 0; v < 4; ++v)
                xb[t.wn * xs_floats<TL>() + (((b * KMAX + j) * FU::NSP + s2) * 4 + v) * 64] = sacc[b][j][s2][v];
        }
      __syncthreads();
#pragma unroll
      for (int b = 0; b < NSB; ++b)
        if (owner(b) == t.wn) {
          float4v sum[KMAX][FU::NSP];
#pragma unroll
          for (int w = 0; w < TL::WAVES_N; ++w)
#pragma unroll
            for (int j = 0; j < KMAX; ++j)
#pragma unroll
              for (int s2 = 0; s2 < FU::NSP; ++s2)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                  const float x = w == t.wn ? sacc[b][j][s2][v]
                                            : xb[w * xs_floats<TL>() + (((b * KMAX + j) * FU::NSP + s2) * 4 + v) * 64];
                  sum[j][s2][v] = w == 0 ? x : sum[j][s2][v] + x;
                }
          typename FU::Tok own;
          if constexpr (!PRELOAD) token_of(own, b);
          FU::store_s(PRELOAD ? pre[PRELOAD ? b : 0] : own, sum, spart + (size_t)t.n_tile * T * k * R, k, q);
        }
    }
  }
};

// ---------------------------------------------------------------- s partial reduction
// s_down[perm[p]][w] = sum over row tiles of spart[tile][p][w], in a fixed order: a block
// owns 256 consecutive outputs (four per lane, k * r is a multiple of 4 so they belong to one
// token), its NW wavefronts each sum every NW-th tile, and the NW sums are added in
// wavefront order.
template <int NW, class ST>
__global__ __launch_bounds__(64 * NW) void sreduce_kernel(const ST* __restrict__ spart,
                                                          const int* __restrict__ perm, int T, int kr, int n_tiles,
                                                          float* __restrict__ s_down) {
  __shared__ float4v part[NW][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const size_t total = (size_t)T * kr;
  const size_t idx = ((size_t)blockIdx.x * 64 + lane) * 4;
  float4v sum = {0.f, 0.f, 0.f, 0.f};
  if (idx < total) {
#pragma unroll 8
    for (int nt = wave; nt < n_tiles; nt += NW) sum += *(const float4v*)(spart + (size_t)nt * total + idx);
  }
  part[wave][lane] = sum;
  __syncthreads();
  if (wave == 0 && idx < total) {
    float4v s2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) s2 += part[w][lane];
    *(float4v*)(s_down + (size_t)perm[idx / kr] * kr + idx % kr) = s2;
  }
}

// The same for the down-projection that is joined with the combine, as the operand of its main loop: the gated sums
// g_j s_j in FP16 at the rank rows of expert e_j, zero elsewhere, sext [KRp / 32][T][32] in sorted rows.  A block owns
// 256 / (k r) whole rows.
template <int NW>
__global__ __launch_bounds__(64 * NW) void sext_kernel(const float* __restrict__ spart, const int* __restrict__ perm,
                                                       const int* __restrict__ expert_idx, const float* __restrict__ gate,
                                                       int T, int K, int k, int r, int KRp, int n_tiles,
                                                       half_t* __restrict__ sext, int* __restrict__ zero) {
  __shared__ float4v part[NW][64];
  __shared__ __attribute__((aligned(16))) half_t out[64 * 128];   // at most 64 rows (k r = 4), KRp <= 128
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (zero != nullptr && blockIdx.x == 0)
    for (int i = tid; i < GEMM_PARTS; i += 64 * NW) zero[i] = 0;
  const int kr = k * r, rows = 256 / kr, p0 = blockIdx.x * rows, lr = lane * 4 / kr, at = lane * 4 - lr * kr, p = p0 + lr;
  const bool in = lr < rows && p < T;
  int slot = 0;
  float g = 0.f;
  if (wave == 0 && in) {
    const size_t pair = (size_t)perm[p] * k + at / r;
    slot = expert_idx[pair] % K;
    g = gate[pair];
  }
  float4v sum = {0.f, 0.f, 0.f, 0.f};
  if (in) {
    const float* src = spart + (size_t)p * kr + at;
#pragma unroll 8
    for (int nt = wave; nt < n_tiles; nt += NW) sum += *(const float4v*)(src + (size_t)nt * T * kr);
  }
  part[wave][lane] = sum;
  for (int i = tid; i < rows * KRp / 8; i += 64 * NW) ((half8*)out)[i] = half8{0, 0, 0, 0, 0, 0, 0, 0};
  __syncthreads();
  if (wave == 0 && in) {
    float4v s2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) s2 += part[w][lane];
    *(half4*)(out + lr * KRp + slot * r + at % r) =
        half4{(half_t)(g * s2[0]), (half_t)(g * s2[1]), (half_t)(g * s2[2]), (half_t)(g * s2[3])};
  }
  __syncthreads();
  for (int i = tid; i < rows * KRp / 8; i += 64 * NW) {
    const int blk = i / (4 * rows), rem = i - blk * 4 * rows, row = rem >> 2;
    if (p0 + row < T)
      *(half8*)(sext + ((size_t)blk * T + p0 + row) * 32 + (rem & 3) * 8) = *(const half8*)(out + row * KRp + blk * 32 + (rem & 3) * 8);
  }
}

// ---------------------------------------------------------------- combine
// y[perm[p]] = Yb[p] + U2cat^T (d x K*r) . sext[p],   sext[p][e_j*r + rho] = g_j s_j[rho].
// One workgroup: 32 sorted rows x NSPAN blocks of 32 output columns; the expanded,
// gated s vectors of the 32 rows are built once in LDS as f16.
constexpr int CB_WAVES = 4;
constexpr int CB_NPW = 4;  // 32-column blocks per wavefront

__global__ __launch_bounds__(CB_WAVES * 64) void combine_kernel(
    const half_t* __restrict__ u2t, const half_t* __restrict__ yb, const float* __restrict__ s_down,
    const int* __restrict__ perm, const int* __restrict__ offsets, const int* __restrict__ expert_idx,
    const float* __restrict__ gate, int G, int K, int k, int r, int KRp, int d, int n_groups,
    half_t* __restrict__ y) {
  __shared__ __attribute__((aligned(16))) half_t sext[32 * (512 + 8)];
  __shared__ unsigned s_cmask;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, ml = lane & 31;
  const int ngrp = blockIdx.x % n_groups;
  int slot = blockIdx.x / n_groups;
  int c = 0, m0 = 0, m_end = 0;
  for (; c < G; ++c) {
    int lo = offsets[c], hi = offsets[c + 1];
    int tiles = (hi - lo + 31) / 32;
    if (slot < tiles) {
      m0 = lo + slot * 32;
      m_end = hi;
      break;
    }
    slot -= tiles;
  }
  if (c == G) return;
  const int lds = KRp + 8;
  for (int i = tid; i < 32 * lds / 8; i += CB_WAVES * 64) ((half8*)sext)[i] = half8{0, 0, 0, 0, 0, 0, 0, 0};
  if (tid == 0) s_cmask = 0;
  __syncthreads();
  for (int idx = tid; idx < 32 * k * r; idx += CB_WAVES * 64) {
    int rho = idx % r, j = (idx / r) % k, m = idx / (r * k);
    int p = m0 + m;
    if (p >= m_end) continue;
    int tok = perm[p];
    int e = min(max(expert_idx[(size_t)tok * k + j] - c * K, 0), K - 1);
    float v = gate[(size_t)tok * k + j] * s_down[((size_t)tok * k + j) * r + rho];
    sext[m * lds + e * r + rho] = (half_t)v;
    if (rho == 0) atomicOr(&s_cmask, (0xffffffffu >> (31 - (e * r + r - 1) / 16)) & (0xffffffffu << ((e * r) / 16)));
  }
  __syncthreads();
  const unsigned cmask = s_cmask;
  const int p = m0 + ml;
  const bool valid = p < m_end;
  const int tok = valid ? perm[p] : 0;
  const half_t* u2c = u2t + (size_t)c * d * KRp;
  const int n_chunks = KRp / 16;
  for (int i = 0; i < CB_NPW; ++i) {
    int nb = ((ngrp * CB_WAVES + wave) * CB_NPW + i) * 32;
    if (nb >= d) break;
    float16v acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    const half_t* u2row = u2c + (size_t)(nb + ml) * KRp + 8 * h;
    for (int kc = 0; kc < n_chunks; ++kc) {
      if (!((cmask >> kc) & 1u)) continue;
      half8 fa = *(const half8*)(u2row + kc * 16);
      half8 fb = *(const half8*)(sext + ml * lds + kc * 16 + 8 * h);
      acc = mfma16(fa, fb, acc);
    }
    if (valid) {
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        int n = nb + 8 * qd + 4 * h;
        half4 b4 = *(const half4*)(yb + (size_t)p * d + n);
        half4 o;
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = (half_t)(acc[4 * qd + v] + (float)b4[v]);
        *(half4*)(y + (size_t)tok * d + n) = o;
      }
    }
  }
}

template <int R, int KMAX>
hipError_t launch_gemm1_rk(const cmoe_dims& dm, const GemmArgs& g, int T, const int* perm, const int* expert_idx,
                           const float* gate, const half_t* u1t, const half_t* v2p, const half_t* t1, bool t1_by_token,
                           half_t* a, float* spart, hipStream_t st) {
  if (dm.KRp <= 128) {
    EpiFusedUp<R, KMAX, true> epi{u1t, v2p, t1, perm, expert_idx, gate, a, spart, T, dm.k, dm.K, dm.KRp, dm.d_ff, t1_by_token};
    return launch_gemm(g, T, epi, st);
  }
  EpiFusedUp<R, KMAX, false> epi{u1t, v2p, t1, perm, expert_idx, gate, a, spart, T, dm.k, dm.K, dm.KRp, dm.d_ff, false};
  return launch_gemm(g, T, epi, st);
}

template <int R>
hipError_t launch_gemm1_r(const cmoe_dims& dm, const GemmArgs& g, int T, const int* perm, const int* expert_idx,
                          const float* gate, const half_t* u1t, const half_t* v2p, const half_t* t1, bool t1_by_token,
                          half_t* a, float* spart, hipStream_t st) {
  if (dm.k <= 1) return launch_gemm1_rk<R, 1>(dm, g, T, perm, expert_idx, gate, u1t, v2p, t1, t1_by_token, a, spart, st);
  if (dm.k <= 2) return launch_gemm1_rk<R, 2>(dm, g, T, perm, expert_idx, gate, u1t, v2p, t1, t1_by_token, a, spart, st);
  if (dm.k <= 4) return launch_gemm1_rk<R, 4>(dm, g, T, perm, expert_idx, gate, u1t, v2p, t1, t1_by_token, a, spart, st);
  return launch_gemm1_rk<R, 8>(dm, g, T, perm, expert_idx, gate, u1t, v2p, t1, t1_by_token, a, spart, st);
}

}  // namespace

// With a packed copy of the bases (per cluster W1 as [d/32][d_ff][32], then all of W2 as
// [d_ff/32][d][32]) the weight operand is read from it: row stride 32, block stride rows * 32.
static void use_packed_base(GemmArgs& g, const cmoe_dims& dm, const cmoe_weights& w, bool second) {
  if (w.packed == nullptr) return;
  const cmoe_packed_layout PL = cmoe_packed(dm);
  g.W = (const half_t*)((const char*)w.packed + (second ? PL.w2 : PL.w1));
  g.ldw = 32;
  g.kstep_w = (long)(second ? dm.d : dm.d_ff) * 32;
}

hipError_t launch_gemm1(const cmoe_dims& dm, const cmoe_weights& w, const half_t* x, int x_div, int T,
                        const int* perm,
                        const int* offsets, const int* expert_idx, const float* gate, const half_t* u1t,
                        const half_t* v2p, const half_t* t1, bool t1_by_token, half_t* a, float* spart, hipStream_t st) {
  GemmArgs g{(const half_t*)w.w1_base, (long)dm.d_ff * dm.d, dm.d, dm.d_ff, x, dm.d, perm, dm.d, offsets, dm.G,
             (dm.d_ff + TileBig::BN - 1) / TileBig::BN};
  g.x_div = x_div;
  use_packed_base(g, dm, w, false);
  switch (dm.r) {
    case 4: return launch_gemm1_r<4>(dm, g, T, perm, expert_idx, gate, u1t, v2p, t1, t1_by_token, a, spart, st);
    case 8: return launch_gemm1_r<8>(dm, g, T, perm, expert_idx, gate, u1t, v2p, t1, t1_by_token, a, spart, st);
    case 16: return launch_gemm1_r<16>(dm, g, T, perm, expert_idx, gate, u1t, v2p, t1, t1_by_token, a, spart, st);
    default: return launch_gemm1_r<32>(dm, g, T, perm, expert_idx, gate, u1t, v2p, t1, t1_by_token, a, spart, st);
  }
}

hipError_t launch_sreduce(const cmoe_dims& dm, int T, const int* perm, const float* spart, int n_parts,
                          float* s_down, hipStream_t st) {
  int kr = dm.k * dm.r;
  size_t n = (size_t)T * kr;
  const dim3 grid((unsigned)((n + 255) / 256));
  if (n_parts > 128)
    hipLaunchKernelGGL((sreduce_kernel<16, float>), grid, dim3(1024), 0, st, spart, perm, T, kr, n_parts, s_down);
  else
    hipLaunchKernelGGL((sreduce_kernel<4, float>), grid, dim3(256), 0, st, spart, perm, T, kr, n_parts, s_down);
  return hipGetLastError();
}

hipError_t launch_sext(const cmoe_dims& dm, int T, const int* perm, const int* expert_idx, const float* gate, const float* spart,
                       int n_parts, half_t* sext, int* zero, hipStream_t st) {
  const int rows = 256 / (dm.k * dm.r);
  auto go = [&](auto kern, int nw) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((T + rows - 1) / rows)), dim3(64 * nw), 0, st, spart, perm, expert_idx, gate, T,
                       dm.K, dm.k, dm.r, dm.KRp, n_parts, sext, zero);
  };
  if (n_parts > 128) go(sext_kernel<16>, 16); else go(sext_kernel<4>, 4);
  return hipGetLastError();
}

hipError_t launch_gemm2(const cmoe_dims& dm, const cmoe_weights& w, const half_t* a, int T, const int* offsets,
                        const int* rowmap, half_t* y_base_sorted, hipStream_t st) {
  // a is [d_ff / 32][T][32]
  GemmArgs g{(const half_t*)w.w2_base, (long)dm.d * dm.d_ff, dm.d_ff, dm.d, a, 32, nullptr, dm.d_ff, offsets,
             dm.G, (dm.d + TileBig::BN - 1) / TileBig::BN};
  g.kstep_x = (long)T * 32;
  use_packed_base(g, dm, w, true);
  EpiStore epi{y_base_sorted, rowmap, dm.d, dm.d};
  return launch_gemm(g, T, epi, st);
}

hipError_t launch_combine(const cmoe_dims& dm, const half_t* u2t, const half_t* y_base_sorted, const float* s_down,
                          const int* perm, const int* offsets, const int* expert_idx, const float* gate, int T,
                          half_t* y, hipStream_t st) {
  int n_blocks32 = dm.d / 32;
  int per_wg = CB_WAVES * CB_NPW;
  int n_groups = (n_blocks32 + per_wg - 1) / per_wg;
  int m_slots = (T + 31) / 32 + dm.G;
  hipLaunchKernelGGL(combine_kernel, dim3((unsigned)(n_groups * m_slots)), dim3(CB_WAVES * 64), 0, st, u2t,
                     y_base_sorted, s_down, perm, offsets, expert_idx, gate, dm.G, dm.K, dm.k, dm.r, dm.KRp, dm.d,
                     n_groups, y);
  return hipGetLastError();
}

// Down-projection with the residual of the second matrix and the return to token order
// fused into it (K*r <= 128).  rperm: token of each row of A; sext: see sext_kernel.  parts, arrivals: scratch for parts of the
// contraction (GEMM_PARTS of GEMM_PART values; counts, zero), NULL: not split.
hipError_t launch_gemm2_combine(const cmoe_dims& dm, const cmoe_weights& w, const half_t* a, int T,
                                const int* offsets, const int* rperm, const half_t* u2t, const half_t* sext,
                                const int* expert_idx, half_t* y, float* parts, int* arrivals, hipStream_t st) {
  GemmArgs g{(const half_t*)w.w2_base, (long)dm.d * dm.d_ff, dm.d_ff, dm.d, a, 32, nullptr, dm.d_ff, offsets,
             dm.G, (dm.d + TileBig::BN - 1) / TileBig::BN};
  g.kstep_x = (long)T * 32;
  // an XCD can be left with few enough tiles to split: four, or eight of groups that hold no more than a quarter's
  // tokens (a launch prepared for it has more workgroups, which cost 0.7 us where they find nothing to do)
  const int least = ((T + TileBig::BM - 1) / TileBig::BM) * g.n_tiles, most = least + dm.G * g.n_tiles;
  const int few = XCD_CUS / (T <= TileQuad::BM * dm.G ? 4 : 8);
  bool can = false;
  if (dm.d_ff / 32 >= SPLIT_BLOCKS)
    for (int mine = least / 8; mine <= (most + 7) / 8 && !can; ++mine) can = mine % XCD_CUS >= 1 && mine % XCD_CUS <= few;
  if (can) {
    g.parts = (float4v*)parts;
    g.arrivals = arrivals;
  }
  use_packed_base(g, dm, w, true);
  if (dm.d_ff / 32 >= EXT_BLOCKS) {
    g.W2 = u2t;
    g.w2_cstride = (long)dm.d * dm.KRp;
    g.ldw2 = dm.KRp;
    g.Kc2 = dm.KRp;
    g.X2 = sext;
  }
  EpiDownCombine epi{u2t, (const half_t*)w.u2_s, sext, rperm, expert_idx, y, dm.k, dm.K, dm.r, dm.KRp, dm.d, dm.q, T};
  return launch_gemm(g, T, epi, st);
}

// Grouped product with a plain store, for callers outside the forward path:
//   out[rowmap ? rowmap[p] : p][n] = sum_k X[row(p)][k_g + k] * W_g[n][k_g + k],
// W_g = W + g * w_gstride, row(p) = gather ? gather[p] / x_div : p, rows p of group g in
// [offsets[g], offsets[g+1]); k runs over [0, Kc) or over the group's krange.  offsets == NULL (with a
// FP32 output): the groups have rows / n_groups rows each and all read the same rows of X.  At most
// RowTiles::MAX_GROUPS groups.
hipError_t launch_gemm_plain(const half_t* W, long w_gstride, int ldw, int N, const half_t* X, int ldx,
                             const int* gather, int x_div, int Kc, const int* offsets, int n_groups, int rows,
                             const int* krange, const int* rowmap, void* out, int ldo, bool out_f32,
                             hipStream_t st, long kstep_w, long kstep_x) {
  if (n_groups > RowTiles::MAX_GROUPS) return hipErrorInvalidValue;
  GemmArgs g{W, w_gstride, ldw, N, X, ldx, gather, Kc, offsets, n_groups, (N + TileBig::BN - 1) / TileBig::BN};
  g.x_div = x_div;
  g.krange = krange;
  if (offsets == nullptr) g.rows_each = rows / n_groups;
  g.kstep_w = kstep_w;
  g.kstep_x = kstep_x;
  if (N <= 64 && !out_f32) {
    // a few output columns per row (products into rank space)
    EpiStore epi{(half_t*)out, rowmap, ldo, N};
    hipLaunchKernelGGL((gemm_thin_kernel<EpiStore>), dim3((unsigned)((rows + 127) / 128 + n_groups)), dim3(256), 0, st, g,
                       epi);
    return hipGetLastError();
  }
  if (out_f32) {
    EpiStoreT<float> epi{(float*)out, rowmap, ldo, N};
    return launch_gemm(g, rows, epi, st);
  }
  EpiStore epi{(half_t*)out, rowmap, ldo, N};
  return launch_gemm(g, rows, epi, st);
}

// out[n / 32][p][n % 32] = sum_k W_c[n][k] X[gather[p]][k] for the sorted rows p of cluster c.
hipError_t launch_gemm_blocked(const half_t* W, long w_gstride, int ldw, long kstep_w, int N, const half_t* X, int ldx,
                               const int* gather, int Kc, const int* offsets, int n_groups, int rows, half_t* out,
                               hipStream_t st) {
  GemmArgs g{W, w_gstride, ldw, N, X, ldx, gather, Kc, offsets, n_groups, (N + TileBig::BN - 1) / TileBig::BN};
  g.kstep_w = kstep_w;
  return launch_gemm(g, rows, EpiStoreBlocked{out, rows, N}, st);
}

// dx[rperm[p]] = B1^T dhsum[p] + sum_j V1^T q_j + sum_j dl_j v_{e_j}; w1t = B1^T in 32-column blocks, dhsum
// [d_ff / 32][T][32].
hipError_t launch_gemm_input_grad(const cmoe_dims& dm, const half_t* w1t, const half_t* dhsum, int T, const int* offsets,
                                  const half_t* v1cat, const int* offe, const half_t* q, const int* es, const int* rperm,
                                  const float* dl, const half_t* router_expert, float* dx, hipStream_t st) {
  GemmArgs g{w1t, (long)dm.d * dm.d_ff, 32, dm.d, dhsum, 32, nullptr, dm.d_ff, offsets, dm.G,
             (dm.d + TileBig::BN - 1) / TileBig::BN};
  g.kstep_w = (long)dm.d * 32;
  g.kstep_x = (long)T * 32;
  return launch_gemm(g, T, EpiInputGrad{v1cat, offe, q, es, rperm, dl, router_expert, dx, dm.k, dm.K, dm.r, dm.KRp, dm.d}, st);
}

// packed[c][(k / 32) * N + n][k % 32] = base[c][n][k].  A workgroup takes 64 rows n (four
// threads per row, 16 bytes each) and walks the 32-column blocks of a quarter of K: every
// store instruction of the workgroup writes 4 KiB of contiguous memory.
__global__ __launch_bounds__(256) void pack_base_kernel(const half_t* __restrict__ base, int N, int K,
                                                        half_t* __restrict__ packed) {
  const size_t mat = (size_t)N * K;
  const int n = blockIdx.x * 64 + (threadIdx.x >> 2), c8 = (threadIdx.x & 3) * 8;
  if (n >= N) return;
  const half_t* src = base + blockIdx.z * mat + (size_t)n * K + c8;
  half_t* dst = packed + blockIdx.z * mat + (size_t)n * 32 + c8;
  const int nb = K / 32, per = (nb + 3) / 4, b0 = blockIdx.y * per, b1 = min(nb, b0 + per);
#pragma unroll 4
  for (int kb = b0; kb < b1; ++kb) *(half8*)(dst + (size_t)kb * N * 32) = *(const half8*)(src + kb * 32);
}

hipError_t launch_pack_bases(const cmoe_dims& dm, const cmoe_weights& w, half_t* packed, hipStream_t st) {
  const cmoe_packed_layout PL = cmoe_packed(dm);
  char* pk = (char*)packed;
  hipLaunchKernelGGL(pack_base_kernel, dim3((dm.d_ff + 63) / 64, 4, dm.G), dim3(256), 0, st, (const half_t*)w.w1_base,
                     dm.d_ff, dm.d, (half_t*)(pk + PL.w1));
  hipLaunchKernelGGL(pack_base_kernel, dim3((dm.d + 63) / 64, 4, dm.G), dim3(256), 0, st, (const half_t*)w.w2_base,
                     dm.d, dm.d_ff, (half_t*)(pk + PL.w2));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the FP16 panels of all clusters' factors (Sec. 3.4: INT4 is the stored form; the panels are
  // what the matrix cores read)
  return launch_dequant_ffn(dm, w, nullptr, nullptr, (half_t*)(pk + PL.v1cat), (half_t*)(pk + PL.u1t), (half_t*)(pk + PL.v2p),
                            (half_t*)(pk + PL.u2t), st);
}
