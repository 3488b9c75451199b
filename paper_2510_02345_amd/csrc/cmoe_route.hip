// Two-stage hierarchical router (Sec. 3.3, Eq. 9 and Eq. 10) and the stable
// token-to-cluster permutation (the single-device part of group-level dispatch).
#include <mutex>
#include <type_traits>

#include "cmoe_rows.h"

namespace {

__device__ __forceinline__ float dot8(half8 a, half8 b, float acc) {
#pragma unroll
  for (int i = 0; i < 8; ++i) acc = fmaf((float)a[i], (float)b[i], acc);
  return acc;
}

// One round of (largest key, lowest lane) over the first n lanes, skipping lanes already
// taken.  Returns the winning lane; marks it taken.
__device__ __forceinline__ int select_round(float key, bool& taken, int lane, int n) {
  float m = (lane < n && !taken) ? key : -INFINITY;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  const unsigned long long who = __ballot(lane < n && !taken && key == m);
  const int j = who ? __ffsll((long long)who) - 1 : 0;   // who is non-empty while fewer than n lanes are taken
  if (lane == j) taken = true;
  return j;
}

constexpr int ROUTE_WAVES = 4;

// One wavefront per token.  The token's row stays in registers for both stages: z_g over
// all G prototypes, then l_j over the K routing vectors of the winning cluster only, so
// the work per token is (G + K) dot products of length d (Sec. 3.3).
template <int MAXC>
__global__ __launch_bounds__(ROUTE_WAVES * 64) void route_kernel(
    const half_t* __restrict__ x, const half_t* __restrict__ rc, const half_t* __restrict__ re,
    const float* __restrict__ bias, int T, int d, int G, int K, int k, int* __restrict__ cluster_id,
    int* __restrict__ expert_idx, float* __restrict__ gate) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * ROUTE_WAVES + (threadIdx.x >> 6);
  if (t >= T) return;
  const int nchunk = d >> 3;
  half8 xv[MAXC];
#pragma unroll
  for (int i = 0; i < MAXC; ++i) {
    int ch = lane + 64 * i;
    xv[i] = (ch < nchunk) ? *(const half8*)(x + (size_t)t * d + ch * 8) : half8{0, 0, 0, 0, 0, 0, 0, 0};
  }
  // stage 1: the softmax of Eq. 9 is monotone, so the most probable cluster is the
  // largest logit; strict '>' keeps the lowest index on ties
  float best = -INFINITY;
  int c = 0;
  for (int g = 0; g < G; ++g) {
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      int ch = lane + 64 * i;
      if (ch < nchunk) acc = dot8(xv[i], *(const half8*)(rc + (size_t)g * d + ch * 8), acc);
    }
    acc = wave_sum(acc);
    if (bias != nullptr) acc += bias[g];
    if (acc > best) {
      best = acc;
      c = g;
    }
  }
  // stage 2: logits of the K experts of cluster c; lane j keeps l_j
  float mine = -INFINITY;
  for (int j = 0; j < K; ++j) {
    float acc = 0.f;
    const half_t* v = re + (size_t)(c * K + j) * d;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      int ch = lane + 64 * i;
      if (ch < nchunk) acc = dot8(xv[i], *(const half8*)(v + ch * 8), acc);
    }
    acc = wave_sum(acc);
    if (lane == j) mine = acc;
  }
  // top-k by k rounds of (largest value, lowest lane) selection over the wavefront
  float sel_l[8];
  int sel_j[8];
  float lmax = 0.f;
  const float key = rank_key(mine);
  bool taken = false;
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    sel_l[a] = 0.f;
    sel_j[a] = 0;
    if (a < k) {
      const int j = select_round(key, taken, lane, K);
      sel_l[a] = __shfl(mine, j, 64);
      sel_j[a] = j;
      if (a == 0) lmax = sel_l[a];
    }
  }
  if (lane == 0) {
    cluster_id[t] = c;
    float den = 0.f;
    float ex[8];
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      ex[a] = (a < k) ? expf(sel_l[a] - lmax) : 0.f;
      den += ex[a];
    }
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      if (a < k) {
        expert_idx[(size_t)t * k + a] = c * K + sel_j[a];
        gate[(size_t)t * k + a] = ex[a] / den;
      }
    }
  }
}

// ---------------------------------------------------------------- routing variants
// Top-g clusters per token (Sec. 3.3, "Top-g_1 groups"), router temperature (Sec. 3.5) and
// optional scaling by the cluster probability of Eq. 9.  One wavefront per token; lane g
// keeps z_g, lane j keeps l_j.  Outputs are laid out per (token, selected cluster) pair
// a = 0..top_g-1, i.e. as top_g "virtual tokens" per token:
//   cluster_id [T][top_g], expert_idx [T][top_g][k], gate [T][top_g][k]
// gate = w_a * softmax(l_sel / tau), w_a = p_g (scaled) or p_g / sum of the selected p_g.
template <int MAXC>
__global__ __launch_bounds__(ROUTE_WAVES * 64) void route_multi_kernel(
    const half_t* __restrict__ x, const half_t* __restrict__ rc, const half_t* __restrict__ re,
    const float* __restrict__ bias, int T, int d, int G, int K, int k, int top_g, float inv_tau, int scale,
    int* __restrict__ cluster_id, int* __restrict__ expert_idx, float* __restrict__ gate) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * ROUTE_WAVES + (threadIdx.x >> 6);
  if (t >= T) return;
  const int nchunk = d >> 3;
  half8 xv[MAXC];
#pragma unroll
  for (int i = 0; i < MAXC; ++i) {
    int ch = lane + 64 * i;
    xv[i] = (ch < nchunk) ? *(const half8*)(x + (size_t)t * d + ch * 8) : half8{0, 0, 0, 0, 0, 0, 0, 0};
  }
  auto dot = [&](const half_t* v) {
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      int ch = lane + 64 * i;
      if (ch < nchunk) acc = dot8(xv[i], *(const half8*)(v + ch * 8), acc);
    }
    return wave_sum(acc);
  };
  auto wave_max = [&](float m) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    return m;
  };
  // Eq. 9 with temperature: p_g = softmax(z / tau)
  float zmine = -INFINITY;
  for (int g = 0; g < G; ++g) {
    float z = dot(rc + (size_t)g * d);
    if (bias != nullptr) z += bias[g];
    if (lane == g) zmine = z;
  }
  const float zmax = wave_max(zmine);
  const float ez = (lane < G) ? expf((zmine - zmax) * inv_tau) : 0.f;
  const float pz = ez / wave_sum(ez);
  // the top_g clusters: rounds of (largest logit, lowest lane)
  int sel_c[8];
  float sel_p[8];
  float psum = 0.f;
  const float zkey = rank_key(zmine);
  bool ztaken = false;
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    sel_c[a] = 0;
    sel_p[a] = 0.f;
    if (a < top_g) {
      const int g = select_round(zkey, ztaken, lane, G);
      sel_c[a] = g;
      sel_p[a] = __shfl(pz, g, 64);
      psum += sel_p[a];
    }
  }
#pragma unroll
  for (int a = 0; a < 8; ++a) {
    if (a >= top_g) continue;
    const int c = sel_c[a];
    const float wa = scale ? sel_p[a] : sel_p[a] / psum;
    float mine = -INFINITY;
    for (int j = 0; j < K; ++j) {
      const float l = dot(re + (size_t)(c * K + j) * d);
      if (lane == j) mine = l;
    }
    float sel_l[8];
    int sel_j[8];
    const float key = rank_key(mine);
    bool taken = false;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      sel_l[b] = 0.f;
      sel_j[b] = 0;
      if (b < k) {
        const int j = select_round(key, taken, lane, K);
        sel_l[b] = __shfl(mine, j, 64);
        sel_j[b] = j;
      }
    }
    if (lane == 0) {
      const size_t vt = (size_t)t * top_g + a;
      cluster_id[vt] = c;
      float den = 0.f, ex[8];
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        ex[b] = (b < k) ? expf((sel_l[b] - sel_l[0]) * inv_tau) : 0.f;
        den += ex[b];
      }
#pragma unroll
      for (int b = 0; b < 8; ++b)
        if (b < k) {
          expert_idx[vt * k + b] = c * K + sel_j[b];
          gate[vt * k + b] = wa * (ex[b] / den);
        }
    }
  }
}

// y[t][:] = sum_a yrep[t top_g + a][:] (FP32, a ascending)
__global__ __launch_bounds__(256) void sum_groups_kernel(const half_t* __restrict__ yrep, int top_g, int d,
                                                         half_t* __restrict__ y) {
  const int t = blockIdx.y, col = (blockIdx.x * 256 + threadIdx.x) * 8;
  if (col >= d) return;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = 0.f;
  for (int a = 0; a < top_g; ++a) {
    const half8 v = *(const half8*)(yrep + ((size_t)t * top_g + a) * d + col);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] += (float)v[i];
  }
  half8 o;
#pragma unroll
  for (int i = 0; i < 8; ++i) o[i] = (half_t)acc[i];
  *(half8*)(y + (size_t)t * d + col) = o;
}

// Few tokens: one workgroup (eight wavefronts) per token, the logits of a stage spread over
// the wavefronts so that their dot products run side by side instead of one after another.  ALL: few router
// rows altogether, and the logits of every expert are taken with the clusters', so that the second stage
// waits for no load (one token, 2 + 8 rows of 768: 4.3 -> 3.7 us).
constexpr int RS_WAVES = 8;
constexpr int RS_ALL = 16;   // router rows up to which every logit is taken at once
template <int MAXC, bool ALL>
__global__ __launch_bounds__(RS_WAVES * 64) void route_small_kernel(
    const half_t* __restrict__ x, const half_t* __restrict__ rc, const half_t* __restrict__ re,
    const float* __restrict__ bias, int T, int d, int G, int K, int k, int* __restrict__ cluster_id,
    int* __restrict__ expert_idx, float* __restrict__ gate) {
  __shared__ float zs[64];
  __shared__ float ls[ALL ? RS_ALL : 64];
  __shared__ int cs;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = blockIdx.x;
  const int nchunk = d >> 3;
  half8 xv[MAXC];
#pragma unroll
  for (int i = 0; i < MAXC; ++i) {
    int ch = lane + 64 * i;
    xv[i] = (ch < nchunk) ? *(const half8*)(x + (size_t)t * d + ch * 8) : half8{0, 0, 0, 0, 0, 0, 0, 0};
  }
  auto dot = [&](const half_t* v) {
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; ++i) {
      int ch = lane + 64 * i;
      if (ch < nchunk) acc = dot8(xv[i], *(const half8*)(v + ch * 8), acc);
    }
    return wave_sum(acc);
  };
  if (ALL) {
    // at most two rows a wavefront, both in flight
    const int n = G + G * K;
    auto row = [&](int i) { return i < G ? rc + (size_t)i * d : re + (size_t)(i - G) * d; };
    const int i0 = wave, i1 = wave + RS_WAVES;
    const float l0 = dot(row(min(i0, n - 1))), l1 = dot(row(min(i1, n - 1)));
    if (lane == 0) {
      if (i0 < G) zs[i0] = bias != nullptr ? l0 + bias[i0] : l0; else if (i0 < n) ls[i0 - G] = l0;
      if (i1 < G) zs[i1] = bias != nullptr ? l1 + bias[i1] : l1; else if (i1 < n) ls[i1 - G] = l1;
    }
  } else {
    for (int g = wave; g < G; g += RS_WAVES) {
      float z = dot(rc + (size_t)g * d);
      if (bias != nullptr) z += bias[g];
      if (lane == 0) zs[g] = z;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float best = -INFINITY;
    int c = 0;
    for (int g = 0; g < G; ++g)
      if (zs[g] > best) {
        best = zs[g];
        c = g;
      }
    cs = c;
  }
  __syncthreads();
  const int c = cs;
  if (!ALL) {
    for (int j = wave; j < K; j += RS_WAVES) {
      float l = dot(re + (size_t)(c * K + j) * d);
      if (lane == 0) ls[j] = l;
    }
    __syncthreads();
  }
  if (wave == 0) {
    const float mine = (lane < K) ? ls[(ALL ? c * K : 0) + lane] : -INFINITY;
    float sel_l[8];
    int sel_j[8];
    float lmax = 0.f;
    const float key = rank_key(mine);
    bool taken = false;
#pragma unroll
    for (int a = 0; a < 8; ++a) {
      sel_l[a] = 0.f;
      sel_j[a] = 0;
      if (a < k) {
        const int j = select_round(key, taken, lane, K);
        sel_l[a] = __shfl(mine, j, 64);
        sel_j[a] = j;
        if (a == 0) lmax = sel_l[a];
      }
    }
    if (lane == 0) {
      cluster_id[t] = c;
      float den = 0.f;
      float ex[8];
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        ex[a] = (a < k) ? expf(sel_l[a] - lmax) : 0.f;
        den += ex[a];
      }
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        if (a < k) {
          expert_idx[(size_t)t * k + a] = c * K + sel_j[a];
          gate[(size_t)t * k + a] = ex[a] / den;
        }
      }
    }
  }
}

__global__ void zero_offsets_kernel(int G, int* offsets) {
  if ((int)threadIdx.x <= G) offsets[threadIdx.x] = 0;
}

}  // namespace

namespace {
// ---------------------------------------------------------------- permutation
// Stable counting sort by blocks of SORT_BLOCK items, one thread per item.
//   item i -> bin.  Plain: bin = id, id(i) = ids[i * stride] / div clamped to the bins.  PAIR: id is
//   the token's cluster c and bin = c NK + (pair key of the token inside its cluster): the
//   refined order of the fused up-projection, ranked together with the plain order by cluster.
// sort_rank_kernel ranks a block; what it needs of the other blocks are the counts per bin over
// all blocks and over the earlier ones.  It makes them itself
//   - from the ids, up to SORT_SELF items (one launch),
//   - from the per-block histograms of sort_hist_kernel, up to SORT_SUM_BLOCKS blocks and
//     SORT_SUM_COUNTS counts (two),
//   - else from those histograms after sort_scan_kernel has summed them over the blocks (three).
// Everything here is latency, not bandwidth: a launch costs about as much as a block's ranks.
// Histogram, scan, ranks and a one-workgroup-per-cluster pair sort were four launches: 21 -> 8 us
// of kernel time at 4096 tokens and 2 clusters (now one launch), 31 -> 11 us at 16384 tokens
// with Zipf loads and 27 -> 14 us at 32768 tokens and 8 clusters (two launches).
// The third launch pays once every block's sums over the counts of all blocks take longer than it:
// whole forward with 4096 bins (64 clusters of 64 keys) 138 us either way at 16 blocks, 237 us with
// two launches and 231 with three at 32 blocks, 778 and 756 at 128; with 2048 bins 162 and 161 at
// 32, 504 and 498 at 128; with 1024 bins no difference from 32 to 128; with 512 bins 98.8 and 101.3
// at 64, 153 and 157 at 128.
constexpr int SORT_BLOCK = PERMUTE_BLOCK, SORT_WAVES = SORT_BLOCK / 64;
constexpr int SORT_SELF = 4 * SORT_BLOCK;
constexpr int SORT_SUM_BLOCKS = 128;
constexpr int SORT_SUM_COUNTS = 1 << 16;
constexpr int SORT_BINS = 4096;   // bins of a sort: 64 clusters x 64 pair keys, 64 x 32 experts

// Exclusive sum over the workgroup's 1024 threads, in thread order; contains one barrier, and
// the caller separates two uses of ws by another.
__device__ __forceinline__ int block_exclusive(int v, int* ws) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(incl, off, 64);
    if (lane >= off) incl += u;
  }
  if (lane == 63) ws[wave] = incl;
  __syncthreads();
  int before = 0;
#pragma unroll
  for (int w = 0; w < SORT_WAVES; ++w) before += w < wave ? ws[w] : 0;
  return before + incl - v;
}

// Sort key of a token inside its cluster c: its (first, second) selected expert, or the first
// alone when K * K keys do not fit 64.  Expert slots outside the cluster (inconsistent caller
// input) are clamped into it.
__device__ __forceinline__ int pair_key(const int* expert_idx, int tok, int c, int K, int k, int two_keys) {
  const int* e = expert_idx + (size_t)tok * k;
  const int j0 = min(max(e[0] - c * K, 0), K - 1);
  return two_keys ? j0 * K + min(max(e[1] - c * K, 0), K - 1) : j0;
}

struct SortArgs {
  const int* ids;
  int stride, div, n, n_ids;     // items and ids' bins
  const int* expert_idx;         // PAIR
  int K, k, two_keys, nk;        // PAIR: nk keys per cluster
  int n_blocks, bins;            // bins = n_ids (plain) or n_ids * nk
};
// (id, bin) of item i < n
template <bool PAIR>
__device__ __forceinline__ void sort_bin(const SortArgs& a, int i, int& id, int& bin) {
  const int raw = a.ids[(size_t)i * a.stride];
  id = min(max(a.div == 1 ? raw : raw / a.div, 0), a.n_ids - 1);
  bin = PAIR ? id * a.nk + pair_key(a.expert_idx, i, id, a.K, a.k, a.two_keys) : id;
}

// counts[block][bin]
template <bool PAIR>
__global__ __launch_bounds__(SORT_BLOCK) void sort_hist_kernel(SortArgs a, int* __restrict__ counts) {
  __shared__ int hist[SORT_BINS];
  const int i = blockIdx.x * SORT_BLOCK + threadIdx.x;
  int id = 0, bin = 0;
  if (i < a.n) sort_bin<PAIR>(a, i, id, bin);
  for (int b = threadIdx.x; b < a.bins; b += SORT_BLOCK) hist[b] = 0;
  __syncthreads();
  if (i < a.n) atomicAdd(&hist[bin], 1);   // integer counts: order-independent
  __syncthreads();
  for (int b = threadIdx.x; b < a.bins; b += SORT_BLOCK) counts[(size_t)blockIdx.x * a.bins + b] = hist[b];
}

// counts[block][bin] -> the bin's count in earlier blocks, totals in counts[n_blocks][bin].
__global__ __launch_bounds__(64) void sort_scan_kernel(SortArgs a, int* __restrict__ counts) {
  const int b = blockIdx.x * 64 + threadIdx.x;
  if (b >= a.bins) return;
  int run = 0;
  for (int blk0 = 0; blk0 < a.n_blocks; blk0 += 16) {
    int v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = blk0 + u < a.n_blocks ? counts[(size_t)(blk0 + u) * a.bins + b] : 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if (blk0 + u < a.n_blocks) counts[(size_t)(blk0 + u) * a.bins + b] = run;
      run += v[u];
    }
  }
  counts[(size_t)a.n_blocks * a.bins + b] = run;
}

enum { SORT_FROM_IDS = 0, SORT_FROM_HIST = 1, SORT_FROM_SCAN = 2 };
// perm[row] = item, inv_perm[item] = row in the order by id; offsets[id] = first row of an id.
// PAIR: rowmap[refined row] = row, perm2[refined row] = item in the order by bin.
// dyn: LDS by sort_lds.
template <bool PAIR>
__device__ __forceinline__ void sort_rank_block(const SortArgs& a, int mode, const int* __restrict__ counts,
                                                int* __restrict__ perm, int* __restrict__ inv_perm,
                                                int* __restrict__ offsets, int* __restrict__ rowmap,
                                                int* __restrict__ perm2, int* dyn) {
  __shared__ int ws[SORT_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, me = blockIdx.x, bins = a.bins;
  int* tot = dyn;                 // [bins] count over all blocks, then first row of the bin
  int* bef = tot + bins;          // [bins] count in earlier blocks
  int* idb = bef + bins;          // [n_ids] PAIR: count of an id in earlier blocks
  unsigned char* wc = (unsigned char*)(idb + (PAIR ? a.n_ids : 0));          // [SORT_WAVES][bins] items of a wavefront
  unsigned char* wid = wc + SORT_WAVES * ((bins + 3) & ~3);                  // [SORT_WAVES][n_ids], PAIR
  const int ldw = (bins + 3) & ~3, ldi = (a.n_ids + 3) & ~3;
  const int i = me * SORT_BLOCK + tid;
  const bool in = i < a.n;
  int id = 0, bin = 0;
  if (in) sort_bin<PAIR>(a, i, id, bin);
  const int words = 2 * bins + (PAIR ? a.n_ids : 0) + SORT_WAVES * (ldw + (PAIR ? ldi : 0)) / 4;
  for (int w = tid; w < words; w += SORT_BLOCK) dyn[w] = 0;
  __syncthreads();
  // ranks inside the wavefront: lanes with the same bin (and the same id)
  auto match = [&](int val, int bits) {
    unsigned long long same = __ballot(in);
    for (int b = 0; b < bits; ++b) {
      const unsigned long long m = __ballot((val >> b) & 1);
      same &= ((val >> b) & 1) ? m : ~m;
    }
    return same;
  };
  const unsigned long long lower = (1ull << lane) - 1ull;
  const unsigned long long sb = match(bin, 32 - __builtin_clz(bins));
  const int rank_b = __popcll(sb & lower);
  if (in && rank_b == 0) wc[wave * ldw + bin] = (unsigned char)__popcll(sb);
  int rank_i = rank_b;
  if (PAIR) {
    const unsigned long long si = match(id, 32 - __builtin_clz(a.n_ids));
    rank_i = __popcll(si & lower);
    if (in && rank_i == 0) wid[wave * ldi + id] = (unsigned char)__popcll(si);
  }
  // counts over all blocks and over the earlier ones
  if (mode == SORT_FROM_IDS) {
    for (int b0 = 0; b0 < a.n_blocks; ++b0) {
      const int i2 = b0 * SORT_BLOCK + tid;
      int id2 = id, bin2 = bin;
      if (b0 != me && i2 < a.n) sort_bin<PAIR>(a, i2, id2, bin2);
      if (i2 < a.n) {
        atomicAdd(&tot[bin2], 1);
        if (b0 < me) {
          atomicAdd(&bef[bin2], 1);
          if (PAIR) atomicAdd(&idb[id2], 1);
        }
      }
    }
  } else if (mode == SORT_FROM_HIST) {
    // threads beyond the bins share the blocks
    int width = 1;
    while (width < bins && width < SORT_BLOCK) width <<= 1;
    const int parts = SORT_BLOCK / width, part = tid / width;
    const int per = (a.n_blocks + parts - 1) / parts, b0 = part * per, b1 = min(a.n_blocks, b0 + per);
    for (int b = tid % width; b < bins; b += width) {
      int t = 0, f = 0;
#pragma unroll 8
      for (int blk = b0; blk < b1; ++blk) {
        const int v = counts[(size_t)blk * bins + b];
        t += v;
        f += blk < me ? v : 0;
      }
      if (t) atomicAdd(&tot[b], t);
      if (f) {
        atomicAdd(&bef[b], f);
        if (PAIR) atomicAdd(&idb[b / a.nk], f);
      }
    }
  } else {
    for (int b = tid; b < bins; b += SORT_BLOCK) {
      const int f = counts[(size_t)me * bins + b];
      tot[b] = counts[(size_t)a.n_blocks * bins + b];
      bef[b] = f;
      if (PAIR && f) atomicAdd(&idb[b / a.nk], f);
    }
  }
  __syncthreads();
  {   // first row of every bin: exclusive sum over the bins, four consecutive bins per thread
    int n4[4], sum = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      n4[u] = 4 * tid + u < bins ? tot[4 * tid + u] : 0;
      sum += n4[u];
    }
    int at = block_exclusive(sum, ws);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (4 * tid + u < bins) tot[4 * tid + u] = at;
      at += n4[u];
    }
  }
  __syncthreads();
  const int nk = PAIR ? a.nk : 1;
  if (me == 0)
    for (int g = tid; g <= a.n_ids; g += SORT_BLOCK) offsets[g] = g < a.n_ids ? tot[g * nk] : a.n;
  if (!in) return;
  int row = tot[id * nk] + rank_i + (PAIR ? idb[id] : bef[id]);
  const unsigned char* col = PAIR ? wid + id : wc + id;
  const int ldc = PAIR ? ldi : ldw;
#pragma unroll
  for (int w = 0; w < SORT_WAVES; ++w) row += w < wave ? col[w * ldc] : 0;
  perm[row] = i;
  inv_perm[i] = row;
  if (PAIR) {
    int fine = tot[bin] + bef[bin] + rank_b;
#pragma unroll
    for (int w = 0; w < SORT_WAVES; ++w) fine += w < wave ? wc[w * ldw + bin] : 0;
    rowmap[fine] = row;
    perm2[fine] = i;
  }
}

template <bool PAIR>
__global__ __launch_bounds__(SORT_BLOCK) void sort_rank_kernel(SortArgs a, int mode, const int* __restrict__ counts,
                                                              int* __restrict__ perm, int* __restrict__ inv_perm,
                                                              int* __restrict__ offsets, int* __restrict__ rowmap,
                                                              int* __restrict__ perm2) {
  extern __shared__ int dyn[];
  sort_rank_block<PAIR>(a, mode, counts, perm, inv_perm, offsets, rowmap, perm2, dyn);
}

// The same and, in further workgroups, t1 = V1 x in token order, which needs the router's decision but not the
// permutation: a workgroup takes 32 rows of x and the 16-row blocks of ONE cluster's rank rows that one of their
// (virtual) tokens selected, its first four wavefronts a quarter of the contraction each.  It takes as long as the longer
// of the two launches that it replaces, 10.4 us where they took 7.3 and 9.9 (777 tokens of 4 clusters of width 1024).
struct T1Tokens {
  const half_t *x, *v1cat;
  const int *cluster_id, *expert_idx;   // per virtual token
  half_t* t1;                           // [T][k][r], virtual tokens
  int rows, x_div;                      // rows of x; virtual tokens of each
  int d, G, K, k, r, KRp;
};
constexpr int ST_NA = 4, ST_PAIRS = 16;   // blocks of 16 rank rows at a time; (virtual token, expert) pairs of a row, at most
__device__ __forceinline__ void t1_tokens_block(const T1Tokens& a, int blk, char* smem) {
  __shared__ int es[RW_M][ST_PAIRS];      // first rank row of the pair's expert in its cluster; -1: another cluster's
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (wave >= RW_WAVES) return;   // the barriers below wait for the wavefronts that have not ended (s_barrier)
  const int c = blk % a.G, row0 = blk / a.G * RW_M, t16 = lane & 15, q = lane >> 4;
  const int row = row0 + (lane & (RW_M - 1));
  unsigned need = 0u;
  for (int p = 0; p < a.x_div * a.k; ++p) {
    const int vt = row * a.x_div + p / a.k;
    int e0 = -1;
    if (row < a.rows && a.cluster_id[vt] == c) {
      e0 = min(max(a.expert_idx[(size_t)vt * a.k + p % a.k] - c * a.K, 0), a.K - 1) * a.r;
      need |= block_mask(e0, a.r);
    }
    if (tid < RW_M) es[tid][p] = e0;
  }
  need = wave_or(need);
  const half_t* vc = a.v1cat + (size_t)c * a.KRp * a.d;
  const int steps = a.d / 64, it0 = wave * steps / RW_WAVES, it1 = (wave + 1) * steps / RW_WAVES;
  while (need != 0u) {
    int blocks[ST_NA];
    const int n = take_blocks(need, blocks);
    unsigned order = 0u;   // the blocks' numbers, eight bits each
#pragma unroll
    for (int i = 0; i < ST_NA; ++i) order |= (unsigned)blocks[i] << (8 * i);
    auto pass = [&](auto na) {
      constexpr int NA = decltype(na)::value;
      float4v acc[NA][RW_MT];
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int b = 0; b < RW_MT; ++b) acc[i][b] = float4v{0.f, 0.f, 0.f, 0.f};
      rows_product_ring<NA>(smem + wave * RowsRing<NA>::NS * RowsRing<NA>::STAGE, lane,
                            [&](int i) {
                              return i < NA * 16 ? vc + ((size_t)((order >> (8 * (i >> 4))) & 255) * 16 + (i & 15)) * a.d
                                                 : a.x + (size_t)min(row0 + i - NA * 16, a.rows - 1) * a.d;
                            },
                            it0, it1, acc);
      __syncthreads();   // es is complete, the rings have been read
      rows_reduce<NA>((float4v*)smem, wave, lane, acc, [&](int i, int b, const float4v& s) {
        const int m = b * 16 + t16, rr = (int)((order >> (8 * i)) & 255) * 16 + 4 * q;
        if (i >= n || row0 + m >= a.rows) return;
        for (int p = 0; p < a.x_div * a.k; ++p) {
          const int e0 = es[m][p];
          if (e0 >= 0 && rr >= e0 && rr < e0 + a.r)
            *(half4*)(a.t1 + ((size_t)(row0 + m) * a.x_div * a.k + p) * a.r + (rr - e0)) =
                half4{(half_t)s[0], (half_t)s[1], (half_t)s[2], (half_t)s[3]};
        }
      });
      __syncthreads();   // the sums have been read
    };
    if (n <= 2) pass(std::integral_constant<int, 2>{}); else pass(std::integral_constant<int, ST_NA>{});
  }
}
// 1024 threads leave 128 registers a thread, and the product of t1 spills 18; the times at sort_takes_t1 are with them.
constexpr int ST_LDS = RowsRing<2>::SMEM > RowsRing<ST_NA>::SMEM ? RowsRing<2>::SMEM : RowsRing<ST_NA>::SMEM;
__global__ __launch_bounds__(SORT_BLOCK) void sort_rank_t1_kernel(SortArgs a, int mode, const int* __restrict__ counts,
                                                                  int* __restrict__ perm, int* __restrict__ inv_perm,
                                                                  int* __restrict__ offsets, int* __restrict__ rowmap,
                                                                  int* __restrict__ perm2, T1Tokens t) {
  __shared__ __attribute__((aligned(1024))) char smem[ST_LDS];
  if ((int)blockIdx.x < a.n_blocks)
    sort_rank_block<true>(a, mode, counts, perm, inv_perm, offsets, rowmap, perm2, (int*)smem);
  else
    t1_tokens_block(t, (int)blockIdx.x - a.n_blocks, smem);
}

// Up to 1024 items in up to 64 bins: one workgroup with a thread per item and no counters to clear.
// Lane g counts bin g of its wavefront from the same ballots that rank the items, the sum over the
// bins is a wavefront scan, and one barrier joins the wavefronts (none for up to 64 items).
// Against the general kernel, which clears and scans its counters: 3.5 -> 2.2 us for 300 items and
// 2 bins, 4.0 -> 2.7 us for 1024, 4.1 -> 3.2 us for 1024 items and 64 bins.
constexpr int SORT_FEW = SORT_BLOCK;
__global__ __launch_bounds__(SORT_FEW) void sort_few_kernel(SortArgs a, int* __restrict__ perm, int* __restrict__ inv_perm,
                                                            int* __restrict__ offsets) {
  __shared__ int wc[SORT_FEW / 64][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const bool in = tid < a.n;
  int id = 0, bin = 0;
  if (in) sort_bin<false>(a, tid, id, bin);
  unsigned long long same = __ballot(in), of_lane = same;   // lanes with this lane's bin; with bin `lane`
  for (int b = 0; b < 32 - __builtin_clz(a.bins); ++b) {
    const unsigned long long m = __ballot((id >> b) & 1);
    same &= ((id >> b) & 1) ? m : ~m;
    of_lane &= ((lane >> b) & 1) ? m : ~m;
  }
  const int cnt = lane < a.bins ? __popcll(of_lane) : 0;
  int total = cnt, before = 0;
  if (nw > 1) {
    wc[wave][lane] = cnt;
    __syncthreads();
    total = 0;
    for (int w = 0; w < nw; ++w) {
      const int v = wc[w][lane];
      total += v;
      before += w < wave ? v : 0;
    }
  }
  const int first = wave_inclusive_sum(total) - total;
  const int row = __shfl(first + before, id, 64) + __popcll(same & ((1ull << lane) - 1ull));
  if (wave == 0) {
    if (lane < a.bins) offsets[lane] = first;
    if (lane == 0) offsets[a.bins] = a.n;
  }
  if (!in) return;
  perm[row] = tid;
  inv_perm[tid] = row;
}

// The pair sort alone, for a permutation the caller already has: one workgroup per cluster, the
// rows of the cluster in chunks of SORT_BLOCK.  The token and the key of a thread's first PS_KEEP
// rows (tid + j SORT_BLOCK) are read once, all loads in flight together, and stay in registers for
// both passes; rows beyond come from memory in each pass, chunk by chunk.  Bound by that chain of
// loads: with chunk after chunk read in both passes it took 7.8 instead of 6.8 us for 2 clusters of
// 2048 rows, 14.4 instead of 12.6 us for 4 of 4096 and 17.4 instead of 14.3 us for 8 of 4096.
constexpr int PS_KEEP = 8;
__global__ __launch_bounds__(SORT_BLOCK) void pair_sort_kernel(const int* __restrict__ perm,
                                                              const int* __restrict__ offsets,
                                                              const int* __restrict__ expert_idx, int K, int k,
                                                              int two_keys, int* __restrict__ rowmap,
                                                              int* __restrict__ perm2) {
  __shared__ int next[64];   // next refined row of every key
  __shared__ int wcount[SORT_WAVES][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = blockIdx.x, lo = offsets[c], n = offsets[c + 1] - lo;
  if (n <= 0) return;
  int tok[PS_KEEP], key[PS_KEEP];
#pragma unroll
  for (int j = 0; j < PS_KEEP; ++j) tok[j] = tid + j * SORT_BLOCK < n ? perm[lo + tid + j * SORT_BLOCK] : 0;
#pragma unroll
  for (int j = 0; j < PS_KEEP; ++j)
    key[j] = tid + j * SORT_BLOCK < n ? pair_key(expert_idx, tok[j], c, K, k, two_keys) : 0;
  if (tid < 64) next[tid] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PS_KEEP; ++j)
    if (tid + j * SORT_BLOCK < n) atomicAdd(&next[key[j]], 1);
  for (int i = tid + PS_KEEP * SORT_BLOCK; i < n; i += SORT_BLOCK)
    atomicAdd(&next[pair_key(expert_idx, perm[lo + i], c, K, k, two_keys)], 1);
  __syncthreads();
  if (wave == 0) {
    const int cnt = next[lane];
    next[lane] = lo + wave_inclusive_sum(cnt) - cnt;
  }
  auto chunk = [&](int i, int tok, int key) {   // chunks in order keep the sort stable
    const bool in = i < n;
    unsigned long long same = __ballot(in);   // lanes of this wavefront holding the same key
#pragma unroll
    for (int b = 0; b < 6; ++b) {
      const unsigned long long m = __ballot((key >> b) & 1);
      same &= ((key >> b) & 1) ? m : ~m;
    }
    wcount[wave][lane] = 0;
    __syncthreads();
    const int below = __popcll(same & ((1ull << lane) - 1ull));
    if (in && below == 0) wcount[wave][key] = __popcll(same);
    __syncthreads();
    if (in) {
      int pos = next[key] + below;
      for (int w = 0; w < wave; ++w) pos += wcount[w][key];
      rowmap[pos] = lo + i;
      perm2[pos] = tok;
    }
    __syncthreads();
    if (tid < 64) {
      int add = 0;
#pragma unroll
      for (int w = 0; w < SORT_WAVES; ++w) add += wcount[w][tid];
      next[tid] += add;
    }
    __syncthreads();
  };
#pragma unroll
  for (int j = 0; j < PS_KEEP; ++j) {
    if (j * SORT_BLOCK >= n) break;   // uniform over the workgroup
    chunk(tid + j * SORT_BLOCK, tok[j], key[j]);
  }
  for (int i0 = PS_KEEP * SORT_BLOCK; i0 < n; i0 += SORT_BLOCK) {
    const int i = i0 + tid, t = i < n ? perm[lo + i] : 0;
    chunk(i, t, i < n ? pair_key(expert_idx, t, c, K, k, two_keys) : 0);
  }
}

inline int two_keys_of(const cmoe_dims& dm) { return (dm.k >= 2 && dm.K * dm.K <= 64) ? 1 : 0; }

// LDS of sort_rank_block; n_ids: 0 without PAIR
constexpr size_t sort_lds(int bins, int n_ids) {
  return 4 * (2 * (size_t)bins + n_ids) + SORT_WAVES * (size_t)(((bins + 3) & ~3) + ((n_ids + 3) & ~3));
}
static_assert(sort_lds(SORT_BINS, 64) <= ST_LDS, "a permutation whose launch takes t1 along");

template <bool PAIR>
hipError_t go_sort(SortArgs a, int* perm, int* inv_perm, int* offsets, int* rowmap, int* perm2, int* counts,
                   hipStream_t st, const T1Tokens* t1 = nullptr) {
  a.n_blocks = (a.n + SORT_BLOCK - 1) / SORT_BLOCK;
  a.bins = PAIR ? a.n_ids * a.nk : a.n_ids;
  const size_t lds = sort_lds(a.bins, PAIR ? a.n_ids : 0);
  if (t1 != nullptr && lds > ST_LDS) return hipErrorInvalidValue;
  const bool sum = a.n_blocks <= SORT_SUM_BLOCKS && a.n_blocks * a.bins <= SORT_SUM_COUNTS;
  const int mode = a.n <= SORT_SELF ? SORT_FROM_IDS : sum ? SORT_FROM_HIST : SORT_FROM_SCAN;
  const dim3 grid(a.n_blocks), block(SORT_BLOCK);
  if (mode != SORT_FROM_IDS) hipLaunchKernelGGL((sort_hist_kernel<PAIR>), grid, block, 0, st, a, counts);
  if (mode == SORT_FROM_SCAN) hipLaunchKernelGGL(sort_scan_kernel, dim3((a.bins + 63) / 64), dim3(64), 0, st, a, counts);
  if (PAIR && t1 != nullptr) {
    hipLaunchKernelGGL(sort_rank_t1_kernel, dim3(a.n_blocks + (t1->rows + RW_M - 1) / RW_M * t1->G), block, 0, st, a, mode,
                       (const int*)counts, perm, inv_perm, offsets, rowmap, perm2, *t1);
    return hipGetLastError();
  }
  if (lds > 65536) {   // 64 clusters with 64 pair keys each
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sort_rank_kernel<PAIR>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((sort_rank_kernel<PAIR>), grid, block, lds, st, a, mode, (const int*)counts, perm, inv_perm, offsets,
                     rowmap, perm2);
  return hipGetLastError();
}
}  // namespace

// Refines the cluster-sorted order: inside every cluster, rows are ordered by (first
// selected expert, second selected expert, original order).  Cluster boundaries (offsets)
// do not move.  Rows of a 16-token block then mostly share their experts, so the fused
// up-projection skips most rank chunks.
hipError_t launch_pair_sort(const cmoe_dims& dm, const int* perm, const int* offsets, const int* expert_idx, int* rowmap,
                            int* perm2, hipStream_t st) {
  hipLaunchKernelGGL(pair_sort_kernel, dim3(dm.G), dim3(SORT_BLOCK), 0, st, perm, offsets, expert_idx, dm.K, dm.k,
                     two_keys_of(dm), rowmap, perm2);
  return hipGetLastError();
}

// The permutation and the pair order of a step together; the cluster of token i is ids[i * stride] / div.
// counts: sort_counts(T, G * 64) ints.
hipError_t launch_sort_pairs(const cmoe_dims& dm, const int* ids, int stride, int div, const int* expert_idx, int T,
                             int* perm, int* inv_perm, int* offsets, int* counts, int* rowmap, int* perm2,
                             hipStream_t st) {
  const int two = two_keys_of(dm);
  SortArgs a{ids, stride, div, T, dm.G, expert_idx, dm.K, dm.k, two, two ? dm.K * dm.K : dm.K, 0, 0};
  return go_sort<true>(a, perm, inv_perm, offsets, rowmap, perm2, counts, st);
}

// Whether a step's t1 rides along with its permutation (launch_sort_pairs_t1): while the launch is at most a workgroup per
// CU (each takes its whole LDS).  Whole forward with two launches and with one: 4 clusters of 1024 x 4096, 300 tokens
// 69.7 and 66.5 us, 777 68.6 and 65.8, 1500 (190 workgroups) 81.5 and 77.5, 2500 (319) 106.4 and 108.5; 2 of 768 x 3072, 600
// tokens 60.3 and 57.8, 2000 71.6 and 67.2, 4096 (260) 91.8 and 91.4; 8 of 2048 x 8192, 777 (201) 188.1 and 183.4, 1300 (330)
// 202.7 and 210.2.  Rows of t1 of whole 16 bytes, which the up-projection gathers by token.
bool sort_takes_t1(const cmoe_dims& dm, int T, int x_div) {
  const int rows = T / x_div, workgroups = (rows + RW_M - 1) / RW_M * dm.G + (T + SORT_BLOCK - 1) / SORT_BLOCK;
  return T > SKINNY_T && dm.k <= 2 && dm.k * dm.r <= 32 && dm.k * dm.r % 8 == 0 && dm.KRp <= 128 && x_div * dm.k <= ST_PAIRS &&
         workgroups <= 256;
}
// The permutation and the pair order of a step of T (virtual) tokens, x_div of each row of x, and t1 of all of them in
// token order.
hipError_t launch_sort_pairs_t1(const cmoe_dims& dm, const int* cluster_id, const int* expert_idx, int T, const half_t* x, int x_div,
                                const half_t* v1cat, half_t* t1, int* perm, int* inv_perm, int* offsets, int* counts,
                                int* rowmap, int* perm2, hipStream_t st) {
  const int two = two_keys_of(dm);
  SortArgs a{cluster_id, 1, 1, T, dm.G, expert_idx, dm.K, dm.k, two, two ? dm.K * dm.K : dm.K, 0, 0};
  const T1Tokens t{x, v1cat, cluster_id, expert_idx, t1, T / x_div, x_div, dm.d, dm.G, dm.K, dm.k, dm.r, dm.KRp};
  return go_sort<true>(a, perm, inv_perm, offsets, rowmap, perm2, counts, st, &t);
}

// Stable sort of n > 0 items by id(i) = ids[i * stride] / div into at most SORT_BINS bins.
// counts: sort_counts(n, bins) ints.
hipError_t launch_sort_ids(const int* ids, int stride, int div, int n, int bins, int* perm, int* inv_perm, int* offsets,
                           int* counts, hipStream_t st) {
  SortArgs a{ids, stride, div, n, bins, nullptr, 1, 1, 0, 1, 1, bins};
  if (n <= SORT_FEW && bins <= 64) {
    hipLaunchKernelGGL(sort_few_kernel, dim3(1), dim3((n + 63) / 64 * 64), 0, st, a, perm, inv_perm, offsets);
    return hipGetLastError();
  }
  return go_sort<false>(a, perm, inv_perm, offsets, nullptr, nullptr, counts, st);
}

// The router for at most SKINNY_T tokens.
static hipError_t launch_route_small(const cmoe_dims& dm, const cmoe_weights& w, const half_t* x, int T, int* cluster_id,
                                     int* expert_idx, float* gate, hipStream_t st) {
  const int chunks_per_lane = (dm.d / 8 + 63) / 64;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(T), dim3(RS_WAVES * 64), 0, st, x, (const half_t*)w.router_cluster,
                       (const half_t*)w.router_expert, w.cluster_bias, T, dm.d, dm.G, dm.K, dm.k, cluster_id, expert_idx, gate);
  };
  auto pick = [&](auto all) {
    constexpr bool ALL = decltype(all)::value;
    if (chunks_per_lane <= 2) go(route_small_kernel<2, ALL>);
    else if (chunks_per_lane <= 4) go(route_small_kernel<4, ALL>);
    else if (chunks_per_lane <= 8) go(route_small_kernel<8, ALL>);
    else go(route_small_kernel<16, ALL>);
  };
  if (dm.G + dm.G * dm.K <= RS_ALL) pick(std::true_type{}); else pick(std::false_type{});
  return hipGetLastError();
}

hipError_t launch_route(const cmoe_dims& dm, const cmoe_weights& w, const half_t* x, int T, int* cluster_id,
                        int* expert_idx, float* gate, hipStream_t st) {
  dim3 grid((T + ROUTE_WAVES - 1) / ROUTE_WAVES), block(ROUTE_WAVES * 64);
  const half_t* rc = (const half_t*)w.router_cluster;
  const half_t* re = (const half_t*)w.router_expert;
  int chunks_per_lane = (dm.d / 8 + 63) / 64;
  if (T > SKINNY_T && dm.G + dm.G * dm.K <= 128)
    return launch_route_rows(dm, w, x, T, cluster_id, expert_idx, gate, st);
  if (T <= SKINNY_T) return launch_route_small(dm, w, x, T, cluster_id, expert_idx, gate, st);
  if (chunks_per_lane <= 2)
    hipLaunchKernelGGL(route_kernel<2>, grid, block, 0, st, x, rc, re, w.cluster_bias, T, dm.d, dm.G, dm.K, dm.k,
                       cluster_id, expert_idx, gate);
  else if (chunks_per_lane <= 4)
    hipLaunchKernelGGL(route_kernel<4>, grid, block, 0, st, x, rc, re, w.cluster_bias, T, dm.d, dm.G, dm.K, dm.k,
                       cluster_id, expert_idx, gate);
  else if (chunks_per_lane <= 8)
    hipLaunchKernelGGL(route_kernel<8>, grid, block, 0, st, x, rc, re, w.cluster_bias, T, dm.d, dm.G, dm.K, dm.k,
                       cluster_id, expert_idx, gate);
  else
    hipLaunchKernelGGL(route_kernel<16>, grid, block, 0, st, x, rc, re, w.cluster_bias, T, dm.d, dm.G, dm.K, dm.k,
                       cluster_id, expert_idx, gate);
  return hipGetLastError();
}

hipError_t launch_permute(const cmoe_dims& dm, const int* cluster_id, int T, int* perm, int* inv_perm, int* offsets,
                          int* counts, hipStream_t st) {
  if (T == 0) {
    hipLaunchKernelGGL(zero_offsets_kernel, dim3(1), dim3(128), 0, st, dm.G, offsets);
    return hipGetLastError();
  }
  return launch_sort_ids(cluster_id, 1, 1, T, dm.G, perm, inv_perm, offsets, counts, st);
}

// ---------------------------------------------------------------- permutation without a workspace argument
// The per-block histogram of the three-pass permutation lives in a file-scope device array
// instead of the caller's workspace, for callers that cannot allocate device memory.  Every
// GPU holds its own copy of the array at its own address; the host resolves that address
// once per device and passes it to the kernels like any other buffer.
static const int kStaticBlocks = CMOE_PERMUTE_STATIC_MAX_TOKENS / PERMUTE_BLOCK + 1;   // and a row of totals
static __device__ __align__(256) int scratch[(size_t)kStaticBlocks * 64];
static const int kMaxDevices = 64;
static int* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device (resolved on the first call per device).
static hipError_t scratch_address(int** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    int* p = nullptr;
    e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_permute_static(const cmoe_dims& dm, const int* cluster_id, int T, int* perm, int* inv_perm,
                                 int* offsets, hipStream_t st) {
  int* blk_counts = nullptr;
  // up to SORT_SELF tokens are sorted in one launch without a histogram buffer
  if (T > SORT_SELF) {
    hipError_t e = scratch_address(&blk_counts);
    if (e != hipSuccess) return e;
  }
  // every entry the later passes read is written by the first pass of the same call: nothing
  // has to start at zero, whatever an earlier call left behind
  return launch_permute(dm, cluster_id, T, perm, inv_perm, offsets, blk_counts, st);
}

hipError_t launch_route_multi(const cmoe_dims& dm, const cmoe_weights& w, const half_t* x, int T, int top_g,
                              float temperature, int scale, int* cluster_id, int* expert_idx, float* gate,
                              hipStream_t st) {
  // many tokens and few router rows: matrix-core product, decision in its epilogue (as for the
  // single-cluster router)
  if (T > SKINNY_T && dm.G + dm.G * dm.K <= 128)
    return launch_route_multi_rows(dm, w, x, T, top_g, temperature, scale, cluster_id, expert_idx, gate, st);
  dim3 grid((T + ROUTE_WAVES - 1) / ROUTE_WAVES), block(ROUTE_WAVES * 64);
  const half_t* rc = (const half_t*)w.router_cluster;
  const half_t* re = (const half_t*)w.router_expert;
  const int chunks_per_lane = (dm.d / 8 + 63) / 64;
  const float inv_tau = 1.f / temperature;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, block, 0, st, x, rc, re, w.cluster_bias, T, dm.d, dm.G, dm.K, dm.k, top_g, inv_tau,
                       scale, cluster_id, expert_idx, gate);
  };
  if (chunks_per_lane <= 2) go(route_multi_kernel<2>);
  else if (chunks_per_lane <= 4) go(route_multi_kernel<4>);
  else if (chunks_per_lane <= 8) go(route_multi_kernel<8>);
  else go(route_multi_kernel<16>);
  return hipGetLastError();
}

hipError_t launch_sum_groups(const half_t* yrep, int T, int top_g, int d, half_t* y, hipStream_t st) {
  hipLaunchKernelGGL(sum_groups_kernel, dim3((d / 8 + 255) / 256, T), dim3(256), 0, st, yrep, top_g, d, y);
  return hipGetLastError();
}
