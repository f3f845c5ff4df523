// henn_search.hip -- batched HENN query kernel (Alg. 4 Query, Sec. 2.2).
//
// One query per wavefront.  For each layer from the root down, the wave runs
// a beam search with list width ef_upper (1 = Alg. 4 GreedySearch) on the
// upper layers and max(ef, k) on layer 0, handing the best node down the
// inter-layer edge (Def. HENN: the same point one layer below).
//
// The beam keeps one ascending list W of (distance, id, expanded) keys, in
// registers or in LDS (pick_list_blocks), and repeatedly expands
// the smallest unexpanded entry; this is the
// two-heap SEARCH-LAYER of HNSW (the candidate set the paper relies on for
// k > 1) in an equivalent form: the expansion sequence and the final list
// are identical under the strict (distance, id) order.  Visited nodes are
// remembered in a direct-mapped LDS table that may forget (never invent)
// entries; a forgotten node that comes back is either already in W (caught
// by the duplicate check) or no better than W's worst (rejected again).
//
// Per expansion: one adjacency row (a lane a neighbour), the visited filter,
// gathers of the fresh neighbours' rows (LPN lanes per row, each lane a run of
// CPL 8-coordinate chunks; up to kGatherRows rows a lane group in flight), the
// canonical FP32 reduction (henn_device.h), and the new keys' way into W: one
// insertion each where W is in registers, with the next entry's adjacency row
// read ahead, or a merge by rank computation in LDS.
// Precision forms traverse BF16 / FP8 rows and re-rank the first
// min(|W|, rerank_factor*k) entries from the FP32 copy at the end.
//
// The library compiles this file ten times: HENN_PART 0 holds the host
// functions and root-scan kernels, parts 1 .. 9 the search and serving
// kernels of FP32 / BF16 / FP8 rows with the list in LDS or in two or four
// registers a lane, so that the instantiations build in parallel.  Without
// HENN_PART one translation unit holds everything.
#include <math.h>

#include <algorithm>
#include <atomic>

#include "henn_device.h"
#include "henn_internal.h"

#ifndef HENN_PART
#define HENN_PART -1
#endif
#define HENN_COMMON_PART (HENN_PART <= 0)

namespace henn {

#if HENN_COMMON_PART
size_t search_lds_per_wave(int ef_cap, int vis_bits, int vis_bytes, int blocks) {
  const size_t vis = ((size_t)1 << vis_bits) * vis_bytes, list = (size_t)ef_cap * 8;
  if (blocks == 0) return list + 64 * 8 * 2 + 64 * 4 * 2 + vis;
  // the list is in registers; its final copy takes the table's place
  return 64 * 8 + 64 * 4 * 3 + (vis > list ? vis : list);
}
#endif

// The fresh neighbours of an expansion, by compacted slot: crow (the row's
// first chunk index, row * chunks per row), cidk (id << 1, the low word of
// its key) and csc (FP8: its scale); then their keys in ckey.
//
// NB = 0: the list W is in LDS and merged in place; a merge ranks the kept
// keys in kstage (which holds the scales until then) and reuses it as the map
// of the list positions that take a kept key.
// NB > 0: the list is in registers (RegList); W is where its final copy goes,
// over the visited table, which is dead by then.
struct WaveLds {
  uint64_t* W;
  uint64_t* ckey;    // candidate keys (by compacted slot)
  uint64_t* kstage;  // NB = 0 only
  float* csc;
  uint32_t* crow;
  uint32_t* cidk;
  void* vis;  // 2^vis_bits entries: uint8 or uint16 tags, or int32 ids
  int lane;   // this lane's number, opaque to the compiler (see fresh_lane)
};

// The lane number as a value the compiler cannot see through.  Taken once per
// query: what is derived from it (offsets, masks) is then computed where it
// is used and not kept in registers across the queries of a persistent wave.
__device__ inline int fresh_lane() {
  int l = lane_id();
  asm volatile("" : "+v"(l));
  return l;
}

template <int NB>
__device__ inline WaveLds carve(char* base, int ef_cap) {
  WaveLds s;
  s.lane = lane_id();
  if constexpr (NB == 0) {
    s.W = reinterpret_cast<uint64_t*>(base);
    s.ckey = s.W + ef_cap;
    s.kstage = s.ckey + 64;
    s.csc = reinterpret_cast<float*>(s.kstage);
    s.crow = reinterpret_cast<uint32_t*>(s.kstage + 64);
    s.cidk = s.crow + 64;
    s.vis = s.cidk + 64;
  } else {
    s.ckey = reinterpret_cast<uint64_t*>(base);
    s.kstage = nullptr;
    s.csc = reinterpret_cast<float*>(s.ckey + 64);
    s.crow = reinterpret_cast<uint32_t*>(s.csc + 64);
    s.cidk = s.crow + 64;
    s.vis = s.cidk + 64;
    s.W = static_cast<uint64_t*>(s.vis);
  }
  return s;
}

// The beam's list in registers: 64 NB positions, position 64 b + l in lane l
// of w[b], ascending (distance, id) keys without the expanded flag; ex[b]
// holds one bit per position (uniform), set where there is nothing to expand.
// A list of width efl <= 64 NB occupies the last efl positions: the ones
// below hold a key under every real one, the ones not filled yet a key above
// every real one.  So the last position is the threshold a new key has to
// beat, whether the list is full or not, and an evicted entry falls off the
// end.
template <int NB>
struct RegList {
  uint64_t w[NB];
  uint64_t ex[NB];
};

__device__ inline uint64_t readlane_u64(uint64_t v, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
  return ((uint64_t)hi << 32) | lo;
}

// Value of the next lower lane (DPP wave_shr:1); lane 0 gets first.
__device__ inline uint64_t lane_above(uint64_t v, uint64_t first) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(
      (int)(uint32_t)first, (int)(uint32_t)v, 0x138, 0xF, 0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(
      (int)(uint32_t)(first >> 32), (int)(uint32_t)(v >> 32), 0x138, 0xF, 0xF, false);
  return ((uint64_t)hi << 32) | lo;
}
// The same where lane 0's value does not matter.
__device__ inline uint64_t lane_above_any(uint64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)v, 0x138, 0xF, 0xF, true);
  const uint32_t hi =
      (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), 0x138, 0xF, 0xF, true);
  return ((uint64_t)hi << 32) | lo;
}

// An empty list of width efl holding the one unexpanded entry `key`.
template <int NB>
__device__ inline void list_start(RegList<NB>& L, int lane, int efl, uint64_t key) {
  const int off = 64 * NB - efl;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int pos = 64 * b + lane;
    L.w[b] = pos < off ? 1ull : pos == off ? key : ~0ull;
    L.ex[b] = ~ballot(pos == off);
  }
}

// Inserts the uniform key k below the list's threshold; false when it is
// there already (a row the visited table forgot).  One compare gives every
// position's side of k; the positions above move up by one lane.
template <int NB>
__device__ inline bool list_insert(RegList<NB>& L, int off, uint64_t k) {
  bool lt[NB];
  uint64_t m[NB], dup = 0;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    lt[b] = L.w[b] < k;
    m[b] = ballot(lt[b]);
    dup |= ballot((uint32_t)L.w[b] == (uint32_t)k);  // ids are unique; the fillers' are odd
  }
  if (dup) return false;
#pragma unroll
  for (int b = NB - 1; b >= 0; --b) {
    if (m[b] == ~0ull) continue;
    const uint64_t e = L.ex[b];
    if (b == 0 || m[b > 0 ? b - 1 : 0] == ~0ull) {
      // k lands in this block, at its first position not below it
      const uint64_t at = ~m[b] & (m[b] + 1);
      const uint64_t up = lane_above_any(L.w[b]);
      const uint64_t v = __builtin_amdgcn_inverse_ballot_w64(at) ? k : up;
      L.w[b] = lt[b] ? L.w[b] : v;
      L.ex[b] = (e & m[b]) | ((e & ~m[b]) << 1);
    } else {
      const int pb = b > 0 ? b - 1 : 0;
      L.w[b] = lane_above(L.w[b], readlane_u64(L.w[pb], 63));
      L.ex[b] = (e << 1) | (L.ex[pb] >> 63);
    }
  }
  return true;
}

// The list's entries, flagged as in the LDS form, to / from n entries of
// memory (LDS or HBM).
template <int NB>
__device__ inline void list_store(const RegList<NB>& L, int lane, int efl, int n, uint64_t* out, bool flags) {
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int i = 64 * b + lane - (64 * NB - efl);
    const uint64_t f = (flags && __builtin_amdgcn_inverse_ballot_w64(L.ex[b])) ? 1ull : 0ull;
    if (i >= 0 && i < n) out[i] = L.w[b] | f;
  }
}
template <int NB>
__device__ inline void list_load(RegList<NB>& L, int lane, int efl, int n, const uint64_t* in) {
  const int off = 64 * NB - efl;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int i = 64 * b + lane - off;
    uint64_t v = i < 0 ? 1ull : ~0ull;
    if (i >= 0 && i < n) {
      v = in[i];
      if ((v >> 32) == 0) v |= 1ull << 32;  // above the fillers (see gather_pass)
    }
    L.ex[b] = ballot((v & 1ull) != 0);
    L.w[b] = (i >= 0 && i < n) ? wkey_strip(v) : v;
  }
}

// Largest power of two <= v (0 for v <= 0).
__device__ inline int pow2_floor(int v) { return v <= 0 ? 0 : 1 << (31 - __clz(v)); }

__device__ inline int next_pow2_dev(int v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

// Ascending bitonic sort of n (a power of two) keys in this wave's LDS.
__device__ inline void wave_bitonic_sort(uint64_t* A, int n) {
  const int lane = lane_id();
  for (int size = 2; size <= n; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = lane; i < (n >> 1); i += 64) {
        const int lo = 2 * i - (i & (stride - 1));
        const int hi = lo + stride;
        const bool asc = (lo & size) == 0;
        const uint64_t x = A[lo], y = A[hi];
        if ((x > y) == asc) {
          A[lo] = y;
          A[hi] = x;
        }
      }
      wave_sync();
    }
  }
}

// One lane computes a whole distance with the same canonical order as
// group_distance: chunk sums (eight sequential FMAs), then the pairwise tree
// over P leaves, built left to right with a stack of partial sums (leaf c
// merges with the pending left siblings named by the set low bits of c).
template <int KIND, int P>
__device__ inline float serial_distance(const float (&q)[P][8], const char* row, float scale,
                                        int nchunks, int metric) {
  float stack[8];
  float v = 0.0f;
#pragma unroll
  for (int c = 0; c < P; ++c) {
    v = 0.0f;
    if (c < nchunks) {
      float x[8];
      Chunk<KIND>::load(row, c, x);
      v = metric == 0 ? chunk_l2(q[c], x, scale, KIND == kFP8) : chunk_ip(q[c], x);
    }
#pragma unroll
    for (int l = 0; (1 << l) < P; ++l) {
      if (c & (1 << l)) {
        v = stack[l] + v;
      } else {
        stack[l] = v;
        break;
      }
    }
  }
  if (metric != 0) v = (KIND == kFP8) ? -(scale * v) : -v;
  return v;
}

// Exhaustive scan of the complete-graph root for a batch of queries: one
// thread per query (its vector in registers), root rows staged through LDS
// tiles shared by the 256 queries of a block; the root is split over
// blockIdx.y and each split writes its best (distance, position) key.
constexpr int kRootTile = 32;

template <int KIND, int P>
__global__ __launch_bounds__(256) void k_root_scan(const float* Q, int64_t nq, int d, int nchunks,
                                                   int metric, const void* rvec,
                                                   const float* rscale, int64_t rsize,
                                                   int64_t row_bytes, int64_t rows_per_split,
                                                   uint64_t* best_out) {
  extern __shared__ __align__(16) char tile[];
  float* tscale = reinterpret_cast<float*>(tile + kRootTile * row_bytes);
  const int64_t qi = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool qv = qi < nq;
  float q[P][8];
#pragma unroll
  for (int c = 0; c < P; ++c) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = c * 8 + j;
      q[c][j] = (qv && e < d) ? Q[qi * d + e] : 0.0f;
    }
  }
  const int64_t r0 = (int64_t)blockIdx.y * rows_per_split;
  const int64_t r1 = r0 + rows_per_split < rsize ? r0 + rows_per_split : rsize;
  uint64_t best = ~0ull;
  for (int64_t rt = r0; rt < r1; rt += kRootTile) {
    const int nr = (int)(r1 - rt < kRootTile ? r1 - rt : kRootTile);
    __syncthreads();
    const uint2* src = reinterpret_cast<const uint2*>(static_cast<const char*>(rvec) + rt * row_bytes);
    uint2* dst = reinterpret_cast<uint2*>(tile);
    const int64_t nwords = (nr * row_bytes) >> 3;
    for (int64_t i = threadIdx.x; i < nwords; i += 256) dst[i] = src[i];
    if (KIND == kFP8 && (int)threadIdx.x < nr) tscale[threadIdx.x] = rscale[rt + threadIdx.x];
    __syncthreads();
    for (int r = 0; r < nr; ++r) {
      const float sc = KIND == kFP8 ? tscale[r] : 1.0f;
      const float dist = serial_distance<KIND, P>(q, tile + r * row_bytes, sc, nchunks, metric);
      const uint64_t key = wkey(dist, (int32_t)(rt + r));
      best = key < best ? key : best;
    }
  }
  if (qv) best_out[(int64_t)blockIdx.y * nq + qi] = best;
}

#if HENN_COMMON_PART
template <int KIND>
static bool launch_root_scan_kind(const SearchArgs& a, int P, int splits, int64_t rows_per_split,
                                  uint64_t* out, hipStream_t st) {
  const SearchLayer& R = a.layer[a.num_layers - 1];
  const size_t lds = kRootTile * (size_t)R.row_bytes + kRootTile * sizeof(float);
  const dim3 grid((unsigned)((a.nq + 255) / 256), (unsigned)splits);
#define HENN_ROOT(PP)                                                                          \
  if (P == PP) {                                                                               \
    hipLaunchKernelGGL((k_root_scan<KIND, PP>), grid, dim3(256), lds, st, a.Q, a.nq, a.d,      \
                       a.nchunks, a.metric, R.vec, R.scale, (int64_t)R.size, R.row_bytes,      \
                       rows_per_split, out);                                                   \
    return true;                                                                               \
  }
  HENN_ROOT(1) HENN_ROOT(2) HENN_ROOT(4) HENN_ROOT(8) HENN_ROOT(16)
#undef HENN_ROOT
  return false;
}

int root_scan_splits(int64_t nq, int64_t root_size, int64_t* rows_per_split) {
  const int64_t qblocks = (nq + 255) / 256;
  int64_t splits = (2048 + qblocks - 1) / qblocks;
  const int64_t max_splits = (root_size + kRootTile - 1) / kRootTile;
  splits = splits < 1 ? 1 : splits > max_splits ? max_splits : splits;
  if (splits > 64) splits = 64;
  int64_t per = (root_size + splits - 1) / splits;
  per = (per + kRootTile - 1) / kRootTile * kRootTile;
  *rows_per_split = per;
  return (int)((root_size + per - 1) / per);
}

bool launch_root_scan(int storage, const SearchArgs& a, int splits, int64_t rows_per_split,
                      uint64_t* out, hipStream_t st) {
  const int P = next_pow2(a.nchunks);
  if (P > 16) return false;
  switch (storage) {
    case kF32: return launch_root_scan_kind<kF32>(a, P, splits, rows_per_split, out, st);
    case kBF16: return launch_root_scan_kind<kBF16>(a, P, splits, rows_per_split, out, st);
    case kFP8: return launch_root_scan_kind<kFP8>(a, P, splits, rows_per_split, out, st);
    default: return false;
  }
}

#endif  // HENN_COMMON_PART

// Exhaustive canonical scan of a complete-graph root by one wave (two rows
// per lane group in flight); every lane returns the best (distance,
// position) key.
template <int KIND, int LPN, int CPL>
__device__ uint64_t root_scan_wave(const SearchArgs& a, const SearchLayer& R,
                                   const float (&q)[CPL][8], int lane) {
  constexpr int G = 64 / LPN;
  const int t = lane % LPN, g = lane / LPN;
  uint64_t best = ~0ull;
  for (int base = 0; base < R.size; base += 2 * G) {
    const int c0 = base + g, c1 = base + G + g;
    const bool v0 = c0 < R.size, v1 = c1 < R.size;
    const float s0 = (KIND == kFP8 && v0) ? R.scale[c0] : 1.0f;
    const float s1 = (KIND == kFP8 && v1) ? R.scale[c1] : 1.0f;
    const void* const rows[2] = {
        static_cast<const char*>(R.vec) + (int64_t)(v0 ? c0 : 0) * R.row_bytes,
        static_cast<const char*>(R.vec) + (int64_t)(v1 ? c1 : 0) * R.row_bytes};
    const float sc[2] = {s0, s1};
    const bool vd[2] = {v0, v1};
    float dd[2];
    group_distances<KIND, LPN, CPL, 2>(q, rows, sc, t, a.nchunks, a.metric, vd, dd);
    const float d0 = dd[0], d1 = dd[1];
    if (v0) {
      const uint64_t k0 = wkey(d0, c0);
      best = k0 < best ? k0 : best;
    }
    if (v1) {
      const uint64_t k1 = wkey(d1, c1);
      best = k1 < best ? k1 : best;
    }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const uint64_t o = shfl_xor_u64(best, m);
    best = o < best ? o : best;
  }
  return best;
}

// Exact check after the MFMA root shortlist (one query per half wave).  With
// a(y) the Gram value of root row y (BF16 products of the centred stored
// values and the centred query, FP32 accumulation, the query-norm term
// dropped) and c(y) the canonical distance, both are within an absolute
// bound of the exact distance that scales with
// N = |q - mean|^2 + max_y |y - mean|^2 + |mean|^2 (L2; uncentred for IP):
//   |a - e| <= (2^-8 + 2^-18 + (3 dpad + 35) 2^-24) N
// (each BF16 rounding is within 2^-9 relative, so a product of two is
// within 2^-8 + 2^-18 of 2 |y_k| |q_k|, which sums to at most N; the FP32
// sums add the rest), and |c - e| <= (10 + log2 chunks) 2^-23 N.  A row
// whose Gram value exceeds a_min + M, M = (2^-7 + 2^-14 + 32 (dpad + 16)
// 2^-24) N (above twice the sum of both bounds), has c(y) > c(argmin_a), so
// the nearest root member under (distance, position) is among the rows with
// a <= a_min + M.  Each split of the Gram pass listed every row within M of
// a threshold at or above a_min: so the list holds all of them unless it
// overflowed, and then the wave scans the root.
template <int KIND, int LPN, int CPL>
__global__ __launch_bounds__(256) void k_root_check(SearchArgs a, RootShortlist sl, uint64_t* out) {
  // Two queries a wave, one a half wave (lanes 0..31 and 32..63): 10,000
  // queries fit one round of resident waves.  A half holds its query's 64
  // list entries two a lane and evaluates the kept rows G at a time.
  static_assert(kRootCap == 64, "two list entries per lane of a half wave");
  static_assert(LPN <= 32, "a lane group inside a half wave");
  constexpr int G = 32 / LPN;
  const int lane = lane_id(), t = lane % LPN, hl = lane & 31, half = lane >> 5;
  const int g = hl / LPN;
  const int64_t qi = (int64_t)blockIdx.x * 8 + (threadIdx.x >> 6) * 2 + half;
  const bool qv = qi < a.nq;
  const int64_t qs = qv ? qi : 0;  // reads of a missing second query stay in bounds
  __shared__ int32_t rows_all[4][2][64];
  int32_t* rows = rows_all[threadIdx.x >> 6][half];
  const SearchLayer& R = a.layer[a.num_layers - 1];
  float q[CPL][8];
  // an overflowed list: the whole wave loads that query and scans the root
  // for it (first, so that the scan's registers are free afterwards)
  const int cnt = qv ? sl.cnt[qs] : 0;
  const bool over = cnt > kRootCap;
  const uint64_t ovm = ballot(over);
  uint64_t best_over = ~0ull;
#pragma unroll 1
  for (int hq = 0; hq < 2; ++hq) {
    if (ovm & (1ull << (32 * hq))) {
      load_query<CPL>(a.Q + (qi - half + hq) * a.d, a.d, t, q);
      const uint64_t k = root_scan_wave<KIND, LPN, CPL>(a, R, q, lane);
      if (half == hq) best_over = k;
    }
  }
  load_query<CPL>(a.Q + qs * a.d, a.d, t, q);
  // entries past the count hold stale values (dropped)
  const uint2 e0 = sl.ent[qs * kRootCap + hl], e1 = sl.ent[qs * kRootCap + 32 + hl];
  const bool l0 = !over && hl < cnt, l1 = !over && hl + 32 < cnt;
  const float v0 = l0 ? __uint_as_float(e0.x) : INFINITY;
  const float v1 = l1 ? __uint_as_float(e1.x) : INFINITY;
  float amin = fminf(v0, v1);
#pragma unroll
  for (int m = 16; m >= 1; m >>= 1) amin = fminf(amin, __shfl_xor(amin, m));
  const float T = amin + (qv ? sl.mq[qs] : 0.0f);
  // the rows with a <= T, gathered into rows[] (first entries, then second)
  const bool k0 = l0 && v0 <= T, k1 = l1 && v1 <= T;
  const uint32_t h0 = (uint32_t)(ballot(k0) >> (32 * half));
  const uint32_t h1 = (uint32_t)(ballot(k1) >> (32 * half));
  const uint32_t below = (1u << hl) - 1u;
  const int n0 = __popc(h0), total = n0 + __popc(h1);
  wave_sync();
  if (k0) rows[__popc(h0 & below)] = (int32_t)e0.y;
  if (k1) rows[n0 + __popc(h1 & below)] = (int32_t)e1.y;
  wave_sync();
  // the longer list sets the trip count: every lane joins each butterfly
  const int tmax = max(total, __shfl_xor(total, 32));
  uint64_t best = ~0ull;
  for (int b = 0; b < tmax; b += G) {
    const int32_t row = b + g < total ? rows[b + g] : -1;
    const bool valid = row >= 0;
    const float sc = (KIND == kFP8 && valid) ? R.scale[row] : 1.0f;
    const char* rp = static_cast<const char*>(R.vec) + (int64_t)(valid ? row : 0) * R.row_bytes;
    const float dist = group_distance<KIND, LPN, CPL>(q, rp, sc, t, a.nchunks, a.metric, valid);
    if (valid) {
      const uint64_t k = wkey(dist, row);
      best = k < best ? k : best;
    }
  }
#pragma unroll
  for (int m = 16; m >= 1; m >>= 1) {
    const uint64_t o = shfl_xor_u64(best, m);
    best = o < best ? o : best;
  }
  if (over) best = best_over;
  if (qv && hl == 0) out[qi] = best;
}

// Loads this query's k and beam width and finds the entry of the first
// searched layer: the root's smallest id, or the exact root nearest when the
// root carries the complete graph (from k_root_scan's or k_root_check's keys
// when given).
template <int KIND, int LPN, int CPL>
__device__ void start_query(const SearchArgs& a, int64_t qi, const float (&q)[CPL][8],
                            int lane, QState& st) {
  constexpr int G = 64 / LPN;
  const int t = lane % LPN, g = lane / LPN;
  // (written as two reads: a select between the addresses would make it a
  // vector load from the argument segment)
  int k = uni(a.k_all), ef = uni(a.ef_all);
  if (a.k_arr) k = uni(a.k_arr[qi]);
  if (a.ef_arr) ef = uni(a.ef_arr[qi]);
  k = min(max(k, 1), a.k_max);
  st.k = k;
  st.ef0 = min(max(ef, k), a.ef_cap);
  st.exps = st.evals = st.exps0 = st.evals0 = 0;
  st.need_init = 1;
  st.wsize = 0;
  int top = a.num_layers - 1;
  if (a.root_complete && top >= 1 && a.root_best) {
    // complete graph on the root, scanned by k_root_scan: min over the splits
    const SearchLayer& R = a.layer[top];
    uint64_t best = ~0ull;
    for (int sp = 0; sp < a.root_splits; ++sp) {
      const uint64_t kk = a.root_best[(int64_t)sp * a.nq + qi];
      best = kk < best ? kk : best;
    }
    best = uni_u64(best);
    st.evals = R.size;
    st.cur = uni(R.down[wkey_id(best)]);
    st.cur_d = wkey_dist(best);
    st.li = top - 1;
  } else if (a.root_complete && top >= 1) {
    // complete graph on the root: exhaustive scan for its nearest member
    const SearchLayer& R = a.layer[top];
    const uint64_t best = uni_u64(root_scan_wave<KIND, LPN, CPL>(a, R, q, lane));
    st.evals = R.size;
    st.cur = uni(R.down[wkey_id(best)]);
    st.cur_d = wkey_dist(best);
    st.li = top - 1;
  } else {
    // entry: the smallest id of the root layer (position 0)
    const SearchLayer& R = a.layer[top];
    const float sc = (KIND == kFP8) ? R.scale[0] : 1.0f;
    float dd = group_distance<KIND, LPN, CPL>(q, R.vec, sc, t, a.nchunks, a.metric, g == 0);
    st.cur_d = uni_f(dd);  // lane 0 holds group 0's distance
    st.cur = 0;
    st.li = top;
  }
}

// Rows each lane group gathers per pass of an expansion.
constexpr int kGatherRows = 3;

// FP8 traversal distances, one chunk of 8 coordinates at a time.  The
// converter turns two codes into f16 values multiplied by a power of two:
// it takes only the exponent of its FP32 scale operand, so with the row
// scale s = 2^e m (1 <= m < 2) it yields c 2^e exactly, and t = q - m (c 2^e)
// = q - s c is one packed f16 FMA with the query rounded to f16 (qh); sum t^2
// is accumulated in FP32 by pairwise dot products (each product exact).
// Inner products convert the codes unscaled and accumulate sum q c the same
// way, the caller applying -s.  This is the precision form's arithmetic: f16
// keeps 11 significant bits against the 4 of an E4M3 code, and the final
// list is re-ranked in FP32.  Chunk sums then go through the canonical tree,
// so the result does not depend on the launch shape.
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));

template <int CPL>
__device__ inline void query_f16(const float (&q)[CPL][8], h2_t (&qh)[CPL][4]) {
#pragma unroll
  for (int i = 0; i < CPL; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) qh[i][k] = h2_t{(_Float16)q[i][2 * k], (_Float16)q[i][2 * k + 1]};
}

// The mantissa m of a positive scale s = 2^e m, as an f16 pair.
__device__ inline h2_t scale_mantissa(float s) {
  const _Float16 m = (_Float16)__uint_as_float((__float_as_uint(s) & 0x007fffffu) | 0x3f800000u);
  return h2_t{m, m};
}

__device__ inline float fp8_chunk_l2(const uint2 w, const h2_t (&qh)[4], float s, h2_t nm) {
  const h2_t x0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w.x, s, false);
  const h2_t x1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w.x, s, true);
  const h2_t x2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w.y, s, false);
  const h2_t x3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w.y, s, true);
  // nm = -m: t = q - m x in one rounding
  const h2_t t0 = __builtin_elementwise_fma(nm, x0, qh[0]);
  const h2_t t1 = __builtin_elementwise_fma(nm, x1, qh[1]);
  const h2_t t2 = __builtin_elementwise_fma(nm, x2, qh[2]);
  const h2_t t3 = __builtin_elementwise_fma(nm, x3, qh[3]);
  float acc = __builtin_amdgcn_fdot2(t0, t0, 0.0f, false);
  acc = __builtin_amdgcn_fdot2(t1, t1, acc, false);
  acc = __builtin_amdgcn_fdot2(t2, t2, acc, false);
  return __builtin_amdgcn_fdot2(t3, t3, acc, false);
}

__device__ inline float fp8_chunk_ip(const uint2 w, const h2_t (&qh)[4]) {
  const h2_t x0 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w.x, 1.0f, false);
  const h2_t x1 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w.x, 1.0f, true);
  const h2_t x2 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w.y, 1.0f, false);
  const h2_t x3 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w.y, 1.0f, true);
  float acc = __builtin_amdgcn_fdot2(qh[0], x0, 0.0f, false);
  acc = __builtin_amdgcn_fdot2(qh[1], x1, acc, false);
  acc = __builtin_amdgcn_fdot2(qh[2], x2, acc, false);
  return __builtin_amdgcn_fdot2(qh[3], x3, acc, false);
}

// One chunk's partial distance in the traversal: the canonical FP32 sum
// (henn_device.h) for FP32 and BF16 rows, the f16 form above for FP8 rows.
template <int KIND, bool L2>
__device__ inline float traversal_chunk(const ChunkRaw<KIND>& raw, const float (&q)[8],
                                        const h2_t (&qh)[4], float sc, h2_t nm) {
  if constexpr (KIND == kFP8) {
    return L2 ? fp8_chunk_l2(raw.a, qh, sc, nm) : fp8_chunk_ip(raw.a, qh);
  } else {
    float x[8];
    raw.decode(x);
    return L2 ? chunk_l2(q, x, 1.0f, false) : chunk_ip(q, x);
  }
}

// This lane's chunk sums of NR fetched rows (tree over its CPL chunks; chunks
// past the row are dropped unless FULL), and their lane-group sums: rows 2p
// and 2p + 1 share one butterfly (group_distances_paired), after which the
// even lanes of a group hold row 2p's sum and the odd lanes row 2p + 1's, in
// d[2p]; an odd last row's sum is in d[NR - 1].
template <int KIND, int LPN, int CPL, int NR, bool FULL, bool L2>
__device__ inline void gather_sums(const ChunkRaw<KIND> (&raw)[NR][CPL], const float (&q)[CPL][8],
                                   const h2_t (&qh)[CPL][4], const float (&sc)[NR], int t,
                                   int nchunks, float (&d)[NR]) {
  float ts[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    // FP8: minus the mantissa of the row's scale (fp8_chunk_l2)
    const h2_t nm = (KIND == kFP8 && L2) ? -scale_mantissa(sc[r]) : h2_t{0, 0};
    float part[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const float v = traversal_chunk<KIND, L2>(raw[r][i], q[i], qh[i], sc[r], nm);
      part[i] = (FULL || t * CPL + i < nchunks) ? v : 0.0f;
    }
    ts[r] = tree_sum<CPL>(part);
    // wide rows: one row's arithmetic at a time, or the rows' decoded values
    // overflow the registers
    if constexpr (CPL * NR >= 16) __builtin_amdgcn_sched_barrier(0);
  }
  constexpr int NP = (LPN >= 2) ? NR / 2 : 0;  // row pairs
  const bool odd = (lane_id() & 1) != 0;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    float v = (odd ? ts[2 * p + 1] : ts[2 * p]) + dpp_mov<0xB1>(odd ? ts[2 * p] : ts[2 * p + 1]);
    d[2 * p] = group_sum_from2<LPN>(v);
  }
#pragma unroll
  for (int r = 2 * NP; r < NR; ++r) d[r] = group_sum<LPN>(ts[r]);
}

// What every expansion needs of the arguments, read once per query: a read
// inside the loop would be a scalar-memory round trip in the chain.
struct StepArgs {
  int vis_bits, vis_bytes, nchunks, metric;
  __device__ explicit StepArgs(const SearchArgs& a)
      : vis_bits(uni(a.vis_bits)), vis_bytes(uni(a.vis_bytes)), nchunks(uni(a.nchunks)),
        metric(uni(a.metric)) {}
};

// Visited table: byte offset of id u's entry and the value stored there (see
// vis_tag_bytes; 4-byte entries hold the id itself, at a hashed slot).
__device__ inline void vis_slot(const StepArgs& a, int32_t u, uint32_t& at, uint32_t& tag) {
  uint32_t h = (uint32_t)u & ((1u << a.vis_bits) - 1u);
  tag = ((uint32_t)u >> a.vis_bits) + 1u;
  if (a.vis_bytes == 4) {
    h = ((uint32_t)u * 2654435761u) >> (32 - a.vis_bits);
    tag = (uint32_t)u;
  }
  at = h << (a.vis_bytes >> 1);
}

// Stores the tag where mark is set.  The width is decided outside of the
// predicated stores, so that those are single instructions.
__device__ inline void vis_mark(const StepArgs& a, const WaveLds& s, uint32_t at, uint32_t tag,
                                bool mark) {
  char* e = static_cast<char*>(s.vis) + at;
  if (a.vis_bytes == 1) {
    if (mark) *reinterpret_cast<uint8_t*>(e) = (uint8_t)tag;
  } else {
    if (mark) *reinterpret_cast<uint16_t*>(e) = (uint16_t)tag;
    if (a.vis_bytes == 4 && mark) *reinterpret_cast<uint16_t*>(e + 2) = (uint16_t)(tag >> 16);
  }
}

// One gather pass: rows [base, base + NR * G) of this expansion's fresh
// candidates (crow / cidk / csc of s), their distances, and their keys into ckey.
// FULL: the row has exactly LPN * CPL chunks, so lane t's chunks
// t * CPL .. t * CPL + CPL - 1 are contiguous and read at constant offsets
// from one pointer; otherwise chunk indices past the row are clamped to
// chunk 0 and their sums dropped (group_distances).  Every lane of the
// wave takes part (butterflies); a slot at or past cnt computes the pass's
// first row again and writes nothing.  Distances are the canonical sums of
// henn_device.h.
// after_issue() runs once every load of the pass is issued and before the
// first is waited for: loads return in order, so what it issues does not
// delay them, and is itself back by the time they have been used.
template <int KIND, int LPN, int CPL, int NR, bool FULL, bool L2, typename F>
__device__ inline void gather_pass(const StepArgs& a, const SearchLayer& L,
                                   const float (&q)[CPL][8], const h2_t (&qh)[CPL][4],
                                   const WaveLds& s, int base, int cnt, int t, int g,
                                   F&& after_issue) {
  constexpr int G = 64 / LPN;
  constexpr int CB = KIND == kF32 ? 32 : KIND == kBF16 ? 16 : 8;  // bytes per chunk
  const char* vec = static_cast<const char*>(L.vec);
  const void* rows[NR];
  float sc[NR];
  uint32_t idk[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int ci = base + r * G + g;
    // an empty slot re-reads the pass's first row, which its group reads anyway
    const int e = ci < cnt ? ci : base;
    const uint32_t ch = s.crow[e] + (FULL ? (uint32_t)(t * CPL) : 0u);
    rows[r] = vec + (size_t)ch * CB;
    idk[r] = s.cidk[e];
    sc[r] = (KIND == kFP8) ? s.csc[e] : 1.0f;
  }
  ChunkRaw<KIND> raw[NR][CPL];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const int c = t * CPL + i;
      raw[r][i].fetch(rows[r], FULL ? i : c < a.nchunks ? c : 0);
    }
  after_issue();
  // keys: (ordered distance bits << 32) | (id << 1).  Squared L2 distances
  // are sums of squares, never negative or -0, so their ordered bits are
  // the float bits with the sign bit set (ordered_bits on that range).  For
  // inner products 0 (a NaN of all ones) would fall below the register list's
  // fillers, and becomes 1.
  constexpr int NP = (LPN >= 2) ? NR / 2 : 0;  // row pairs (gather_sums)
  const bool odd = (lane_id() & 1) != 0;
  float d[NR];
  uint32_t ob[NR];
  gather_sums<KIND, LPN, CPL, NR, FULL, L2>(raw, q, qh, sc, t, a.nchunks, d);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if constexpr (L2) {
      ob[r] = __float_as_uint(d[r]) | 0x80000000u;
    } else {
      constexpr int last = NR - 1;
      const float s0 = sc[r], s1 = sc[r < last ? r + 1 : last];
      const float scale = (r < 2 * NP && (r & 1) == 0 && odd) ? s1 : s0;
      ob[r] = max(ordered_bits((KIND == kFP8) ? -(scale * d[r]) : -d[r]), 1u);
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int r = 2 * p;
    const int ci = base + (r + (odd ? 1 : 0)) * G + g;
    // (a select between array elements would put the array into memory)
    const uint32_t id = idk[r] ^ ((idk[r] ^ idk[r + 1]) & (odd ? 0xffffffffu : 0u));
    if (t < 2 && ci < cnt) s.ckey[ci] = ((uint64_t)ob[r] << 32) | id;
  }
#pragma unroll
  for (int r = 2 * NP; r < NR; ++r) {
    const int ci = base + r * G + g;
    if (t == 0 && ci < cnt) s.ckey[ci] = ((uint64_t)ob[r] << 32) | idk[r];
  }
}

// All gather passes of one expansion, each with every load of its rows in
// flight together: up to kGatherRows * G rows per pass, the last pass sized
// to the rows left.  after_issue: in the first pass (see gather_pass), also
// when there is no row.
template <int KIND, int LPN, int CPL, bool FULL, bool L2, typename F>
__device__ inline void gather_metric(const StepArgs& a, const SearchLayer& L,
                                     const float (&q)[CPL][8], const h2_t (&qh)[CPL][4],
                                     const WaveLds& s, int cnt, int t, int g, F&& after_issue) {
  constexpr int G = 64 / LPN;
  static_assert(kGatherRows == 3, "pass sizes below");
  // three FP32 rows of eight chunks a lane do not fit the registers
  constexpr bool kThree = !(KIND == kF32 && CPL >= 8);
  auto pass = [&](int base, auto&& f) -> int {
    const int rest = cnt - base;
    if constexpr (kThree) {
      if (rest > 2 * G) {
        gather_pass<KIND, LPN, CPL, 3, FULL, L2>(a, L, q, qh, s, base, cnt, t, g, f);
        return 3 * G;
      }
    }
    if (rest > G) {
      gather_pass<KIND, LPN, CPL, 2, FULL, L2>(a, L, q, qh, s, base, cnt, t, g, f);
      return 2 * G;
    }
    gather_pass<KIND, LPN, CPL, 1, FULL, L2>(a, L, q, qh, s, base, cnt, t, g, f);
    return G;
  };
  if (cnt == 0) {
    after_issue();
    return;
  }
  for (int base = pass(0, after_issue); base < cnt;) base += pass(base, [] {});
}

template <int KIND, int LPN, int CPL, bool FULL, typename F>
__device__ inline void gather_all(const StepArgs& a, const SearchLayer& L,
                                  const float (&q)[CPL][8], const h2_t (&qh)[CPL][4],
                                  const WaveLds& s, int cnt, int t, int g, F&& after_issue) {
  // the metric outside of the passes: inside, the two forms' common decoding
  // is done ahead of the branch and held
  if (a.metric == 0)
    gather_metric<KIND, LPN, CPL, FULL, true>(a, L, q, qh, s, cnt, t, g, after_issue);
  else
    gather_metric<KIND, LPN, CPL, FULL, false>(a, L, q, qh, s, cnt, t, g, after_issue);
}

// Starts a layer: the visited set emptied and the entry st.cur marked in it;
// for FP8 rows the entry's distance in the traversal's own form: the one
// handed down (a root scan, or the first distance of the root) is the
// canonical FP32 sum, and the list's duplicate check compares keys.
template <int KIND, int LPN, int CPL, bool FULL, bool EXACT>
__device__ inline void layer_begin(const StepArgs& a, const SearchLayer& L,
                                   const float (&q)[CPL][8], const h2_t (&qh)[CPL][4],
                                   const WaveLds& s, QState& st, int t, int g, uint32_t* vis_bm) {
  const int lane = s.lane;
  if (st.li == 0) {
    st.exps0 = st.exps;
    st.evals0 = st.evals;
  }
  st.evals += 1;  // the entry (its distance is carried down, counted per layer)
  if constexpr (EXACT) {
    // the exact set: one bit per member of the layer, in the workspace
    const int64_t words = ((int64_t)L.size + 31) >> 5;
    for (int64_t i = lane; i < words; i += 64) vis_bm[i] = 0u;
    __builtin_amdgcn_s_waitcnt(0);  // cleared before the first bit is set
  } else {
    // empty: tag 0 (8 / 16-bit) or id -1 (32-bit); at least 256 bytes, so
    // whole 16-byte words
    const int n16 = (a.vis_bytes << a.vis_bits) >> 4;
    const uint32_t e = a.vis_bytes < 4 ? 0u : 0xffffffffu;
    for (int i = lane; i < n16; i += 64) static_cast<uint4*>(s.vis)[i] = make_uint4(e, e, e, e);
  }
  if constexpr (KIND == kFP8) {
    if (lane == 0) {
      s.crow[0] = (uint32_t)st.cur * (uint32_t)a.nchunks;
      s.cidk[0] = (uint32_t)st.cur << 1;
      s.csc[0] = L.scale[st.cur];
    }
    wave_sync();
    gather_all<KIND, LPN, CPL, FULL>(a, L, q, qh, s, 1, t, g, [] {});
    wave_sync();
    st.cur_d = wkey_dist(uni_u64(s.ckey[0]));
  }
  wave_sync();
  if constexpr (EXACT) {
    if (lane == 0) atomicOr(vis_bm + (st.cur >> 5), 1u << (st.cur & 31));
  } else {
    uint32_t at, tag;
    vis_slot(a, st.cur, at, tag);
    vis_mark(a, s, at, tag, lane == 0);
  }
  st.wsize = 1;
  st.need_init = 0;
}

// The lanes whose neighbour u (-1: none) the visited table does not hold; it
// holds them afterwards.  Every lane reads the word that holds its entry (-1
// has a slot too), whatever an entry's width, so that the read needs no
// branches.
__device__ inline uint64_t vis_filter(const StepArgs& a, const WaveLds& s, int32_t u) {
  uint32_t at, tag;
  vis_slot(a, u, at, tag);
  const uint32_t word = *reinterpret_cast<const uint32_t*>(static_cast<char*>(s.vis) + (at & ~3u));
  const uint32_t old = (word >> ((at & 3u) * 8)) & (0xffffffffu >> (32 - 8 * a.vis_bytes));
  const bool fresh = (u >= 0) & (old != tag);
  const uint64_t fm = ballot(fresh);
  wave_sync();
  vis_mark(a, s, at, tag, fresh);
  return fm;
}

// The fresh ones of this expansion's neighbours (u, -1: none; usc: its FP8
// scale) take the compacted slots 0, 1, ...; returns how many.
template <int KIND, bool EXACT>
__device__ inline int take_fresh(const StepArgs& a, const WaveLds& s, int32_t u, float usc,
                                 uint32_t* vis_bm) {
  uint64_t fm;
  if constexpr (EXACT) {
    // exact set: the bit's old value says whether u was seen (the
    // update is atomic, so of lanes holding one id only one finds it new)
    bool fresh = false;
    if (u >= 0) {
      const uint32_t bit = 1u << (u & 31);
      fresh = !(atomicOr(vis_bm + (u >> 5), bit) & bit);
    }
    fm = ballot(fresh);
  } else {
    fm = vis_filter(a, s, u);
  }
  const int rb = rank_below(fm);
  if (__builtin_amdgcn_inverse_ballot_w64(fm)) {
    s.crow[rb] = (uint32_t)u * (uint32_t)a.nchunks;
    s.cidk[rb] = (uint32_t)u << 1;
    if (KIND == kFP8) s.csc[rb] = usc;
  }
  wave_sync();
  return popc64(fm);
}

// Runs up to `budget` expansions from the current state (layer changes are
// free).  Returns true once the layer-0 beam has no unexpanded entry; then
// W (this wave's LDS list) holds the final list (st.wsize entries).  q: this
// lane's FP32 query slice; qh: the same in f16 pairs (read by the FP8 form
// only, which then never reads q).
// This form keeps the list in LDS: beams wider than the register form's 256,
// and the exact visited set (an analysis form).
template <int KIND, int LPN, int CPL, bool FULL, bool EXACT = false>
__device__ bool advance(const SearchArgs& a, const float (&q)[CPL][8], const h2_t (&qh)[CPL][4],
                        WaveLds s, uint64_t* W, QState& st, int budget, uint32_t* vis_bm) {
  const int lane = s.lane, t = lane % LPN, g = lane / LPN;
  const StepArgs h(a);
  for (;;) {
    const SearchLayer L = a.layer[st.li];
    const int efl = st.li == 0 ? st.ef0 : min(a.ef_upper, a.ef_cap);
    if (st.need_init) {
      layer_begin<KIND, LPN, CPL, FULL, EXACT>(h, L, q, qh, s, st, t, g, vis_bm);
      if (lane == 0) W[0] = wkey(st.cur_d, st.cur);
      wave_sync();
    }
    int wsize = st.wsize;
    bool layer_done = false;
    while (budget > 0) {
      // smallest unexpanded entry of W
      int pos = -1;
      for (int base = 0; base < wsize; base += 64) {
        const int i = base + lane;
        const bool un = i < wsize && !(W[i] & 1ull);
        const uint64_t m = ballot(un);
        if (m) {
          pos = base + __ffsll((unsigned long long)m) - 1;
          break;
        }
      }
      if (pos < 0) {
        layer_done = true;
        break;
      }
      --budget;
      const uint64_t ck = uni_u64(W[pos]);
      wave_sync();
      if (lane == 0) W[pos] = ck | 1ull;
      const int32_t c = wkey_id(ck);
      ++st.exps;

      // neighbour ids (and, for FP8 rows, their scales) and the visited filter
      int32_t u = -1;
      float usc = 1.0f;
      if (lane < L.deg) {
        u = L.adj[(int64_t)c * L.deg + lane];
        if (KIND == kFP8) usc = L.adj_scale[(int64_t)c * L.deg + lane];
      }
      const int cnt = take_fresh<KIND, EXACT>(h, s, u, usc, vis_bm);
      st.evals += cnt;

      // gather + distance (the scales ride in kstage, free until the merge)
      gather_all<KIND, LPN, CPL, FULL>(h, L, q, qh, s, cnt, t, g, [] {});
      wave_sync();

      // merge the new keys into W (truncated to efl)
      const uint64_t key = lane < cnt ? s.ckey[lane] : ~0ull;
      bool keep = lane < cnt;
      if (keep && wsize >= efl) keep = key < wkey_strip(W[efl - 1]);
      // nothing can enter a full list: skip the merge (common late in a search)
      if (!ballot(keep)) continue;
      // lo = number of W entries below key (fixed-step lower bound: the trip
      // count depends only on the wave-uniform list size)
      int lo = 0;
      for (int step = pow2_floor(wsize); step > 0; step >>= 1)
        if (lo + step <= wsize && wkey_strip(W[lo + step - 1]) < key) lo += step;
      if (keep && lo < wsize && wkey_strip(W[lo]) == key) keep = false;  // already in W
      const uint64_t km = ballot(keep);
      const int nk = popc64(km);
      if (nk == 0) continue;
      if (keep) s.kstage[rank_below(km)] = key;
      // pad to a multiple of 4 (at most 64 slots) with keys below which
      // nothing ranks, so the count below reads four keys per step
      const int nk4 = (nk + 3) & ~3;
      if (lane >= nk && lane < nk4) s.kstage[lane] = ~0ull;
      wave_sync();
      int rk = 0;  // kept keys below this one
      if (keep)
        for (int j = 0; j < nk4; j += 4)
          rk += (s.kstage[j] < key) + (s.kstage[j + 1] < key) + (s.kstage[j + 2] < key) +
                (s.kstage[j + 3] < key);
      // a kept key lands at p = lo + rk: the p are distinct and ascend with
      // the key; the entries below the smallest stay where they are
      const int p = lo + rk;
      const uint64_t m0 = ballot(keep && rk == 0);
      const int lo_min = uni(__shfl(lo, __ffsll((unsigned long long)m0) - 1));
      const int nsize = min(efl, wsize + nk);
      wave_sync();
      // slot map (in kstage, free again): bit x of word x >> 6 marks the
      // positions that take a kept key; nsize <= 2048 needs at most 32 words.
      // The words are cleared as 32-bit halves: a 64-bit zero is otherwise
      // kept live in two registers through the whole expansion loop.
      uint64_t* slot = s.kstage;
      const int w0 = lo_min >> 6;
      if (lane <= ((nsize - 1) >> 6) - w0) {
        uint32_t* sw = reinterpret_cast<uint32_t*>(slot + w0 + lane);
        sw[0] = 0u;
        sw[1] = 0u;
      }
      wave_sync();
      if (keep && p < nsize) atomicOr(reinterpret_cast<unsigned long long*>(&slot[p >> 6]),
                                      1ull << (p & 63));
      wave_sync();
      // in place, by output position: a position x in [lo_min, nsize) that
      // takes no key takes W[x - K(x)], K(x) the key positions below x.  The
      // source never lies above x, so blocks of 64 go from the top down and
      // each reads its sources whole before it writes.
      int kb = popc64(ballot(keep && p < nsize));  // then: key positions below block b
      for (int b = (nsize - 1) & ~63; b >= 0 && b + 64 > lo_min; b -= 64) {
        const int x = b + lane;
        const uint64_t mask = uni_u64(slot[b >> 6]);
        kb -= popc64(mask);
        const int below = rank_below(mask);
        const int kx = kb + below;
        // x takes a key when the count through this lane exceeds the one
        // below (counted, not tested as mask & (1 << lane): that lane mask
        // would stay live in two registers)
        const bool is_key = rank_below(mask >> 1) + (int)(mask & 1ull) != below;
        const bool mv = x >= lo_min && x < nsize && !is_key && kx > 0;
        uint64_t wv = 0;
        if (mv) wv = W[x - kx];
        wave_sync();
        if (mv) W[x] = wv;
        wave_sync();
      }
      if (keep && p < nsize) W[p] = key;
      wave_sync();
      wsize = nsize;
    }
    st.wsize = wsize;
    if (!layer_done) return false;
    if (st.li == 0) return true;
    // hand the best node down the inter-layer edge
    const uint64_t best = uni_u64(W[0]);
    st.cur = uni(L.down[wkey_id(best)]);
    st.cur_d = wkey_dist(best);
    st.li -= 1;
    st.need_init = 1;
    wave_sync();
  }
}

// The same traversal with the list in registers (ef_cap <= 64 NB; the caller
// holds it in R).  An expansion is a chain of two memory round trips (the
// adjacency row, then the fresh rows) and the list work between them, and a
// launch that does not fill the chip runs at that chain's latency.  Here the
// list costs no LDS round trip, only compares, ballots and lane moves, and the
// neighbours of the entry that comes next as the list stands are read while
// this one's rows are: unless a new key overtakes it, the next expansion
// starts with its adjacency row at hand.  Against the list in LDS and no
// reading ahead, k_search with its root scan: one query on 10,000 x 32 FP32,
// beam 32, 77 -> 54 us; 48 queries on 300,000 x 128 FP8, beam 84, 260 -> 194;
// 100,000 with mixed beams on 1.2M x 128 FP8 7.08 -> 5.68 ms.
template <int KIND, int LPN, int CPL, bool FULL, int NB>
__device__ bool advance_reg(const SearchArgs& a, const float (&q)[CPL][8],
                            const h2_t (&qh)[CPL][4], WaveLds s, RegList<NB>& R, QState& st,
                            int budget) {
  const int lane = s.lane, t = lane % LPN, g = lane / LPN;
  const StepArgs h(a);
  for (;;) {
    const SearchLayer L = a.layer[st.li];
    const int efl = st.li == 0 ? st.ef0 : min(a.ef_upper, a.ef_cap);
    const int off = 64 * NB - efl;
    if (st.need_init) {
      layer_begin<KIND, LPN, CPL, FULL, false>(h, L, q, qh, s, st, t, g, nullptr);
      uint64_t k0 = wkey(st.cur_d, st.cur);
      if ((k0 >> 32) == 0) k0 |= 1ull << 32;  // above the fillers (see gather_pass)
      list_start(R, lane, efl, uni_u64(k0));
      wave_sync();
    }
    // lanes past the row read its last entry and drop it
    const int al = min(lane, L.deg - 1);
    auto read_row = [&](int32_t c, int32_t& u, float& usc) {
      u = L.adj[(int64_t)c * L.deg + al];
      if (KIND == kFP8) usc = L.adj_scale[(int64_t)c * L.deg + al];
    };
    // the first unexpanded entry's id, -1 for none, and its place (b_out,
    // bit); every block's candidate is read and one selected, which is
    // cheaper than a branch
    auto first_open = [&](int& b_out, uint64_t& bit) -> int32_t {
      int32_t id = -1;
      bit = 0;
      b_out = 0;
#pragma unroll
      for (int b = NB - 1; b >= 0; --b) {
        const uint64_t m = ~R.ex[b];
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)R.w[b],
                                                                m ? __builtin_ctzll(m) : 0);
        id = m ? (int32_t)(lo >> 1) : id;
        bit = m ? m & (0ull - m) : bit;
        b_out = m ? b : b_out;
      }
      return id;
    };
    bool layer_done = false;
    int32_t next = -1, next_u = -1;  // the entry read ahead, its neighbours
    float next_usc = 1.0f;
    while (budget > 0) {
      int b = 0;
      uint64_t bit = 0;
      const int32_t c = first_open(b, bit);
      if (c < 0) {
        layer_done = true;
        break;
      }
      --budget;
      ++st.exps;
#pragma unroll
      for (int i = 0; i < NB; ++i) R.ex[i] |= i == b ? bit : 0ull;
      int32_t u = next_u;
      float usc = next_usc;
      if (c != next) read_row(c, u, usc);
      next = first_open(b, bit);
      const int cnt = take_fresh<KIND, false>(h, s, lane < L.deg ? u : -1, usc, nullptr);
      st.evals += cnt;
      gather_all<KIND, LPN, CPL, FULL>(h, L, q, qh, s, cnt, t, g,
                                       [&] { read_row(next >= 0 ? next : c, next_u, next_usc); });
      wave_sync();
      const uint64_t key = lane < cnt ? s.ckey[lane] : ~0ull;
      uint64_t open = ballot(key < readlane_u64(R.w[NB - 1], 63));
      while (open) {
        const uint64_t k = readlane_u64(key, __builtin_ctzll(open));
        open &= open - 1;
        if (list_insert(R, off, k)) {
          st.wsize += 1;
          open &= ballot(key < readlane_u64(R.w[NB - 1], 63));
        }
      }
      wave_sync();  // the candidate slots are read before the next expansion writes them
    }
    st.wsize = min(st.wsize, efl);
    if (!layer_done) return false;
    if (st.li == 0) return true;
    // hand the best node down the inter-layer edge
    uint64_t best = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b)
      if (off >> 6 == b) best = readlane_u64(R.w[b], off & 63);
    st.cur = uni(L.down[wkey_id(best)]);
    st.cur_d = wkey_dist(best);
    st.li -= 1;
    st.need_init = 1;
    wave_sync();
  }
}

// Writes the first k results (after the FP32 re-rank for the precision
// forms) to out_ids / out_dist (k_max entries, padded) and the counters.
template <int KIND, int LPN, int CPL>
__device__ void finish_query(const SearchArgs& a, const float (&q)[CPL][8], int lane,
                             uint64_t* W, const QState& st, int32_t* out_ids, float* out_dist,
                             int32_t* counters) {
  constexpr int G = 64 / LPN;
  const int t = lane % LPN, g = lane / LPN;
  const int k = st.k, wsize = st.wsize;
  if (a.rerank_vec == nullptr) {
    for (int j = lane; j < a.k_max; j += 64) {
      int32_t id = -1;
      float dd = INFINITY;
      if (j < k && j < wsize) {
        id = wkey_id(W[j]);
        dd = wkey_dist(W[j]);
        if (a.ids0) id = a.ids0[id];
      }
      out_ids[j] = id;
      out_dist[j] = dd;
    }
  } else {
    // FP32 re-rank of the first min(|W|, rerank_factor*k) entries
    const int nr = min(wsize, a.rerank_factor * k);
    for (int base = 0; base < nr; base += G) {
      const int ci = base + g;
      const bool valid = ci < nr;
      const int32_t id = valid ? wkey_id(W[ci]) : 0;
      const float dist = group_distance<kF32, LPN, CPL>(
          q, a.rerank_vec + (int64_t)id * a.dpad, 1.0f, t, a.nchunks, a.metric, valid);
      // in place: a group reads its entry before the distance and writes it after
      if (valid && t == 0) W[ci] = wkey(dist, id);
    }
    const int n2 = next_pow2_dev(nr);
    for (int i = nr + lane; i < n2; i += 64) W[i] = ~0ull;
    wave_sync();
    wave_bitonic_sort(W, n2);
    for (int j = lane; j < a.k_max; j += 64) {
      int32_t id = -1;
      float dd = INFINITY;
      if (j < k && j < nr) {
        id = wkey_id(W[j]);
        dd = wkey_dist(W[j]);
        if (a.ids0) id = a.ids0[id];
      }
      out_ids[j] = id;
      out_dist[j] = dd;
    }
  }
  if (counters && lane == 0) {
    counters[0] = st.exps;
    counters[1] = st.evals;
    counters[2] = st.exps - st.exps0;
    counters[3] = st.evals - st.evals0;
  }
  wave_sync();
}

// The per-query time output, read from the kernel's argument segment (where a
// is) at the point of use through an opaque pointer: the traversal keeps its
// scalar registers full, and a pointer held across it would spill.  The
// segment's address comes from the kernel: asked for here, it is null wherever
// the compiler makes a called function of search_one.
__device__ __forceinline__ int64_t* query_ns_arg(const SearchArgs& a) {
  auto* kp = (const __attribute__((address_space(4))) char*)&a;
  asm volatile("" : "+s"(kp));
  return reinterpret_cast<const SearchArgs*>((const char*)kp)->query_ns;
}

template <int KIND, int LPN, int CPL, bool FULL, bool EXACT, int NB>
__device__ void search_one(const SearchArgs& a, int64_t qi, WaveLds s) {
  s.lane = fresh_lane();
  // the constant-rate clock when times are asked for; the start waits in the
  // query's output word (volatile: a memory round trip, so no register stays
  // live across the traversal)
  if (int64_t* qt = query_ns_arg(a)) {
    if (s.lane == 0) *reinterpret_cast<volatile int64_t*>(qt + qi) = (int64_t)wall_clock64();
  }
  const int t = s.lane % LPN;
  float q[CPL][8];
  load_query<CPL>(a.Q + qi * a.d, a.d, t, q);
  QState st;
  start_query<KIND, LPN, CPL>(a, qi, q, s.lane, st);
  h2_t qh[CPL][4];
  if constexpr (KIND == kFP8) query_f16<CPL>(q, qh);
  uint64_t* W = s.W;
  if constexpr (NB == 0) {
    uint32_t* vis_bm = EXACT ? a.vis_exact + qi * a.vis_exact_words : nullptr;
    advance<KIND, LPN, CPL, FULL, EXACT>(a, q, qh, s, W, st, 0x7fffffff, vis_bm);
  } else {
    RegList<NB> R;
    advance_reg<KIND, LPN, CPL, FULL, NB>(a, q, qh, s, R, st, 0x7fffffff);
    list_store(R, s.lane, st.ef0, st.wsize, W, false);
    wave_sync();
  }
  // the FP8 traversal holds only the f16 query; the FP32 re-rank reads it again
  if constexpr (KIND == kFP8) load_query<CPL>(a.Q + qi * a.d, a.d, t, q);
  finish_query<KIND, LPN, CPL>(a, q, s.lane, W, st, a.out_ids + qi * a.k_max,
                               a.out_dist + qi * a.k_max,
                               a.counters ? a.counters + qi * 4 : nullptr);
  int64_t* qt = query_ns_arg(a);
  if (qt && s.lane == 0) {
    volatile int64_t* slot = reinterpret_cast<volatile int64_t*>(qt + qi);
    const uint32_t ticks = (uint32_t)((uint64_t)wall_clock64() - (uint64_t)*slot);
    *slot = (int64_t)((double)ticks * a.clock_ns);
  }
}

// ---------------------------------------------------------- serving ------
// One tick of the serving form: every active slot advances by at most
// `budget` expansions.  A slot's state (QState, its list W and visited
// table) lives in HBM between ticks at arena + state_off[slot]; it is
// loaded into this wave's LDS, advanced, and stored back.  A slot that
// finishes appends its slot and result row to the tick's compact completion
// list.  The traversal is the batch kernel's own code, so
// a request's result does not depend on which others share its ticks.
template <int KIND, int LPN, int CPL, bool FULL, int NB>
__device__ __forceinline__ void serve_step_body(const SearchArgs& a, const ServeArgs& sv,
                                                int per_wave_bytes, int waves_per_block) {
  extern __shared__ __align__(16) char smem[];
  const int wave = uni(threadIdx.x >> 6);
  const int64_t idx = (int64_t)blockIdx.x * waves_per_block + wave;
  if (blockIdx.x == 0 && threadIdx.x == 0) *sv.done_clear = 0;
  if (idx >= sv.n_active) return;
  const int lane = lane_id(), t = lane % LPN;
  const int32_t slot = uni(sv.active[idx]);
  WaveLds s = carve<NB>(smem + (size_t)wave * per_wave_bytes, a.ef_cap);
  float q[CPL][8];
  load_query<CPL>(a.Q + (int64_t)slot * a.d, a.d, t, q);
  QState st = sv.states[slot];
  st.li = uni(st.li);
  st.need_init = uni(st.need_init);
  st.wsize = uni(st.wsize);
  st.cur = uni(st.cur);
  st.cur_d = uni_f(st.cur_d);
  st.k = uni(st.k);
  st.ef0 = uni(st.ef0);
  char* base = sv.arena + sv.state_off[slot];
  uint64_t* gW = reinterpret_cast<uint64_t*>(base);
  uint32_t* gvis = reinterpret_cast<uint32_t*>(base + (size_t)sv.cap[slot] * 8);
  const int vis_n = (1 << a.vis_bits) * a.vis_bytes / 4;  // 32-bit words of the table
  // the list's width in the layer the state was saved in
  auto width = [&]() { return st.li == 0 ? st.ef0 : min(a.ef_upper, a.ef_cap); };
  RegList<NB == 0 ? 1 : NB> R;
  if (st.li == kSlotNew) {
    start_query<KIND, LPN, CPL>(a, slot, q, lane, st);
  } else if (!st.need_init) {
    if constexpr (NB == 0) {
      for (int i = lane; i < st.wsize; i += 64) s.W[i] = gW[i];
    } else {
      list_load(R, lane, width(), st.wsize, gW);
    }
    for (int i = lane; i < vis_n; i += 64) static_cast<uint32_t*>(s.vis)[i] = gvis[i];
    wave_sync();
  }
  uint64_t* W = s.W;
  h2_t qh[CPL][4];
  if constexpr (KIND == kFP8) query_f16<CPL>(q, qh);
  bool done;
  if constexpr (NB == 0) {
    done = advance<KIND, LPN, CPL, FULL>(a, q, qh, s, W, st, sv.budget, nullptr);
  } else {
    done = advance_reg<KIND, LPN, CPL, FULL, NB>(a, q, qh, s, R, st, sv.budget);
    if (done) {
      list_store(R, s.lane, st.ef0, st.wsize, W, false);
      wave_sync();
    }
  }
  if (done) {
    if constexpr (KIND == kFP8) load_query<CPL>(a.Q + (int64_t)slot * a.d, a.d, t, q);
    // finished: append (slot, row) to this tick's compact completion list
    int pos = 0;
    if (lane == 0) pos = atomicAdd(sv.done_count, 1);
    pos = __shfl(pos, 0);
    int32_t* row = sv.done_rows + (int64_t)pos * (1 + 2 * a.k_max);
    finish_query<KIND, LPN, CPL>(a, q, s.lane, W, st, row + 1,
                                 reinterpret_cast<float*>(row + 1 + a.k_max), nullptr);
    st.li = kSlotDone;
    if (lane == 0) row[0] = slot;
  } else if (!st.need_init) {
    if constexpr (NB == 0) {
      for (int i = lane; i < st.wsize; i += 64) gW[i] = W[i];
    } else {
      list_store(R, lane, width(), st.wsize, gW, true);
    }
    for (int i = lane; i < vis_n; i += 64) gvis[i] = static_cast<uint32_t*>(s.vis)[i];
  }
  if (lane == 0) sv.states[slot] = st;
}

template <int KIND, int LPN, int CPL, bool FULL, int NB>
__global__ __launch_bounds__(512) void k_serve_step(SearchArgs a, ServeArgs sv, int per_wave_bytes,
                                                    int waves_per_block) {
  serve_step_body<KIND, LPN, CPL, FULL, NB>(a, sv, per_wave_bytes, waves_per_block);
}

// The FP8 form with at most two chunks per lane fits 80 registers without
// spilling in the traversal loop; held to that, six waves share a SIMD (the
// LDS of a wave at the usual beam widths also allows six).
template <int KIND, int CPL, int NB>
constexpr bool six_waves() { return KIND == kFP8 && CPL <= 2 && NB <= 2; }

template <int KIND, int LPN, int CPL, bool FULL, int NB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(6))) void k_serve_step6(
    SearchArgs a, ServeArgs sv, int per_wave_bytes, int waves_per_block) {
  serve_step_body<KIND, LPN, CPL, FULL, NB>(a, sv, per_wave_bytes, waves_per_block);
}

template <int KIND, int LPN, int CPL, bool FULL, int NB>
static auto serve_kernel() {
  if constexpr (six_waves<KIND, CPL, NB>())
    return &k_serve_step6<KIND, LPN, CPL, FULL, NB>;
  else
    return &k_serve_step<KIND, LPN, CPL, FULL, NB>;
}

static __global__ void k_serve_admit(const float* staged_q, const int32_t* meta, int n_new, int d,
                              float* slot_q, int32_t* slot_k, int32_t* slot_ef,
                              int64_t* state_off, int32_t* cap, QState* states,
                              const uint64_t* root_keys, uint64_t* slot_root) {
  // meta per new request: slot, k, ef, cap, offset (lo, hi)
  const int r = blockIdx.x;
  if (r >= n_new) return;
  const int32_t* m = meta + r * 6;
  const int32_t slot = m[0];
  for (int j = threadIdx.x; j < d; j += blockDim.x)
    slot_q[(int64_t)slot * d + j] = staged_q[(int64_t)r * d + j];
  if (threadIdx.x == 0) {
    slot_k[slot] = m[1];
    slot_ef[slot] = m[2];
    cap[slot] = m[3];
    state_off[slot] = (int64_t)(((uint64_t)(uint32_t)m[5] << 32) | (uint32_t)m[4]);
    QState st;
    memset(&st, 0, sizeof(st));
    st.li = kSlotNew;
    states[slot] = st;
    if (root_keys) slot_root[slot] = root_keys[r];
  }
}

template <int KIND, int LPN, int CPL, bool FULL, int NB>
static void launch_serve_one(const SearchArgs& a, const ServeArgs& sv, int wpb, hipStream_t st) {
  const size_t per_wave = search_lds_per_wave(a.ef_cap, a.vis_bits, a.vis_bytes, NB);
  const unsigned blocks = (unsigned)((sv.n_active + wpb - 1) / wpb);
  auto kern = serve_kernel<KIND, LPN, CPL, FULL, NB>();
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * wpb), per_wave * wpb, st, a, sv,
                     (int)per_wave, wpb);
}

template <int KIND, int LPN, int CPL, bool FULL, bool EXACT, int NB>
__device__ __forceinline__ void search_kernel_body(const SearchArgs& a, int per_wave_bytes,
                                                   int waves_per_block, int persistent) {
  extern __shared__ __align__(16) char smem[];
  const int wave = uni(threadIdx.x >> 6);
  WaveLds s = carve<NB>(smem + (size_t)wave * per_wave_bytes, a.ef_cap);
  // one copy of the search for both forms: the one-shot form makes one pass
  // of the loop.  The arguments are read afresh in each pass (the pointer is
  // opaque), or the compiler holds them all in registers across the passes.
  for (;;) {
    int64_t qi = (int64_t)blockIdx.x * waves_per_block + wave;
    auto* kp = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(kp));
    const SearchArgs& aa = *reinterpret_cast<const SearchArgs*>((const char*)kp);
    if (persistent) {
      uint32_t w = 0;
      if (lane_id() == 0) w = atomicAdd(aa.work_counter, 1u);
      qi = (int64_t)(uint32_t)uni((int32_t)w);
    }
    if (qi >= aa.nq) break;
    search_one<KIND, LPN, CPL, FULL, EXACT, NB>(aa, qi, s);
    if (!persistent) break;
  }
}

template <int KIND, int LPN, int CPL, bool FULL, int NB, bool EXACT = false>
__global__ __launch_bounds__(512) void k_search(SearchArgs a, int per_wave_bytes,
                                                int waves_per_block, int persistent) {
  search_kernel_body<KIND, LPN, CPL, FULL, EXACT, NB>(a, per_wave_bytes, waves_per_block, persistent);
}

// The same kernel held to 80 registers (see six_waves).
template <int KIND, int LPN, int CPL, bool FULL, int NB>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(6))) void k_search6(
    SearchArgs a, int per_wave_bytes, int waves_per_block, int persistent) {
  search_kernel_body<KIND, LPN, CPL, FULL, false, NB>(a, per_wave_bytes, waves_per_block, persistent);
}

template <int KIND, int LPN, int CPL, bool FULL, int NB>
static auto search_kernel(bool exact) {
  // the exact visited set (an analysis form) runs the general-width kernel
  if constexpr (NB == 0) {
    if (exact) return &k_search<KIND, LPN, CPL, false, 0, true>;
  }
  if constexpr (six_waves<KIND, CPL, NB>())
    return &k_search6<KIND, LPN, CPL, FULL, NB>;
  else
    return &k_search<KIND, LPN, CPL, FULL, NB>;
}

static __global__ void k_reset_counter(uint32_t* c) { *c = 0u; }

template <int KIND, int LPN, int CPL, bool FULL, int NB>
static void launch_one(const SearchArgs& a, const LaunchShape& sh, hipStream_t st) {
  const bool exact = a.vis_exact != nullptr;
  const size_t per_wave = search_lds_per_wave(a.ef_cap, a.vis_bits, a.vis_bytes, NB);
  const int wpb = sh.waves_per_block;
  const size_t lds = per_wave * wpb;
  auto kern = search_kernel<KIND, LPN, CPL, FULL, NB>(exact);
  if (sh.persistent) {
    int blocks = sh.blocks;
    if (blocks <= 0) {
      int dev = 0, cus = 0, per_cu = 0;
      (void)hipGetDevice(&dev);
      (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
      (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &per_cu, reinterpret_cast<const void*>(kern), 64 * wpb, lds);
      blocks = max(1, cus * max(per_cu, 1));
    }
    hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, st, a.work_counter);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * wpb), lds, st, a, (int)per_wave, wpb, 1);
  } else {
    const int64_t blocks = (a.nq + wpb - 1) / wpb;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(64 * wpb), lds, st, a, (int)per_wave,
                       wpb, 0);
  }
}

// Waves of the search kernel of this shape that a CU's registers hold (asked
// of the runtime once per kernel).
template <int KIND, int LPN, int CPL, bool FULL, int NB>
static int resident_waves() {
  static std::atomic<int> waves{0};
  int w = waves.load(std::memory_order_relaxed);
  if (w == 0) {
    auto kern = search_kernel<KIND, LPN, CPL, FULL, NB>(false);
    HENN_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &w, reinterpret_cast<const void*>(kern), 64, 0));
    w = std::max(w, 4);
    waves.store(w, std::memory_order_relaxed);
  }
  return w;
}

#define HENN_SEARCH_COMBOS(X) \
  X(1, 1) X(2, 1) X(4, 1) X(2, 2) X(4, 2) X(8, 1) X(2, 4) X(4, 4) X(8, 2) X(16, 1) X(8, 4) \
  X(16, 2) X(4, 8) X(16, 4) X(16, 8)

template <int KIND, int NB>
bool search_dispatch(const SearchArgs& a, const LaunchShape& sh, hipStream_t st) {
#define HENN_TRY(LPN, CPL)                              \
  if (sh.lanes_per_vec == LPN && sh.chunks_per_lane == CPL) { \
    if (a.nchunks == LPN * CPL)                         \
      launch_one<KIND, LPN, CPL, true, NB>(a, sh, st);  \
    else                                                \
      launch_one<KIND, LPN, CPL, false, NB>(a, sh, st); \
    return true;                                        \
  }
  HENN_SEARCH_COMBOS(HENN_TRY)
#undef HENN_TRY
  return false;
}

template <int KIND, int NB>
int waves_dispatch(int nchunks, int lpn, int cpl) {
#define HENN_TRY(LPN, CPL)                                               \
  if (lpn == LPN && cpl == CPL)                                          \
    return nchunks == LPN * CPL ? resident_waves<KIND, LPN, CPL, true, NB>() \
                                : resident_waves<KIND, LPN, CPL, false, NB>();
  HENN_SEARCH_COMBOS(HENN_TRY)
#undef HENN_TRY
  return 4;
}

template <int KIND, int NB>
bool serve_dispatch(const SearchArgs& a, const ServeArgs& sv, const LaunchShape& sh,
                    hipStream_t st) {
#define HENN_TRY(LPN, CPL)                                        \
  if (sh.lanes_per_vec == LPN && sh.chunks_per_lane == CPL) {     \
    if (a.nchunks == LPN * CPL)                                   \
      launch_serve_one<KIND, LPN, CPL, true, NB>(a, sv, sh.waves_per_block, st);  \
    else                                                          \
      launch_serve_one<KIND, LPN, CPL, false, NB>(a, sv, sh.waves_per_block, st); \
    return true;                                                  \
  }
  HENN_SEARCH_COMBOS(HENN_TRY)
#undef HENN_TRY
  return false;
}

// One translation unit per (rows, list) pair instantiates its kernels; the
// common part only refers to them.
#define HENN_INST(PART, KIND, NB, EXT)                                                       \
  EXT template bool search_dispatch<KIND, NB>(const SearchArgs&, const LaunchShape&,         \
                                              hipStream_t);                                  \
  EXT template int waves_dispatch<KIND, NB>(int, int, int);                                  \
  EXT template bool serve_dispatch<KIND, NB>(const SearchArgs&, const ServeArgs&,            \
                                             const LaunchShape&, hipStream_t);
#if HENN_PART < 0 || HENN_PART == 1
HENN_INST(1, kF32, 0, )
#endif
#if HENN_PART < 0 || HENN_PART == 2
HENN_INST(2, kF32, 2, )
#endif
#if HENN_PART < 0 || HENN_PART == 3
HENN_INST(3, kF32, 4, )
#endif
#if HENN_PART < 0 || HENN_PART == 4
HENN_INST(4, kBF16, 0, )
#endif
#if HENN_PART < 0 || HENN_PART == 5
HENN_INST(5, kBF16, 2, )
#endif
#if HENN_PART < 0 || HENN_PART == 6
HENN_INST(6, kBF16, 4, )
#endif
#if HENN_PART < 0 || HENN_PART == 7
HENN_INST(7, kFP8, 0, )
#endif
#if HENN_PART < 0 || HENN_PART == 8
HENN_INST(8, kFP8, 2, )
#endif
#if HENN_PART < 0 || HENN_PART == 9
HENN_INST(9, kFP8, 4, )
#endif

#if HENN_COMMON_PART
#if HENN_PART == 0
HENN_INST(1, kF32, 0, extern)
HENN_INST(2, kF32, 2, extern)
HENN_INST(3, kF32, 4, extern)
HENN_INST(4, kBF16, 0, extern)
HENN_INST(5, kBF16, 2, extern)
HENN_INST(6, kBF16, 4, extern)
HENN_INST(7, kFP8, 0, extern)
HENN_INST(8, kFP8, 2, extern)
HENN_INST(9, kFP8, 4, extern)
#endif

// The gather addresses a row by its 32-bit first-chunk index.
bool rows_addressable(const SearchArgs& a) {
  for (int i = 0; i < a.num_layers; ++i)
    if ((int64_t)a.layer[i].size * a.nchunks >= (1ll << 32)) return false;
  return true;
}

template <int KIND>
static bool launch_search_kind(const SearchArgs& a, const LaunchShape& s, hipStream_t st) {
  switch (s.list_blocks) {
    case 2: return search_dispatch<KIND, 2>(a, s, st);
    case 4: return search_dispatch<KIND, 4>(a, s, st);
    default: return search_dispatch<KIND, 0>(a, s, st);
  }
}

bool launch_search(int storage, const SearchArgs& a, const LaunchShape& s, hipStream_t st) {
  if (!rows_addressable(a)) return false;
  switch (storage) {
    case kF32: return launch_search_kind<kF32>(a, s, st);
    case kBF16: return launch_search_kind<kBF16>(a, s, st);
    case kFP8: return launch_search_kind<kFP8>(a, s, st);
    default: return false;
  }
}

template <int KIND>
static bool launch_serve_kind(const SearchArgs& a, const ServeArgs& sv, const LaunchShape& sh,
                              hipStream_t st) {
  switch (sh.list_blocks) {
    case 2: return serve_dispatch<KIND, 2>(a, sv, sh, st);
    case 4: return serve_dispatch<KIND, 4>(a, sv, sh, st);
    default: return serve_dispatch<KIND, 0>(a, sv, sh, st);
  }
}

bool launch_serve_step(int storage, const SearchArgs& a, const ServeArgs& sv,
                       const LaunchShape& sh, hipStream_t st) {
  if (sv.n_active <= 0) return true;
  if (!rows_addressable(a)) return false;
  switch (storage) {
    case kF32: return launch_serve_kind<kF32>(a, sv, sh, st);
    case kBF16: return launch_serve_kind<kBF16>(a, sv, sh, st);
    case kFP8: return launch_serve_kind<kFP8>(a, sv, sh, st);
    default: return false;
  }
}

void launch_serve_admit(const float* staged_q, const int32_t* meta, int n_new, int d,
                        float* slot_q, int32_t* slot_k, int32_t* slot_ef, int64_t* state_off,
                        int32_t* cap, QState* states, const uint64_t* root_keys,
                        uint64_t* slot_root, hipStream_t st) {
  if (n_new <= 0) return;
  hipLaunchKernelGGL(k_serve_admit, dim3(n_new), dim3(64), 0, st, staged_q, meta, n_new, d,
                     slot_q, slot_k, slot_ef, state_off, cap, states, root_keys, slot_root);
}

template <int KIND>
static bool launch_root_check_kind(const SearchArgs& a, const RootShortlist& sl, uint64_t* out,
                                   hipStream_t st) {
  int lpn = 0, cpl = 0;
  // two chunks a lane leave five waves a SIMD; with four the compiler takes
  // 184 registers and 10,000 queries on FP8 rows 18.2 us
  pick_row_lanes(a.nchunks, &lpn, &cpl);
  const dim3 grid((unsigned)((a.nq + 7) / 8));  // eight queries a block
#define HENN_TRY(L, C)                                                                       \
  if (lpn == L && cpl == C) {                                                                \
    hipLaunchKernelGGL((k_root_check<KIND, L, C>), grid, dim3(256), 0, st, a, sl, out);         \
    return true;                                                                             \
  }
  HENN_TRY(1, 1) HENN_TRY(2, 1) HENN_TRY(4, 1) HENN_TRY(2, 2) HENN_TRY(4, 2) HENN_TRY(8, 1)
  HENN_TRY(8, 2)
#undef HENN_TRY
  return false;
}

bool launch_root_check(int storage, const SearchArgs& a, const RootShortlist& sl, uint64_t* out,
                       hipStream_t st) {
  if (a.nq <= 0) return true;
  switch (storage) {
    case kF32: return launch_root_check_kind<kF32>(a, sl, out, st);
    case kBF16: return launch_root_check_kind<kBF16>(a, sl, out, st);
    case kFP8: return launch_root_check_kind<kFP8>(a, sl, out, st);
    default: return false;
  }
}

// instantiated (LPN, CPL) pairs
static const int kCombos[][2] = {{1, 1}, {2, 1},  {4, 1},  {2, 2}, {4, 2},  {8, 1},
                                 {2, 4}, {4, 4},  {8, 2},  {16, 1}, {8, 4},  {16, 2},
                                 {4, 8}, {16, 4}, {16, 8}};

// The pair with LPN * CPL = P: the requested lanes, else the fewest lanes
// with at most max_cpl chunks per lane (or the most lanes there are).
static void pick_lanes_at_most(int nchunks, int requested_lpn, int max_cpl, int* lpn, int* cpl) {
  const int P = next_pow2(nchunks);
  int best_l = 0, best_c = 0;
  for (auto& c : kCombos) {
    if (c[0] * c[1] != P) continue;
    if (requested_lpn > 0) {
      if (c[0] == requested_lpn) { best_l = c[0]; best_c = c[1]; }
      continue;
    }
    if (best_l == 0 || (c[1] <= max_cpl ? best_c > max_cpl || c[0] < best_l : c[1] < best_c)) {
      best_l = c[0];
      best_c = c[1];
    }
  }
  *lpn = best_l;
  *cpl = best_c;
}

void pick_lanes(int nchunks, int requested_lpn, int* lpn, int* cpl) {
  pick_lanes_at_most(nchunks, requested_lpn, 4, lpn, cpl);
}

void pick_row_lanes(int nchunks, int* lpn, int* cpl) {
  pick_lanes_at_most(nchunks, 0, 2, lpn, cpl);
}

void pick_search_lanes(int storage, int nchunks, int64_t nq, int cus, int requested_lpn, int* lpn,
                       int* cpl) {
  const int64_t simds = 4ll * cus;
  const bool many = storage == kFP8 ? nq > 3 * simds : nq > 8 * simds;
  pick_lanes_at_most(nchunks, requested_lpn, storage == kF32 || many ? 2 : 4, lpn, cpl);
}

template <int KIND>
static int search_waves_kind(int blocks, int nchunks, int lpn, int cpl) {
  switch (blocks) {
    case 2: return waves_dispatch<KIND, 2>(nchunks, lpn, cpl);
    case 4: return waves_dispatch<KIND, 4>(nchunks, lpn, cpl);
    default: return waves_dispatch<KIND, 0>(nchunks, lpn, cpl);
  }
}

int search_waves(int storage, int blocks, int nchunks, int lpn, int cpl) {
  switch (storage) {
    case kF32: return search_waves_kind<kF32>(blocks, nchunks, lpn, cpl);
    case kBF16: return search_waves_kind<kBF16>(blocks, nchunks, lpn, cpl);
    default: return search_waves_kind<kFP8>(blocks, nchunks, lpn, cpl);
  }
}

int pick_vis_bits(int register_waves, int blocks, int ef_need, int deg, int64_t n, int64_t nq,
                  int cus, int base) {
  // resident waves of a CU: what the kernel's registers leave room for, or
  // what the batch gives it
  const int ef_cap = next_pow2(ef_need);
  const int64_t waves = std::min<int64_t>(register_waves, (nq + cus - 1) / cus);
  int bits = base;
  for (int b = base + 1; b <= 14 && (1ll << b) <= 8ll * ef_need * deg; ++b) {
    if ((int64_t)search_lds_per_wave(ef_cap, b, vis_tag_bytes(n, b), blocks) * waves > 160 * 1024) break;
    bits = b;
  }
  return bits;
}
#endif  // HENN_COMMON_PART

}  // namespace henn
