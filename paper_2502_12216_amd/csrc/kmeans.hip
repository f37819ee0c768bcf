// Prefill K-means clustering of the keys (Sec. 4.2) for gfx950.
//
// One problem per (sequence b, KV head g): n_b keys, C_b clusters, started
// from the keys of the sampled tokens init_idx.  The nearest centroid of a key
// is the largest k.c - ||c||^2 / 2 (ties to the smaller id), contracted on MFMA
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation).  A score depends only on the
// key's and the centroid's bits, so an iteration need not look at a pair again
// whose centroid did not change: every key keeps its best score and a bound
// that no other centroid's score exceeds, and the results are exactly those of
// measuring every pair.  Each iteration:
//   km_assign   full passes (from sampled keys the first two iterations, from a
//               previous clustering the first): every key against every
//               centroid.  Later: every key against the centroids that the
//               last update changed; keys whose own centroid changed and whose
//               best new score does not clear their bound, or is shared by two
//               of them, go to a list, and the listed keys are measured against
//               every centroid.
//   km_merge    takes the listed keys' results in and ends a problem whose
//               assignment step changed nothing.
//   km_update   of the clusters that gained or lost a key: member lists, each
//               member's rank in token order, and the means, summed in that order
//               (fixed, so results are deterministic), rounded to bf16; an empty
//               cluster keeps its centroid.  Centroids that changed are copied
//               to the next iteration's list.
// After the last iteration km_layout scans the clusters' sizes, and km_permute puts
// every token and its K/V rows at its cluster's start plus its rank.
//
// Measured on keys of a 4096-component mixture (65536 x 8 heads, 10
// iterations): the changed centroids are 97, 56, 17, 3, 0.8 ... % of all from the
// second iteration on, the listed keys 3.4, 1.4, 0.2 ... %; on unstructured
// normal keys 77, 42, 35, 31, 27, 22, 18, 13, 9 % and at most 2 %.  Times of 2 / 3 / 10
// iterations, 65536 x 8 keys, against measuring every pair each time (ms): mixture
// 1.21 / 1.58 / 2.17 (1.25 / 1.79 / 5.01), normal keys 1.28 / 1.65 / 3.06 (1.36 / 1.89 / 5.65),
// keys that hardly settle (integers in 16 dimensions) 1.10 / 1.67 / 3.81 (1.13 / 1.60 / 4.92):
// there the second pass, which keeps the bounds, and a third over 97% of the
// centroids cost a call of three iterations 4%.  Deciding by the share of
// changed centroids between that and a full pass gains nothing (0.52 against 0.53 ms).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "common.hpp"
#include "kmeans.hpp"

namespace tactic {

constexpr int kAsgTok = 256;        // tokens per assignment workgroup (4 waves x 64)
constexpr int kAsgCen = 96;         // centroids staged in LDS per step
constexpr int kListCen = 2 * kAsgCen;  // centroids per work item of the listed keys
constexpr int kSliceMax = 2048;     // clusters per slice of the update kernel
constexpr int kSliceCap = 4096;     // keys per slice that it collects in LDS
constexpr int kRankMax = 256;       // members that one wave ranks, of a slice with lists in memory
constexpr int kOrdWords = 512;      // words of LDS per wave for sorting members
constexpr int kBitTokens = 16 * kOrdWords * 32;  // tokens per bitmap window of a workgroup
constexpr int kSmall = 64;          // members of a cluster that one wave takes in one go
constexpr int kStateInts = 64;      // counters of a problem, each in a 64-byte line of its own

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

struct KmArgs {
  const uint16_t* K;
  const uint16_t* V;
  const int64_t* kv_indptr;
  const int64_t* seq_len;     // [B] or null (see tactic_kv_shape)
  const int64_t* cl_indptr;
  int B, Hkv, Cm, iter;
  int64_t total, Ct;
  const int32_t* init_idx;
  const uint16_t* prev_centroids;  // warm start, or null
  const int64_t* prev_cl_indptr;
  uint16_t* centroids;
  float* cnorm;
  int32_t* assign;
  int32_t* offsets;
  int32_t* perm;
  float* best;        // [Hkv][total]: score of the key's centroid
  float* bound;       // [Hkv][total]: no other centroid of the key scores higher
  int32_t* members;   // [Hkv][total]: member lists in arrival order
  int32_t* rank;      // [Hkv][total]: the key's place among its cluster's members in token order
  int32_t* dirty;     // [Hkv][Ct]: 1: the cluster gained or lost a key
  int32_t* moved;     // [Hkv][Ct]: 1: the last update changed the centroid
  uint16_t* d_rows;   // [Hkv][Ct][128]: the changed centroids, in no fixed order,
  float* d_norm;      // their norms
  int32_t* d_id;      // and ids
  int32_t* l_tok;     // [Hkv][total]: the listed keys
  uint64_t* l_key;    // [Hkv][total]: their best (score, id) as an ordered key, 0: none
  uint32_t* l_second; // [Hkv][total]: the second best score, as an ordered key, 0: none
  int32_t* state;     // [BG][kStateInts], see below
  uint16_t* K_sorted;
  uint16_t* V_sorted;
};

// a problem's counters
__device__ __forceinline__ int32_t* n_changed(const KmArgs& a, int p) { return a.state + (int64_t)p * kStateInts; }  // keys that changed cluster
__device__ __forceinline__ int32_t* n_moved(const KmArgs& a, int p) { return n_changed(a, p) + 16; }    // entries of d_rows
__device__ __forceinline__ int32_t* n_listed(const KmArgs& a, int p) { return n_changed(a, p) + 32; }   // entries of l_tok
__device__ __forceinline__ int32_t* done_flag(const KmArgs& a, int p) { return n_changed(a, p) + 48; }

struct Problem {
  int b, g, n, C;
  int64_t tok_base, cl_base, off_base;
};

__device__ __forceinline__ Problem problem(const KmArgs& a, int p) {
  Problem q;
  q.b = p / a.Hkv;
  q.g = p % a.Hkv;
  const int64_t s0 = a.kv_indptr[q.b], c0 = a.cl_indptr[q.b];
  q.n = (int)seq_tokens(a.kv_indptr, a.seq_len, q.b);
  q.C = min((int)(a.cl_indptr[q.b + 1] - c0), a.Cm);
  q.tok_base = (int64_t)q.g * a.total + s0;
  q.cl_base = (int64_t)q.g * a.Ct + c0;
  q.off_base = (int64_t)q.g * (a.Ct + a.B) + c0 + q.b;
  return q;
}

// A slice of a problem's clusters: those whose bit-reversed id lies in [lo, lo + nr),
// local index j standing for reversed id lo + j (at most about half of them are
// ids past the last cluster).  Of equal keys the smallest id takes all: 81
// distinct keys in 65536, 4096 clusters, had 64 of their clusters in the first 128 ids,
// and one workgroup 52000 keys to gather; bit reversal spreads any run of ids
// evenly, for one instruction per key.
struct Slice {
  int lo, nr, shift, C;
  __device__ __forceinline__ int id(int j) const { return (int)__brev((uint32_t)(lo + j) << shift); }  // (>= C: none)
  // place of cluster c on the scale of the reversed ids from the slice's start (c < 0: in no slice)
  __device__ __forceinline__ uint32_t place(int c) const {
    return c < 0 ? 0xffffffffu : __brev((uint32_t)c) - ((uint32_t)lo << shift);
  }
  // places below are in the slice (a place's low bits are 0: one less keeps a slice of all ids in 32 bits)
  __device__ __forceinline__ uint32_t end() const { return ((uint32_t)nr << shift) - 1u; }
  __device__ __forceinline__ int local(uint32_t place) const { return (int)(place >> shift); }
};

// slice s of at most `per` clusters on average: nr <= 2 per (2^bits < 2 C), 0 past the last slice
__device__ __forceinline__ Slice make_slice(int C, int per, int s) {
  Slice x;
  const int ns = (C + per - 1) / per, bits = C > 2 ? 32 - __clz(C - 1) : 1;
  x.C = C;
  x.shift = 32 - bits;
  x.lo = s < ns ? (int)(((int64_t)s << bits) / ns) : 0;
  x.nr = s < ns ? (int)(((int64_t)(s + 1) << bits) / ns) - x.lo : 0;
  return x;
}

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// ---------------------------------------------------------------------------
// init: c0 = K[init_idx] (or the previous clustering's centroid j for a warm
// start), ||c0||^2, per-problem flags.  grid (ceil(Cm/4), BG)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void km_init_kernel(KmArgs a) {
  const int p = blockIdx.y;
  const Problem q = problem(a, p);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *n_changed(a, p) = 0;
    *n_moved(a, p) = 0;
    *n_listed(a, p) = 0;
    *done_flag(a, p) = 0;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sl = lane & 15, grp = lane >> 4;
  const int j = blockIdx.x * 4 + wave;
  if (j >= q.C || grp != 0) return;
  if (sl == 0) a.dirty[q.cl_base + j] = 0;
  if (q.n == 0) return;
  uint4 v;
  const int64_t pc0 = a.prev_centroids ? a.prev_cl_indptr[q.b] : 0;
  const int64_t pc1 = a.prev_centroids ? a.prev_cl_indptr[q.b + 1] : 0;
  if (j < pc1 - pc0) {
    // warm start: the previous clustering's centroid j of this (b, g)
    const int64_t prev_total = a.prev_cl_indptr[a.B];
    v = *reinterpret_cast<const uint4*>(a.prev_centroids + ((int64_t)q.g * prev_total + pc0 + j) * kHeadDim + sl * 8);
  } else {
    const int t = min(max(a.init_idx[q.cl_base + j], 0), q.n - 1);
    v = *reinterpret_cast<const uint4*>(a.K + (q.tok_base + t) * kHeadDim + sl * 8);
  }
  *reinterpret_cast<uint4*>(a.centroids + (q.cl_base + j) * kHeadDim + sl * 8) = v;
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x = bf16lo(w[e]), y = bf16hi(w[e]);
    s = fmaf(x, x, s);
    s = fmaf(y, y, s);
  }
  s = sum16(s);
  if (sl == 0) a.cnorm[q.cl_base + j] = s;
}

// ---------------------------------------------------------------------------
// assignment: 256 threads, 256 keys per workgroup.  A wave owns 64 keys
// (two 32-key MFMA B operands held in registers for the whole pass);
// centroids stream through LDS 96 at a time as the A operand, each tile
// loaded from memory straight into the other of two LDS buffers while the
// one before it is contracted (one barrier per tile).  The nearest
// centroid maximises s = k.c - ||c||^2 / 2; the accumulators of a block start
// at the fp32 -||c||^2 / 2 of their centroid row, so the contraction ends on
// finished scores and the epilogue is the maximum over each lane's 16
// scores of a block (by groups of four), and the search for the row that holds
// it, and for the second largest of the 16, only when some lane of the wave
// improved on its best (strict, so the smaller row wins a tie).  kTrack: also
// the second best score over all rows seen, for the keys' bounds.
//
// kMode 0: every key against every centroid.  From sampled keys almost every
//   centroid moves in the first update (97% on a mixture), so the second
//   iteration measures every pair as well, and only that pass tracks the second
//   best (131072 x 4 sequences x 8 heads, 8192 clusters: first iteration 8.4
//   ms, 9.2 with it; second 8.3 ms, 8.4 as kMode 1 and 2 behind a tracked first;
//   65536 x 8, two iterations 1.37 -> 1.26 ms, ten 2.35 -> 2.26).  From a
//   previous clustering the first pass tracks it and pruning starts at once
//   (two iterations 1.03 ms); a call that ends with the full passes does not track.
// kMode 1: every key against the rows of d_rows.  The search starts from a
//   score that a new best must exceed: the key's bound where its own centroid
//   changed (the unchanged ones do not exceed it), else the value just below
//   its best score (so that an equal score of a smaller id is seen).  A key
//   that finds nothing above its bound, or two equal best rows, is listed.
// kMode 2: the listed keys against every centroid, in work items of 256 keys x
//   kListCen centroids (few keys are listed: whole passes over the centroids
//   would leave most of the device idle), merged by atomic maxima, whose
//   result does not depend on the order.
// grid (ceil(nmax / 256), BG); kMode 2: (work items in flight, BG)
//
// Bound by MFMA and, at late iterations, by reading the keys: 65536 keys x 8
// heads, 4096 centroids, 10 iterations: 5.2 ms when every iteration measures
// every pair.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t score_key(float s) {  // ascending with s, never 0 for a number
  const uint32_t u = __float_as_uint(s + 0.0f);           // -0 -> +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_to_score(uint32_t k) {  // 0 (no score): -inf
  return k == 0 ? -INFINITY : __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
// A float below s with no value between (-inf stays).  Below 0 it is the largest
// negative one, not -0, which compares equal: the key before that of 0 stands for
// no value (score_key reads -0 as 0).
__device__ __forceinline__ float just_below(float s) {
  const uint32_t k = score_key(s);
  return s == -INFINITY ? s : key_to_score(k - (s == 0.0f ? 2u : 1u));
}
__device__ __forceinline__ float second_of4(float a, float b, float c, float d) {
  const float h0 = fmaxf(a, b), l0 = fminf(a, b), h1 = fmaxf(c, d), l1 = fminf(c, d);
  return fmaxf(fmaxf(fminf(h0, h1), l0), l1);
}

// three waves per SIMD: the B operands and accumulators live in VGPRs
template <int kMode, bool kTrack = true>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void km_assign_kernel(KmArgs a) {
  static_assert(kTrack || kMode == 0, "only full passes go without bounds");
  // two centroid tiles (the next one loads while this one is contracted):
  // rows of 16 chunks of 16 bytes, logical chunk c of row r stored at chunk
  // c ^ (r & 15), so that the 32 rows an A-operand read touches at one
  // logical chunk fall in distinct LDS bank groups
  __shared__ __align__(16) uint16_t s_c[2][kAsgCen * kHeadDim];
  __shared__ __align__(16) float s_nh[2][kAsgCen];  // -||c||^2 / 2 (-inf past the last centroid)
  __shared__ int s_n[3];  // kMode 1: keys listed and changed by the workgroup, its first list slot
  const int p = blockIdx.y;
  if (*done_flag(a, p)) return;
  const int nd = kMode == 1 ? *n_moved(a, p) : 0, nl = kMode == 2 ? *n_listed(a, p) : 0;
  if (kMode == 1 && nd == 0) return;  // no centroid changed: no key does
  if (kMode == 0 && a.iter > 1 && *n_moved(a, p) == 0) return;
  if (kMode == 2 && nl == 0) return;
  const Problem q = problem(a, p);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5, col = lane & 31;
  int lplace[2] = {-1, -1};  // kMode 1: the key's place among the workgroup's listed ones
  const int slices = kMode == 2 ? (q.C + kListCen - 1) / kListCen : 1;
  const uint16_t* cbase = (kMode == 1 ? a.d_rows : a.centroids) + q.cl_base * kHeadDim;
  const float* cnorm = (kMode == 1 ? a.d_norm : a.cnorm) + q.cl_base;
  if (kMode < 2 && tid < 3) s_n[tid] = 0;  // (the tile loop's barriers order it before its use)
  for (int64_t item = blockIdx.x;; item += gridDim.x) {  // kMode 0, 1: one item
    const int64_t first = (kMode == 2 ? item / slices : item) * kAsgTok;
    const int c_beg = kMode == 2 ? (int)(item % slices) * kListCen : 0;
    const int c_end = kMode == 2 ? min(c_beg + kListCen, q.C) : (kMode == 1 ? nd : q.C);
    const int m = kMode == 2 ? nl : q.n;
    if (first >= m) break;
    const int i0 = (int)first;

    bf16x8 bt[2][8];
    int tokv[2];  // kMode 2: the key's token
    float best_v[2], sec_v[2] = {-INFINITY, -INFINITY};
    int best_j[2] = {0x7fffffff, 0x7fffffff};
#pragma unroll
    for (int bb = 0; bb < 2; ++bb) {
      const int i = i0 + wave * 64 + bb * 32 + col, ic = min(i, m - 1);
      const int tok = kMode == 2 ? min(max(a.l_tok[q.tok_base + ic], 0), q.n - 1) : ic;
      tokv[bb] = tok;
      const uint16_t* src = a.K + (q.tok_base + tok) * kHeadDim + 64 * half;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (i < m) v = *reinterpret_cast<const uint4*>(src + 8 * s);
        bt[bb][s] = __builtin_bit_cast(bf16x8, v);
      }
      best_v[bb] = -INFINITY;
      if (kMode == 1) {
        const int old = a.assign[q.tok_base + tok];
        best_v[bb] = a.moved[q.cl_base + old] ? a.bound[q.tok_base + tok] : just_below(a.best[q.tok_base + tok]);
      }
    }
    // a tile goes from memory straight to LDS (no registers): each wave moves
    // blocks of 64 chunks; lane L of block blk fills stored chunk
    // blk * 64 + L, i.e. row (blk * 64 + L) / 16, with the row's logical chunk
    // that the swizzle puts there; rows past the end load a valid row (their
    // scores are -inf through the norm term)
    auto stage = [&](int c0, int buf) {
#pragma unroll
      for (int i = 0; i < kAsgCen * 16 / 256; ++i) {
        const int blk = wave * (kAsgCen * 16 / 256) + i, qq = blk * 64 + lane, row = qq >> 4;
        const int grow = min(c0 + row, c_end - 1);
        __builtin_amdgcn_global_load_lds(cbase + (int64_t)grow * kHeadDim + ((qq & 15) ^ (row & 15)) * 8,
                                         (__attribute__((address_space(3))) void*)(s_c[buf] + blk * 512), 16, 0, 0);
      }
    };
    float pfn = (tid < kAsgCen && c_beg + tid < c_end) ? cnorm[c_beg + tid] : 0.f;
    if (kMode == 2) __syncthreads();  // the item before is done with the buffers
    if (c_beg < c_end) stage(c_beg, 0);
    int buf = 0;
    for (int c0 = c_beg; c0 < c_end; c0 += kAsgCen, buf ^= 1) {
      if (tid < kAsgCen) s_nh[buf][tid] = c0 + tid < c_end ? -0.5f * pfn : -INFINITY;
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's tile loads have reached LDS
      __syncthreads();  // every wave's part of the tile and the norms in place; the other buffer free
      if (c0 + kAsgCen < c_end) {
        stage(c0 + kAsgCen, buf ^ 1);
        if (tid < kAsgCen && c0 + kAsgCen + tid < c_end) pfn = cnorm[c0 + kAsgCen + tid];
      }
      const int nblk = min(kAsgCen / 32, (c_end - c0 + 31) / 32);
      for (int cb = 0; cb < nblk; ++cb) {
        // accumulator i of a lane is row 8 (i / 4) + 4 half + i % 4 of the block
        f32x16 acc[2];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float4 x = *reinterpret_cast<const float4*>(s_nh[buf] + cb * 32 + 8 * k + 4 * half);
          acc[0][4 * k] = acc[1][4 * k] = x.x;
          acc[0][4 * k + 1] = acc[1][4 * k + 1] = x.y;
          acc[0][4 * k + 2] = acc[1][4 * k + 2] = x.z;
          acc[0][4 * k + 3] = acc[1][4 * k + 3] = x.w;
        }
        const uint16_t* arow = s_c[buf] + (cb * 32 + col) * kHeadDim;  // row cb * 32 + col: swizzle col & 15
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const bf16x8 av = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(arow + (((8 * half + s) ^ (col & 15)) * 8)));
          acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bt[0][s], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bt[1][s], acc[1], 0, 0, 0);
        }
#pragma unroll
        for (int bb = 0; bb < 2; ++bb) {
          const f32x16 v = acc[bb];
          float g[4];  // maxima of the rows' groups of four
#pragma unroll
          for (int k = 0; k < 4; ++k) g[k] = fmaxf(fmaxf(fmaxf(v[4 * k], v[4 * k + 1]), v[4 * k + 2]), v[4 * k + 3]);
          const float mx = fmaxf(fmaxf(fmaxf(g[0], g[1]), g[2]), g[3]);
          const bool imp = mx > best_v[bb];
          if (__any(imp)) {
            // the first group that holds mx, its first row that does, and the
            // second largest of the 16: the second group maximum or the
            // group's second
            const bool e0 = g[0] == mx, e1 = g[1] == mx, e2 = g[2] == mx;
            float x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = e0 ? v[j] : (e1 ? v[4 + j] : (e2 ? v[8 + j] : v[12 + j]));
            int r = e0 ? 0 : (e1 ? 8 : (e2 ? 16 : 24));
            r += x[0] == mx ? 0 : (x[1] == mx ? 1 : (x[2] == mx ? 2 : 3));
            if (kTrack) {
              const float s2 = fmaxf(second_of4(g[0], g[1], g[2], g[3]), second_of4(x[0], x[1], x[2], x[3]));
              // not improved: the block's maximum is a candidate for the second
              sec_v[bb] = imp ? fmaxf(best_v[bb], s2) : fmaxf(sec_v[bb], mx);
            }
            best_v[bb] = imp ? mx : best_v[bb];
            best_j[bb] = imp ? c0 + cb * 32 + 4 * half + r : best_j[bb];
          } else if (kTrack) {
            sec_v[bb] = fmaxf(sec_v[bb], mx);
          }
        }
      }
    }
    if (kMode == 0) __syncthreads();  // (s_n is cleared where no tile was loaded, too)
#pragma unroll
    for (int bb = 0; bb < 2; ++bb) {
      const float ov = __shfl_xor(best_v[bb], 32, 64), os = __shfl_xor(sec_v[bb], 32, 64);
      const int oj = __shfl_xor(best_j[bb], 32, 64);
      float sec = fmaxf(sec_v[bb], os);
      // (two halves that found nothing hold their start value, not a score)
      if (best_j[bb] != 0x7fffffff || oj != 0x7fffffff) sec = fmaxf(sec, fminf(ov, best_v[bb]));
      if (ov > best_v[bb] || (ov == best_v[bb] && oj < best_j[bb])) {
        best_v[bb] = ov;
        best_j[bb] = oj;
      }
      const int i = i0 + wave * 64 + bb * 32 + col;
      const bool own = half == 0 && i < m;
      const int64_t at = q.tok_base + (kMode == 2 ? tokv[bb] : i);
      if (kMode == 0) {
        bool changed = false;
        if (own) {
          const int jn = min(max(best_j[bb], 0), q.C - 1);
          const int old = a.iter > 1 ? a.assign[at] : jn;
          changed = jn != old;
          if (changed) {
            a.dirty[q.cl_base + old] = 1;
            a.dirty[q.cl_base + jn] = 1;
          }
          if (changed || a.iter == 1) a.assign[at] = jn;
          if (kTrack) {
            a.best[at] = best_v[bb];
            a.bound[at] = sec;
          }
        }
        const uint64_t cm = __ballot(changed);
        if (cm && lane == 0) atomicAdd(&s_n[1], (int)__popcll(cm));
      }
      if (kMode == 1) {
        bool listed = false, changed = false;
        if (own) {
          const int old = a.assign[at];
          const bool found = best_j[bb] != 0x7fffffff;
          const float v = best_v[bb];
          int jn = old;
          float nb, nu = sec;
          if (a.moved[q.cl_base + old]) {
            // (sec holds the old bound: it started the search)
            listed = !found || sec == v;
            nb = v;
            if (!listed) jn = a.d_id[q.cl_base + best_j[bb]];
          } else {
            const float bo = a.best[at];
            nb = bo;
            nu = fmaxf(nu, a.bound[at]);
            if (found) {  // v >= bo
              listed = sec == v;
              const int id = a.d_id[q.cl_base + best_j[bb]];
              if (!listed && (v > bo || id < old)) jn = id;
              nb = v;
              nu = fmaxf(nu, bo);
            }
          }
          if (!listed) {
            a.best[at] = nb;
            a.bound[at] = nu;
            if (jn != old) {
              a.assign[at] = jn;
              a.dirty[q.cl_base + old] = 1;
              a.dirty[q.cl_base + jn] = 1;
              changed = true;
            }
          }
        }
        // one counter update per workgroup: single updates of one address
        // from every wave had doubled the time of a pass over few centroids
        const uint64_t lm = __ballot(listed), cm = __ballot(changed);
        int base = 0;
        if (lane == 0) {
          if (cm) atomicAdd(&s_n[1], (int)__popcll(cm));
          if (lm) base = atomicAdd(&s_n[0], (int)__popcll(lm));
        }
        base = __builtin_amdgcn_readfirstlane(base);  // (every lane is active here)
        if (listed) lplace[bb] = base + __popcll(lm & ((1ull << lane) - 1ull));
      }
      if (kMode == 2 && own && best_j[bb] != 0x7fffffff) {
        // the slot's best so far against this item's: the smaller one, and
        // this item's second, are candidates for the second
        const int64_t slot = q.tok_base + i;
        const uint64_t key = ((uint64_t)score_key(best_v[bb]) << 32) | (0xffffffffu - (uint32_t)best_j[bb]);
        const uint64_t was = atomicMax(reinterpret_cast<unsigned long long*>(a.l_key + slot), (unsigned long long)key);
        uint32_t s2 = (uint32_t)((was < key ? was : key) >> 32);
        if (sec != -INFINITY) s2 = max(s2, score_key(sec));
        if (s2) atomicMax(a.l_second + slot, s2);
      }
    }
    if (kMode != 2) break;
  }
  if (kMode == 0 && a.iter > 1) {
    __syncthreads();
    if (tid == 0 && s_n[1]) atomicAdd(n_changed(a, p), s_n[1]);
  }
  if (kMode == 1) {
    __syncthreads();
    if (tid == 0) {
      if (s_n[0]) s_n[2] = atomicAdd(n_listed(a, p), s_n[0]);
      if (s_n[1]) atomicAdd(n_changed(a, p), s_n[1]);
    }
    __syncthreads();
#pragma unroll
    for (int bb = 0; bb < 2; ++bb) {
      if (lplace[bb] < 0) continue;
      const int64_t slot = q.tok_base + s_n[2] + lplace[bb];
      a.l_tok[slot] = blockIdx.x * kAsgTok + wave * 64 + bb * 32 + col;
      a.l_key[slot] = 0;
      a.l_second[slot] = 0;
    }
  }
}

// ---------------------------------------------------------------------------
// the listed keys' results, the end of a problem.  grid BG, 1024 threads
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void km_merge_kernel(KmArgs a) {
  __shared__ int s_chg;
  const int p = blockIdx.x;
  if (*done_flag(a, p)) return;
  const Problem q = problem(a, p);
  const int tid = threadIdx.x;
  const int nl = *n_listed(a, p);
  if (tid == 0) s_chg = *n_changed(a, p);
  __syncthreads();
  int nchg = 0;
  for (int i = tid; i < nl; i += 1024) {
    const uint64_t key = a.l_key[q.tok_base + i];
    const uint32_t second = a.l_second[q.tok_base + i];
    const int64_t at = q.tok_base + min(max(a.l_tok[q.tok_base + i], 0), q.n - 1);
    const int old = a.assign[at];
    // no centroid scored a number: the last one, as in the first iteration
    const int jn = key ? (int)(0xffffffffu - (uint32_t)key) : q.C - 1;
    a.best[at] = key_to_score((uint32_t)(key >> 32));
    a.bound[at] = key_to_score(second);
    if (jn != old) {
      a.assign[at] = jn;
      a.dirty[q.cl_base + old] = 1;
      a.dirty[q.cl_base + jn] = 1;
      ++nchg;
    }
  }
  if (nchg) atomicAdd(&s_chg, nchg);
  __syncthreads();
  if (tid == 0) {
    *n_changed(a, p) = 0;
    *n_moved(a, p) = 0;  // km_update counts the next ones
    *n_listed(a, p) = 0;
    if (s_chg == 0) *done_flag(a, p) = 1;  // converged: nothing changed
  }
}

// One pass of a workgroup (1024 threads) over a problem's assignments: f(token,
// cluster) for every token, 16 loads in flight per thread.
template <typename F>
__device__ __forceinline__ void for_tokens(const int32_t* assign, int n, F f) {
  constexpr int kIn = 16;
  for (int64_t i0 = threadIdx.x; i0 < n; i0 += 1024 * kIn) {
    int c[kIn];
#pragma unroll
    for (int k = 0; k < kIn; ++k) c[k] = assign[min(i0 + 1024 * k, (int64_t)n - 1)];
#pragma unroll
    for (int k = 0; k < kIn; ++k)
      if (i0 + 1024 * k < n) f((int)(i0 + 1024 * k), c[k]);
  }
}

// Collects the tokens of a slice's clusters in LDS, in no fixed order, and returns
// how many there are (only the first kSliceCap are kept).  One pass over the
// assignments, 16 loads in flight per thread: a wave reserves places for all
// its hits of a step at once, and each thread walks the bits of its own hits
// (an LDS counter update per key, waited for, had taken 15 us per pass over
// 65536 keys, bound by instruction issue).  Ends with a barrier; *s_total is 0
// before.
__device__ __forceinline__ int collect_slice(const int32_t* assign, int n, const Slice& sc, int32_t* s_tok, int* s_total) {
  constexpr int kIn = 16;
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t end = sc.end();
  int c[kIn];  // (as loaded: what is computed here would wait here)
  auto load = [&](int64_t i0) {
#pragma unroll
    for (int k = 0; k < kIn; ++k) c[k] = assign[min(i0 + tid + 1024 * k, (int64_t)n - 1)];
  };
  if (n > 0) load(0);
  for (int64_t i0 = 0; i0 < n; i0 += 1024 * kIn) {
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < kIn; ++k) bits |= sc.place(c[k]) < end ? 1u << k : 0u;
    const int64_t left = (n - i0 - tid + 1023) / 1024;  // this thread's tokens from i0 on
    if (left < kIn) bits &= (1u << max(left, (int64_t)0)) - 1u;
    if (i0 + 1024 * kIn < n) load(i0 + 1024 * kIn);  // travels during the stores below
    const int mine = __popc(bits), incl = wave_incl_scan(mine);
    const int hits = __builtin_amdgcn_readlane(incl, 63);
    if (hits == 0) continue;
    int at = 0;
    if (lane == 0) at = atomicAdd(s_total, hits);
    int pos = __builtin_amdgcn_readfirstlane(at) + incl - mine;
    for (; bits; bits &= bits - 1, ++pos)
      if (pos < kSliceCap) s_tok[pos] = (int)i0 + tid + 1024 * (__ffs((int)bits) - 1);
  }
  __syncthreads();
  return *s_total;
}

// Exclusive scan in place of s[0..count) in LDS by 1024
// threads, and the sum over them of `mine`.  Ends with a barrier.
__device__ __forceinline__ int slice_scan(int32_t* s, int count, int mine, int* s_w) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (count + 1023) / 1024, b0 = min(count, tid * per), b1 = min(count, b0 + per);
  int loc = 0;
  for (int i = b0; i < b1; ++i) loc += s[i];
  const int incl = wave_incl_scan(loc);  // DPP, no LDS
  mine = wave_incl_scan(mine);
  if (lane == 63) {
    s_w[wave] = incl;
    s_w[16 + wave] = mine;
  }
  __syncthreads();
  int run = incl - loc, sum = 0;
  for (int w = 0; w < 16; ++w) {
    run += w < wave ? s_w[w] : 0;
    sum += s_w[16 + w];
  }
  for (int i = b0; i < b1; ++i) {
    const int t = s[i];
    s[i] = run;
    run += t;
  }
  __syncthreads();
  return sum;
}

// Values of y below x among lanes [0, km) of the wave (lanes from km on hold the
// largest value): lane reads at constant lanes, 16 at a time (a read at a
// lane number in a register took about 100 cycles).
__device__ __forceinline__ int count_below(int y, int x, int km) {
  int r = 0;
#pragma unroll
  for (int k0 = 0; k0 < 64; k0 += 16) {
    if (k0 < km) {
#pragma unroll
      for (int k = 0; k < 16; ++k) r += __builtin_amdgcn_readlane(y, k0 + k) < x ? 1 : 0;
    }
  }
  return r;
}

// One wave sorts a cluster's m <= 64 members by token into s_w; rank[token] = its place.
__device__ __forceinline__ void sort_small(const int32_t* list, int m, uint32_t* s_w, int32_t* rank, int lane) {
  const int x = lane < m ? list[lane] : 0x7fffffff;
  const int r = count_below(x, x, m);
  if (lane < m) {
    s_w[r] = (uint32_t)x;
    rank[x] = r;
  }
  __builtin_amdgcn_wave_barrier();
}

// The same for m <= kRankMax members, by counting in LDS.
__device__ __forceinline__ void sort_members(const int32_t* list, int m, uint32_t* s_w, int32_t* rank, int lane) {
  if (m <= kSmall) return sort_small(list, m, s_w, rank, lane);
  constexpr int kE = kRankMax / 64;
  int x[kE], r[kE];
#pragma unroll
  for (int e = 0; e < kE; ++e) {
    const int i = lane + 64 * e;
    x[e] = i < m ? list[i] : 0x7fffffff;
    r[e] = 0;
    s_w[kRankMax + i] = (uint32_t)x[e];
  }
  __builtin_amdgcn_wave_barrier();
  for (int i = 0; i < m; i += 4) {  // (entries past m compare as larger)
    const uint4 y = *reinterpret_cast<const uint4*>(s_w + kRankMax + i);
#pragma unroll
    for (int e = 0; e < kE; ++e)
      r[e] += ((int)y.x < x[e] ? 1 : 0) + ((int)y.y < x[e] ? 1 : 0) + ((int)y.z < x[e] ? 1 : 0) + ((int)y.w < x[e] ? 1 : 0);
  }
#pragma unroll
  for (int e = 0; e < kE; ++e)
    if (lane + 64 * e < m) {
      s_w[r[e]] = (uint32_t)x[e];
      rank[x[e]] = r[e];
    }
  __builtin_amdgcn_wave_barrier();
}

// The workgroup (1024 threads) sorts a cluster's m members (tokens below n) by a
// bitmap of the tokens in s_bits (kBitTokens / 32 words), window by window: into
// `out`, with their ranks.  Bound by the passes over the list and the words, a few
// memory round trips each.  Begins and ends with a barrier.
__device__ __forceinline__ void sort_by_bitmap(const int32_t* list, int m, int n, uint32_t* s_bits, int32_t* out, int32_t* rank,
                                               int* s_w) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int base = 0;
  for (int64_t w0 = 0; w0 < n; w0 += kBitTokens) {
    const int words = (int)((min((int64_t)kBitTokens, n - w0) + 31) / 32);
    const int kw = (words + 1023) / 1024, beg = min(words, tid * kw), end = min(words, beg + kw);  // this thread's words
    __syncthreads();  // the window before is read
    for (int k = tid; k < words; k += 1024) s_bits[k] = 0u;
    __syncthreads();
    constexpr int kIn = 8;
    for (int64_t i0 = tid; i0 < m; i0 += 1024 * kIn) {
      int64_t t[kIn];
#pragma unroll
      for (int k = 0; k < kIn; ++k) t[k] = list[min(i0 + 1024 * k, (int64_t)m - 1)] - w0;  // (the last one again past the end)
#pragma unroll
      for (int k = 0; k < kIn; ++k)
        if (t[k] >= 0 && t[k] < kBitTokens && t[k] + w0 < n) atomicOr(&s_bits[t[k] >> 5], 1u << (t[k] & 31));
    }
    __syncthreads();
    int cnt = 0;
    for (int k = beg; k < end; ++k) cnt += __popc(s_bits[k]);
    const int incl = wave_incl_scan(cnt);
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    int pos = base + incl - cnt, all = 0;
    for (int w = 0; w < 16; ++w) {
      pos += w < wave ? s_w[w] : 0;
      all += s_w[w];
    }
    for (int k = beg; k < end; ++k)
      for (uint32_t b = s_bits[k]; b; b &= b - 1, ++pos) {
        const int t = (int)w0 + k * 32 + __ffs((int)b) - 1;
        out[min(pos, m - 1)] = t;  // (pos < m: the members are distinct)
        rank[t] = pos;
      }
    base += all;
  }
  __threadfence_block();
  __syncthreads();
}

// ---------------------------------------------------------------------------
// centroid = bf16(mean of members), of the slice's clusters that gained or lost a
// key (all of them in the first iteration), and their sizes (into the offsets
// array, scanned at the end).  Their members, collected in LDS by one pass over
// the assignments, are sorted by token and summed:
//  - a wave per cluster of up to 64 members, the next cluster's members sorted
//    while this one's rows are in flight;
//  - larger ones (on a mixture, a centroid between components collects the keys
//    of many: 500 to 1000 of 65536) by four waves, one for each of the four
//    interleaved chains that every sum consists of, with 32 rows of a chain
//    in flight (16 rows at a time in one wave, the largest cluster had set the
//    kernel's time).
// 65536 x 8 keys of a mixture: 73 us in the first iteration (the gather of every
// key), 48 to 21 later.
// A slice of more than kSliceCap keys (a cluster of thousands, or fewer clusters
// than slices) takes two passes and lists in memory: there a wave takes
// clusters of up to kRankMax members, the workgroup sorts each larger one by a
// bitmap, and the four chains' waves sum it.  A wave for each of them (windows of
// 16384 tokens, 16 rows in flight) had made one iteration slower than counting
// tiles and a wave per mean: 65536 x 8 keys of which half are zero, first update 4.54
// ms, now 1.20, ten iterations 37.1 ms, now 12.3 (25.3 by tiles); 131072 x 8 keys, one iteration, 1 / 16 / 256 clusters
// 12.5 / 4.7 / 1.14 ms, now 3.0 / 1.1 / 0.73 (7.6 / 2.7 / 0.73); 81 distinct keys among 65536, two
// iterations 1.20 ms, now 0.66 (1.04).
// grid (slices, BG), 1024 threads; per: clusters per slice
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void km_update_kernel(KmArgs a, int per) {
  // [2 per] starts, [2 per] sizes, [2 per] dirty / place among the changed, [2 per] 16-bit list of the clusters of one wave each
  extern __shared__ __align__(16) int32_t s_dyn[];
  __shared__ __align__(16) uint32_t s_ord[16][kOrdWords];
  __shared__ int32_t s_tok[kSliceCap], s_mem[kSliceCap];
  __shared__ int s_big_lds[kSliceCap / kSmall];
  __shared__ int s_w[32], s_n, s_base, s_total, s_nbig, s_nsmall;
  static_assert(2 * kSliceMax <= kSliceCap, "the collected tokens' place holds a list of a slice's clusters");
  const int p = blockIdx.y;
  if (*done_flag(a, p)) return;
  const Problem q = problem(a, p);
  const Slice sc = make_slice(q.C, per, blockIdx.x);
  const int nc = sc.nr;
  if (nc <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, sl = lane & 15, grp = lane >> 4;
  int32_t *s_beg = s_dyn, *s_cnt = s_dyn + 2 * per, *s_slot = s_dyn + 4 * per;
  uint16_t* s_small = reinterpret_cast<uint16_t*>(s_dyn + 6 * per);
  int any = 0;
  for (int c = tid; c < nc; c += 1024) {
    int d = 0;
    if (sc.id(c) < q.C) {
      const int64_t at = q.cl_base + sc.id(c);
      d = a.iter == 1 ? 1 : a.dirty[at];
      a.dirty[at] = 0;
      a.moved[at] = 0;
    }
    any |= d;
    s_beg[c] = 0;
    s_slot[c] = d;
  }
  if (tid == 0) s_n = s_total = s_nbig = s_nsmall = 0;
  if (!__syncthreads_or(any)) return;
  const int32_t* assign = a.assign + q.tok_base;
  int32_t* rank = a.rank + q.tok_base;
  const int total = collect_slice(assign, q.n, sc, s_tok, &s_total);
  const bool in_lds = total <= kSliceCap;
  const uint32_t end = sc.end();
  int before = 0;  // keys of the slices before this one (the place of its lists in memory)
  constexpr int kE = kSliceCap / 1024;
  int tok_e[kE], cl_e[kE], place[kE];
  if (in_lds) {
#pragma unroll
    for (int e = 0; e < kE; ++e) {
      tok_e[e] = s_tok[max(min(tid + 1024 * e, total - 1), 0)];  // (unused when total is 0)
      place[e] = -1;
    }
#pragma unroll
    for (int e = 0; e < kE; ++e) cl_e[e] = tid + 1024 * e < total ? sc.local(sc.place(assign[tok_e[e]])) : -1;
#pragma unroll
    for (int e = 0; e < kE; ++e)
      if (cl_e[e] >= 0 && s_slot[cl_e[e]]) place[e] = atomicAdd(&s_beg[cl_e[e]], 1);
  } else {
    for_tokens(assign, q.n, [&](int, int c) {
      const uint32_t x = sc.place(c);
      before += __brev((uint32_t)c) < (uint32_t)sc.lo << sc.shift ? 1 : 0;
      if (x < end && s_slot[sc.local(x)]) atomicAdd(&s_beg[sc.local(x)], 1);
    });
  }
  __syncthreads();
  // the clusters to take (a slice may hold many empty or unchanged ones, and numbers that
  // no cluster has): those of more than `large` members, four waves each, and
  // the others (with lists in memory the former in the collected tokens' place)
  const int large = in_lds ? kSmall : kRankMax;
  int* s_big = in_lds ? s_big_lds : s_tok;
  for (int c = tid; c < nc; c += 1024) {
    const int m = s_beg[c];
    s_cnt[c] = m;
    if (s_slot[c]) a.offsets[q.off_base + sc.id(c)] = m;
    if (m == 0) s_slot[c] = -1;  // nothing to do: an empty cluster keeps its centroid
    else if (m > large) s_big[atomicAdd(&s_nbig, 1)] = c;
    else s_small[atomicAdd(&s_nsmall, 1)] = (uint16_t)c;
  }
  __syncthreads();
  before = slice_scan(s_beg, nc, before, s_w);
  int32_t* members = a.members + q.tok_base + before;
  int32_t* sorted = a.perm + q.tok_base + before;  // (perm: scratch until the layout)
  if (in_lds) {
#pragma unroll
    for (int e = 0; e < kE; ++e)
      if (place[e] >= 0) s_mem[s_beg[cl_e[e]] + place[e]] = tok_e[e];
  } else {
    const int room = q.n - before;  // (the lists of the slices' clusters fit: they are disjoint)
    for_tokens(assign, q.n, [&](int t, int c) {
      const uint32_t x = sc.place(c);
      if (x < end && s_cnt[sc.local(x)] > 0) members[min(atomicAdd(&s_beg[sc.local(x)], 1), room - 1)] = t;
    });
    __syncthreads();
    for (int c = tid; c < nc; c += 1024) s_beg[c] -= s_cnt[c];  // the cursors ended at the lists' ends
    __threadfence_block();
  }
  __syncthreads();

  // cluster c of m members with the sums s of its lane's 8 dimensions (the same
  // in the four lane-groups): store the centroid if it changed
  auto finish = [&](int c, int m, const float (&s)[8], const uint4& old) {
    const int64_t at = q.cl_base + sc.id(c);
    const float inv = 1.f / (float)m;
    float cn = 0.f;
    uint32_t out[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint16_t hb = f32_to_bf16_rne(s[e] * inv);
      const float r = __uint_as_float((uint32_t)hb << 16);
      cn = fmaf(r, r, cn);
      if (e & 1) out[e >> 1] |= (uint32_t)hb << 16;
      else out[e >> 1] = hb;
    }
    cn = sum16(cn);
    const bool moved = __any(out[0] != old.x || out[1] != old.y || out[2] != old.z || out[3] != old.w);
    if (moved && grp == 0)
      *reinterpret_cast<uint4*>(a.centroids + at * kHeadDim + sl * 8) = make_uint4(out[0], out[1], out[2], out[3]);
    if (lane == 0) {
      if (moved) {
        a.cnorm[at] = cn;
        a.moved[at] = 1;
      }
      s_slot[c] = moved ? atomicAdd(&s_n, 1) : -1;
    }
  };

  // ---- clusters of more than `large` members
  const int nbig = __builtin_amdgcn_readfirstlane(s_nbig);
  if (nbig > 0) {
    // their members by token, into s_tok (a wave ranks 64 members of a cluster
    // against all of its members) or, from the lists in memory, into `sorted`
    int task = 0;
    for (int i = 0; i < nbig; ++i) {
      const int c = __builtin_amdgcn_readfirstlane(s_big[i]);
      const int b0 = __builtin_amdgcn_readfirstlane(s_beg[c]), m = __builtin_amdgcn_readfirstlane(s_cnt[c]);
      if (!in_lds) {
        sort_by_bitmap(members + b0, m, q.n, &s_ord[0][0], sorted + b0, rank, s_w);
        continue;
      }
      for (int j0 = 0; j0 < m; j0 += 64, ++task) {
        if ((task & 15) != wave) continue;
        const int x = j0 + lane < m ? s_mem[b0 + j0 + lane] : 0x7fffffff;
        int r = 0;
        for (int k0 = 0; k0 < m; k0 += 64) {
          const int y = k0 + lane < m ? s_mem[b0 + k0 + lane] : 0x7fffffff;
          r += count_below(y, x, m - k0);
        }
        if (j0 + lane < m) {
          s_tok[b0 + r] = x;
          rank[x] = r;
        }
      }
    }
    __syncthreads();
    float* s_part = reinterpret_cast<float*>(s_ord);  // [4 clusters][4 chains][128]
    const int quad = wave >> 2, chain = wave & 3;
    for (int i0 = 0; i0 < nbig; i0 += 4) {
      const bool on = i0 + quad < nbig;
      const int c = __builtin_amdgcn_readfirstlane(on ? s_big[i0 + quad] : 0);
      const int b0 = __builtin_amdgcn_readfirstlane(s_beg[c]), m = on ? __builtin_amdgcn_readfirstlane(s_cnt[c]) : 0;
      uint4 old = make_uint4(0, 0, 0, 0);
      if (on && chain == 0) old = *reinterpret_cast<const uint4*>(a.centroids + (q.cl_base + sc.id(c)) * kHeadDim + sl * 8);
      // the chain's rows chain, chain + 4, ...; this lane's two dimensions
      float s0 = 0.f, s1 = 0.f;
      const uint32_t* Kl = reinterpret_cast<const uint32_t*>(a.K + q.tok_base * kHeadDim) + lane;
      const int nr = (m - chain + 3) / 4;
      auto row = [&](int r) {  // (r < nr, or the last row again)
        const int i = b0 + min(chain + 4 * r, m - 1);
        return in_lds ? s_tok[i] : sorted[i];
      };
      int t_next = nr > 0 ? row(lane) : 0;
      for (int r0 = 0; r0 < nr; r0 += 64) {
        const int t = t_next;
        if (r0 + 64 < nr) t_next = row(r0 + 64 + lane);  // travels during the sums
        const int rm = min(64, nr - r0);
#pragma unroll
        for (int k0 = 0; k0 < 64; k0 += 32) {
          if (k0 >= rm) break;
          uint32_t v[32];  // (lanes past the end hold the last row again)
#pragma unroll
          for (int k = 0; k < 32; ++k)
            v[k] = Kl[(int64_t)min(max(__builtin_amdgcn_readlane(t, k0 + k), 0), q.n - 1) * (kHeadDim / 2)];
#pragma unroll
          for (int k = 0; k < 32; ++k)
            if (k0 + k < rm) {
              s0 += bf16lo(v[k]);
              s1 += bf16hi(v[k]);
            }
        }
      }
      if (on) *reinterpret_cast<float2*>(s_part + (quad * 4 + chain) * kHeadDim + 2 * lane) = make_float2(s0, s1);
      __syncthreads();
      if (on && chain == 0) {
        float s[8];
        const float* x = s_part + quad * 4 * kHeadDim + sl * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          s[e] = (x[e] + x[kHeadDim + e]) + (x[2 * kHeadDim + e] + x[3 * kHeadDim + e]);
        finish(c, m, s, old);
      }
      __syncthreads();  // s_part is rewritten
    }
  }

  // ---- the others: a wave per cluster
  constexpr int kHalf = kOrdWords / 2;  // (two buffers of up to kSmall members, or one of the lists in memory)
  auto sort = [&](int c, int buf) {
    const int b0 = __builtin_amdgcn_readfirstlane(s_beg[c]), m = __builtin_amdgcn_readfirstlane(s_cnt[c]);
    if (in_lds) sort_small(s_mem + b0, m, s_ord[wave] + buf * kHalf, rank, lane);
    else sort_members(members + b0, m, s_ord[wave], rank, lane);
  };
  const int nsmall = __builtin_amdgcn_readfirstlane(s_nsmall);
  auto small = [&](int i) { return __builtin_amdgcn_readfirstlane((int)s_small[min(i, nsmall - 1)]); };
  if (wave < nsmall && in_lds) sort(small(wave), 0);
  for (int i = wave, buf = 0; i < nsmall; i += 16, buf ^= 1) {
    const int c = small(i);
    const int m = __builtin_amdgcn_readfirstlane(s_cnt[c]);
    const uint4 old = *reinterpret_cast<const uint4*>(a.centroids + (q.cl_base + sc.id(c)) * kHeadDim + sl * 8);
    if (!in_lds) sort(c, 0);
    const uint32_t* ord = s_ord[wave] + (in_lds ? buf * kHalf : 0);
    // lane-group grp sums members grp, grp + 4, grp + 8, ... in that order;
    // 16 rows per step, their key rows loaded together
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    uint4 v[4];
    auto load = [&](int r0) {
      int tok[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) tok[k] = min(max((int)ord[min(r0 + grp + 4 * k, m - 1)], 0), q.n - 1);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        v[k] = *reinterpret_cast<const uint4*>(a.K + (q.tok_base + tok[k]) * kHeadDim + sl * 8);
    };
    load(0);
    if (i + 16 < nsmall && in_lds) sort(small(i + 16), buf ^ 1);
    for (int r0 = 0; r0 < m; r0 += 16) {
      if (r0 > 0) load(r0);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (r0 + grp + 4 * k >= m) continue;
        const uint32_t w[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[2 * e] += bf16lo(w[e]);
          s[2 * e + 1] += bf16hi(w[e]);
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      s[e] += __shfl_xor(s[e], 16, 64);
      s[e] += __shfl_xor(s[e], 32, 64);
    }
    finish(c, m, s, old);
  }
  // the changed centroids join the problem's list (its order does not matter:
  // equal scores among them list the key); the rows written above are read back
  __threadfence_block();
  __syncthreads();
  if (s_n == 0) return;
  if (tid == 0) s_base = atomicAdd(n_moved(a, p), s_n);
  __syncthreads();
  for (int j = tid >> 4; j < nc; j += 64) {
    if (s_slot[j] < 0) continue;
    const int64_t at = q.cl_base + sc.id(j), to = q.cl_base + s_base + s_slot[j];
    *reinterpret_cast<uint4*>(a.d_rows + to * kHeadDim + sl * 8) =
        *reinterpret_cast<const uint4*>(a.centroids + at * kHeadDim + sl * 8);
    if (sl == 0) {
      a.d_norm[to] = a.cnorm[at];
      a.d_id[to] = sc.id(j);
    }
  }
}

// ---------------------------------------------------------------------------
// offsets: exclusive scan of the cluster sizes, in place.  grid BG, 1024 threads
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void km_layout_kernel(KmArgs a) {
  __shared__ int s_w[16];
  const Problem q = problem(a, blockIdx.x);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int32_t* off = a.offsets + q.off_base;
  constexpr int kPer = 8;
  int carry = 0;
  for (int64_t c0 = 0; c0 < q.C; c0 += 1024 * kPer) {
    const int64_t c = c0 + tid * kPer;
    int v[kPer], loc = 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) v[e] = c + e < q.C ? off[c + e] : 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) loc += v[e];
    const int incl = wave_incl_scan(loc);  // DPP, no LDS
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    int run = carry + incl - loc;
    for (int w = 0; w < 16; ++w) {
      run += w < wave ? s_w[w] : 0;
      carry += s_w[w];
    }
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if (c + e < q.C) off[c + e] = run;
      run += v[e];
    }
    __syncthreads();  // s_w is rewritten
  }
  if (tid == 0) off[q.C] = q.n;
}

// ---------------------------------------------------------------------------
// the cluster order: every token's row is its cluster's first row plus its rank;
// perm[row] = token, K_sorted[row] = K[token] (and V).  Bound by memory: the rows
// are read in token order and written to their places (past the caches: 1% of a
// call of two iterations).  131072 x 2 sequences x 8 heads: with the scan of the sizes 390 us;
// placing the tokens by a pass over the assignments in every slice of the
// clusters, then gathering the rows, had taken 105 + 348.
// grid (ceil(nmax/16), BG), 256 threads
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void km_permute_kernel(KmArgs a) {
  const int p = blockIdx.y;
  const Problem q = problem(a, p);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sl = lane & 15, grp = lane >> 4;
  const int t = blockIdx.x * 16 + wave * 4 + grp;
  if (t >= q.n) return;
  const int64_t src = (q.tok_base + t) * kHeadDim + sl * 8;
  uint4 k = make_uint4(0, 0, 0, 0), v = k;
  if (a.K_sorted) k = load_stream16(a.K + src);
  if (a.V_sorted) v = load_stream16(a.V + src);
  const int c = a.assign[q.tok_base + t], rk = a.rank[q.tok_base + t];
  const int row = min(max(a.offsets[q.off_base + max(c, 0)] + rk, 0), q.n - 1);
  if (sl == 0) a.perm[q.tok_base + row] = t;
  const int64_t dst = (q.tok_base + row) * kHeadDim + sl * 8;
  if (a.K_sorted) store_stream16(a.K_sorted + dst, k);
  if (a.V_sorted) store_stream16(a.V_sorted + dst, v);
}

// ---------------------------------------------------------------------------
// host driver
// ---------------------------------------------------------------------------
namespace {

struct KmLayout {
  int64_t off_cnorm, off_best, off_bound, off_members, off_rank, off_dirty, off_moved;
  int64_t off_drows, off_dnorm, off_did, off_ltok, off_lkey, off_lsecond, off_state, bytes;
};

KmLayout km_layout(int B, int Hkv, int64_t total, int64_t Ct) {
  KmLayout L;
  const int64_t BG = (int64_t)B * Hkv;
  int64_t cur = 0;
  auto take = [&](int64_t bytes) {
    const int64_t o = cur;
    cur = (cur + bytes + 255) / 256 * 256;
    return o;
  };
  const int64_t tok = (int64_t)Hkv * total, cl = (int64_t)Hkv * Ct;
  L.off_cnorm = take(cl * 4);
  L.off_best = take(tok * 4);
  L.off_bound = take(tok * 4);
  L.off_members = take(tok * 4);
  L.off_rank = take(tok * 4);
  L.off_dirty = take(cl * 4);
  L.off_moved = take(cl * 4);
  L.off_drows = take(cl * kHeadDim * 2);
  L.off_dnorm = take(cl * 4);
  L.off_did = take(cl * 4);
  L.off_ltok = take(tok * 4);
  L.off_lkey = take(tok * 8);
  L.off_lsecond = take(tok * 4);
  L.off_state = take(BG * kStateInts * 4);
  L.bytes = cur;
  return L;
}

}  // namespace

size_t kmeans_workspace_bytes(int B, int Hkv, int64_t total, int64_t Ct) {
  return (size_t)km_layout(B, Hkv, total, Ct).bytes;
}

hipError_t run_kmeans(const uint16_t* K, const uint16_t* V, const int64_t* kv_indptr, const int64_t* seq_len,
                      const int64_t* cl_indptr, int B, int Hkv, int64_t total, int64_t nmax,
                      int64_t Ct, int Cm, const int32_t* init_idx, int max_iters,
                      const uint16_t* prev_centroids, const int64_t* prev_cl_indptr, uint16_t* centroids, int32_t* assign, int32_t* offsets, int32_t* perm,
                      uint16_t* K_sorted, uint16_t* V_sorted, void* workspace, hipStream_t st) {
  const KmLayout L = km_layout(B, Hkv, total, Ct);
  char* ws = static_cast<char*>(workspace);
  const int BG = B * Hkv;
  KmArgs a;
  a.K = K;
  a.V = V;
  a.kv_indptr = kv_indptr;
  a.seq_len = seq_len;
  a.cl_indptr = cl_indptr;
  a.B = B;
  a.Hkv = Hkv;
  a.Cm = Cm;
  a.iter = 0;
  a.total = total;
  a.Ct = Ct;
  a.init_idx = init_idx;
  a.prev_centroids = prev_centroids;
  a.prev_cl_indptr = prev_cl_indptr;
  a.centroids = centroids;
  a.cnorm = reinterpret_cast<float*>(ws + L.off_cnorm);
  a.assign = assign;
  a.offsets = offsets;
  a.perm = perm;
  a.best = reinterpret_cast<float*>(ws + L.off_best);
  a.bound = reinterpret_cast<float*>(ws + L.off_bound);
  a.members = reinterpret_cast<int32_t*>(ws + L.off_members);
  a.rank = reinterpret_cast<int32_t*>(ws + L.off_rank);
  a.dirty = reinterpret_cast<int32_t*>(ws + L.off_dirty);
  a.moved = reinterpret_cast<int32_t*>(ws + L.off_moved);
  a.d_rows = reinterpret_cast<uint16_t*>(ws + L.off_drows);
  a.d_norm = reinterpret_cast<float*>(ws + L.off_dnorm);
  a.d_id = reinterpret_cast<int32_t*>(ws + L.off_did);
  a.l_tok = reinterpret_cast<int32_t*>(ws + L.off_ltok);
  a.l_key = reinterpret_cast<uint64_t*>(ws + L.off_lkey);
  a.l_second = reinterpret_cast<uint32_t*>(ws + L.off_lsecond);
  a.state = reinterpret_cast<int32_t*>(ws + L.off_state);
  a.K_sorted = K_sorted;
  a.V_sorted = V_sorted;
  const dim3 g_cl((Cm + 3) / 4, BG), g_tok((unsigned)((nmax + kAsgTok - 1) / kAsgTok), BG);
  // slices of the clusters: at least one workgroup for each of the 256 compute
  // units and few enough keys per slice for LDS (half of kSliceCap on
  // average); no more than the latter needs below 16 clusters (a wave each), and
  // at most kSliceMax clusters
  const int64_t ns_lds = std::max<int64_t>(1, (nmax + kSliceCap / 2 - 1) / (kSliceCap / 2));
  const int64_t ns = std::max<int64_t>((256 + BG - 1) / BG, ns_lds);
  const int64_t least = std::min<int64_t>(16, (Cm + ns_lds - 1) / ns_lds);
  const int per = (int)std::min<int64_t>(kSliceMax, std::max<int64_t>(least, (Cm + ns - 1) / ns));
  const dim3 g_slice((Cm + per - 1) / per, BG);
  const size_t lds_upd = (size_t)per * 28;
  // listed keys: work items in flight per problem, three workgroups on each of
  // the 256 compute units together, at most as many as a problem has items
  const int64_t items = (int64_t)g_tok.x * ((Cm + kListCen - 1) / kListCen);
  const dim3 g_list((unsigned)std::min<int64_t>(items, std::max(8, 768 / BG)), BG);
  hipLaunchKernelGGL(km_init_kernel, g_cl, dim3(256), 0, st, a);
  hipError_t e = hipGetLastError();
  const int full = a.prev_centroids ? 1 : 2;  // iterations that measure every pair; the last of them leaves the bounds
  for (int it = 1; it <= max_iters && e == hipSuccess; ++it) {
    a.iter = it;
    if (it <= full) {
      if (it == full && max_iters > full) hipLaunchKernelGGL((km_assign_kernel<0, true>), g_tok, dim3(256), 0, st, a);
      else hipLaunchKernelGGL((km_assign_kernel<0, false>), g_tok, dim3(256), 0, st, a);
    } else {
      hipLaunchKernelGGL(km_assign_kernel<1>, g_tok, dim3(256), 0, st, a);
      hipLaunchKernelGGL(km_assign_kernel<2>, g_list, dim3(256), 0, st, a);
    }
    if (it > 1) hipLaunchKernelGGL(km_merge_kernel, dim3(BG), dim3(1024), 0, st, a);
    hipLaunchKernelGGL(km_update_kernel, g_slice, dim3(1024), lds_upd, st, a, per);
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    if (!V) a.V_sorted = nullptr;
    hipLaunchKernelGGL(km_layout_kernel, dim3(BG), dim3(1024), 0, st, a);
    hipLaunchKernelGGL(km_permute_kernel, dim3((unsigned)((nmax + 15) / 16), BG), dim3(256), 0, st, a);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace tactic
