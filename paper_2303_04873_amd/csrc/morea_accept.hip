// Acceptance of partial solutions in optimal mixing (Sec. 3): a sampled
// partial solution, inserted into its parent, is kept when the result
// dominates the parent or is not dominated within the current elitist
// archive.  Kept children are written into their parents: the group's new
// coordinates into the parent's points, the dependent tets' records of the
// partial evaluation into the parent's cache, and the parent's totals and
// objectives recomputed from the cache.
//
// Definitions where the paper leaves the details to MO-RV-GOMEA's
// literature (all three objectives are minimised):
//   feasible: flags == 0 in the fold and invalid bits; violation = severity
//     (summed |signed volume| of the violating tets) when a fold bit is set,
//     +inf when the invalid bit is set or an objective or the severity is not
//     finite (NaN or an infinity);
//   child vs parent: constraint domination -- feasible beats infeasible, two
//     infeasible compare violations (strictly smaller wins), two feasible
//     compare by Pareto domination (none worse, one strictly better);
//   archive: feasible objective vectors; a feasible child is non-dominated
//     when no member Pareto-dominates it (an equal member does not);
//   an evaluation whose parent or group index is out of range is rejected;
//   adaptive steering (Sec. 4.3.2): a guidance value above the caller's bound
//     (1.5 times the archive's best) is a hard constraint -- the solution is
//     infeasible and violations compare lexicographically as (fold
//     violation, FP32 excess guidance - bound); an infinite bound is off.
//
// Three launches: the decisions (one thread per evaluation, the archive
// staged through LDS in chunks shared by the block), the write-back (one
// wave per evaluation: 48-byte record pairs as three 16-byte vectors, then
// the group's coordinates), and the per-candidate reduction of the
// evaluation over the parents' caches.
#include <math.h>

#include <algorithm>
#include <stdio.h>
#include <string.h>

#include "morea_internal.h"

namespace morea {
namespace accept {

constexpr int kBlock = 256;
constexpr int kChunk = 512;   // archive members staged per pass (6 KB of LDS)

// Feasibility and the violation pair (fold violation, guidance excess).
__device__ __forceinline__ bool feasible_of(float o0, float o1, float o2, uint8_t f, float sev, float gmax,
                                            float& fold, float& excess) {
  if ((f & 4u) || !isfinite(o0) || !isfinite(o1) || !isfinite(o2) || !isfinite(sev)) {
    fold = excess = INFINITY;
    return false;
  }
  const bool folded = (f & 3u) != 0, over = o2 > gmax;
  fold = folded ? sev : 0.f;
  excess = over ? o2 - gmax : 0.f;
  return !folded && !over;
}

__device__ __forceinline__ bool pareto(float a0, float a1, float a2, float b0, float b1, float b2) {
  return a0 <= b0 && a1 <= b1 && a2 <= b2 && (a0 < b0 || a1 < b1 || a2 < b2);
}

__global__ __launch_bounds__(kBlock) void k_decide(int n_evals, int n_parents, int n_groups,
                                                   const int* __restrict__ eval_parent,
                                                   const int* __restrict__ eval_group,
                                                   const float* __restrict__ child_obj,
                                                   const uint8_t* __restrict__ child_flags,
                                                   const float* __restrict__ child_sev,
                                                   const float* __restrict__ parent_obj,
                                                   const uint8_t* __restrict__ parent_flags,
                                                   const float* __restrict__ parent_sev,
                                                   const float* __restrict__ archive, int n_archive, float gmax,
                                                   uint8_t* __restrict__ accepted) {
  __shared__ float s_arc[kChunk * 3];
  const int e = blockIdx.x * kBlock + threadIdx.x;
  bool decided = true, ok = false;
  float c0 = 0.f, c1 = 0.f, c2 = 0.f;
  if (e < n_evals) {
    const int par = eval_parent[e], g = eval_group[e];
    if (par >= 0 && par < n_parents && g >= 0 && g < n_groups) {
      c0 = child_obj[3 * e];
      c1 = child_obj[3 * e + 1];
      c2 = child_obj[3 * e + 2];
      float fc_fold, fc_exc, fp_fold, fp_exc;
      const bool fc = feasible_of(c0, c1, c2, child_flags[e], child_sev[e], gmax, fc_fold, fc_exc);
      const float p0 = parent_obj[3 * par], p1 = parent_obj[3 * par + 1], p2 = parent_obj[3 * par + 2];
      const bool fp = feasible_of(p0, p1, p2, parent_flags[par], parent_sev[par], gmax, fp_fold, fp_exc);
      const bool less = fc_fold < fp_fold || (fc_fold == fp_fold && fc_exc < fp_exc);
      const bool dom = (fc && fp) ? pareto(c0, c1, c2, p0, p1, p2) : (fc != fp ? fc : less);
      if (dom) {
        ok = true;
      } else if (fc) {
        ok = true;          // until a member of the archive dominates it
        decided = false;
      }
    }
  }
  for (int base = 0; base < n_archive; base += kChunk) {
    if (!__syncthreads_or(decided ? 0 : 1)) break;
    const int m = min(kChunk, n_archive - base);
    for (int i = threadIdx.x; i < 3 * m; i += kBlock) s_arc[i] = archive[3 * static_cast<size_t>(base) + i];
    __syncthreads();
    if (!decided) {
      for (int i = 0; i < m; i++)
        if (pareto(s_arc[3 * i], s_arc[3 * i + 1], s_arc[3 * i + 2], c0, c1, c2)) {
          ok = false;
          decided = true;
          break;
        }
    }
  }
  if (e < n_evals) accepted[e] = ok ? 1 : 0;
}

// One wave per evaluation: the accepted child's dependent-tet records (two
// directions, 48 bytes) into the parent's cache, and its group's new
// coordinates into the parent's points.
__global__ __launch_bounds__(kBlock) void k_write_back(int n_evals, int n_parents, int n_groups, int n_points,
                                                       int n_tets, const int* __restrict__ eval_parent,
                                                       const int* __restrict__ eval_group,
                                                       const uint8_t* __restrict__ accepted,
                                                       const int* __restrict__ row_off,
                                                       const int* __restrict__ item_off,
                                                       const int* __restrict__ grp_off,
                                                       const int* __restrict__ grp_pts,
                                                       const int* __restrict__ dep_off,
                                                       const int* __restrict__ dep_tet,
                                                       const float* __restrict__ new_coords,
                                                       const uint4* __restrict__ new_rec,
                                                       float* __restrict__ parent_pts,
                                                       uint4* __restrict__ parent_rec) {
  const int e = blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  if (e >= n_evals || !accepted[e]) return;
  const int par = eval_parent[e], g = eval_group[e];
  if (par < 0 || par >= n_parents || g < 0 || g >= n_groups) return;
  const int d0 = dep_off[g], nd = dep_off[g + 1] - d0;
  const size_t src = static_cast<size_t>(item_off[e]) * 3;
  for (int i = lane; i < 3 * nd; i += kWave) {
    const int j = i / 3, q = i - 3 * j;
    const size_t dst = (static_cast<size_t>(par) * n_tets + dep_tet[d0 + j]) * 3;
    parent_rec[dst + q] = new_rec[src + 3 * static_cast<size_t>(j) + q];
  }
  const int k0 = grp_off[g], nk = grp_off[g + 1] - k0;
  const size_t row = static_cast<size_t>(row_off[e]);
  for (int i = lane; i < 6 * nk; i += kWave) {
    const int k = i / 6, r = i - 6 * k;   // r = mesh * 3 + axis
    parent_pts[(static_cast<size_t>(par) * 6 + r) * n_points + grp_pts[k0 + k]] = new_coords[(row + k) * 6 + r];
  }
}

// ---------------------------------------------------------------- selection
// Selection and clustering at the start of a generation (Sec. 3: a selection
// of non-dominated solutions of the population, clustered into k equally
// sized clusters), one block of 1024 threads, one solution per thread.
// Definitions where the paper leaves the details to MO-RV-GOMEA's literature:
//   fronts by peeling under the constraint domination above; the selection
//     takes whole fronts in order and the last one it needs in ascending
//     index, up to `size` solutions; invalid solutions are never selected;
//   objectives normalised over the selection, (v - lo) / (hi - lo), 0 where
//     hi == lo; squared Euclidean distances in FP64, contraction off;
//   leaders: the selected solution with the smallest normalised first
//     objective, then repeatedly the one farthest from the leaders so far
//     (ties to the lower index), min(k, |S|) of them;
//   cluster j: the m = min(|S|, ceil(2 |S| / k)) selected solutions nearest
//     to leader j (ties to the lower index), in ascending index;
//   the cluster of a valid solution: its nearest leader (ties to the lower
//     cluster); -1 for an invalid one.
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / kWave;

struct SelShared {
  union {
    uint32_t dom[kSelThreads / 32][kSelThreads];   // [word][solution] dominators, bit by bit
    struct {                                       // once the fronts are known
      double norm[3][kSelThreads];                 // normalised objectives of the population
      double sel[3][kSelThreads];                  // and of the selected solutions, in order
      double key[kSelThreads];                     // distances to the leaders of a pass
      int leader[kSelThreads];
      int who[kSelThreads];                        // index of each selected solution
    };
  };
  // feasible: the objectives, infeasible: the violation (folds, excess, 0);
  // w: bit 0 valid, bit 1 feasible
  float4 sol[kSelThreads];
  uint32_t left[kSelThreads / 32];
  double wkey[kSelThreads / 16];
  int widx[kSelThreads / 16];
  int wsum[kSelWaves];
};

// One step of the lexicographic minimum of (key, idx) over the 16 lanes of a
// DPP row, by the lane permutation `ctrl`.
template <int ctrl>
__device__ __forceinline__ void argmin_step(double& key, int& idx) {
  const uint64_t u = static_cast<uint64_t>(__double_as_longlong(key));
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u), ctrl, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), ctrl, 0xf, 0xf, false);
  const double k2 = __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(hi) << 32 | lo));
  const int i2 = __builtin_amdgcn_update_dpp(0, idx, ctrl, 0xf, 0xf, false);
  const bool less = k2 < key || (k2 == key && i2 < idx);
  key = less ? k2 : key;
  idx = less ? i2 : idx;
}

__device__ __forceinline__ void argmin_row(double& key, int& idx) {
  argmin_step<0xb1>(key, idx);     // quad_perm 1 0 3 2
  argmin_step<0x4e>(key, idx);     // quad_perm 2 3 0 1
  argmin_step<0x141>(key, idx);    // row_half_mirror
  argmin_step<0x140>(key, idx);    // row_mirror
}

// Block-wide minimum of (key, idx) (lexicographic); every thread returns it.
__device__ void block_argmin(SelShared& S, double key, int idx, double& out_key, int& out_idx) {
  const int lane = threadIdx.x & 63;
  argmin_row(key, idx);
  if ((lane & 15) == 0) {
    S.wkey[threadIdx.x >> 4] = key;
    S.widx[threadIdx.x >> 4] = idx;
  }
  __syncthreads();
  key = S.wkey[lane];              // 64 rows of 16 threads
  idx = S.widx[lane];
  argmin_row(key, idx);
#pragma unroll
  for (int d = 16; d <= 32; d <<= 1) {
    const double k2 = __shfl_xor(key, d, 64);
    const int i2 = __shfl_xor(idx, d, 64);
    const bool less = k2 < key || (k2 == key && i2 < idx);
    key = less ? k2 : key;
    idx = less ? i2 : idx;
  }
  out_key = key;
  out_idx = idx;
  __syncthreads();
}

// Block-wide exclusive prefix sum of a flag; *total receives the sum.
__device__ int block_scan(SelShared& S, bool v, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t m = __ballot(v);
  if (lane == 0) S.wsum[w] = __popcll(m);
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < kSelWaves; k++) {
    const int s = S.wsum[k];
    before += k < w ? s : 0;
    all += s;
  }
  __syncthreads();
  *total = all;
  return before + __popcll(m & ((1ull << lane) - 1ull));
}

__device__ __forceinline__ double dist3(const double* a, const double* b) {
#pragma clang fp contract(off)
  double s = 0.0;
  for (int o = 0; o < 3; o++) {
    const double d = a[o] - b[o];
    const double p = d * d;
    s = s + p;
  }
  return s;
}

// Bound: the latency and issue of one block (every step needs the one before);
// 512 solutions, 179 selected into 10 clusters: 83 us, before 337.  The
// dominator rows are split over all threads (several to a solution when the
// population is smaller than the block) and tested without branches (with
// them 106 us of the kernel), the reductions run on DPP rows and 64 row
// results (1.8 us each over shuffles of whole waves), and the clusters'
// members are ranked for as many clusters at a time as the block holds copies
// of the selection.
__global__ __launch_bounds__(kSelThreads) void k_select(int n, int size, int k, float gmax,
                                                        const float* __restrict__ obj,
                                                        const uint8_t* __restrict__ flags,
                                                        const float* __restrict__ sev, int* __restrict__ sel_out,
                                                        int* __restrict__ n_sel_out, int* __restrict__ clu_off,
                                                        int* __restrict__ clu_members,
                                                        int* __restrict__ cluster_of) {
#pragma clang fp contract(off)
  __shared__ SelShared S;
  const int i = threadIdx.x;
  const bool in = i < n;
  float o[3] = {0.f, 0.f, 0.f};
  bool valid = false;
  {
    float fold = 0.f, exc = 0.f;
    bool feas = false;
    if (in) {
      for (int q = 0; q < 3; q++) o[q] = obj[3 * i + q];
      const uint8_t f = flags[i];
      const float sv = sev[i];
      valid = !((f & 4u) || !isfinite(o[0]) || !isfinite(o[1]) || !isfinite(o[2]) || !isfinite(sv));
      feas = feasible_of(o[0], o[1], o[2], f, sv, gmax, fold, exc);
    }
    S.sol[i] = make_float4(feas ? o[0] : fold, feas ? o[1] : exc, feas ? o[2] : 0.f,
                           __int_as_float((valid ? 1 : 0) | (feas ? 2 : 0)));
  }
  const uint64_t vm = __ballot(valid);
  if ((i & 31) == 0) S.left[i >> 5] = static_cast<uint32_t>(vm >> (i & 32));
  __syncthreads();
  // dominators of each solution as bits; thread i takes every parts-th word
  // of solution i % rows
  const int n_words = (n + 31) / 32;
  {
    int rows = kWave;
    while (rows < n) rows <<= 1;
    const int me = i & (rows - 1), parts = kSelThreads / rows;
    const float4 a = S.sol[me];
    const bool a_feas = (__float_as_int(a.w) & 2) != 0;
    for (int w = i / rows; w < n_words; w += parts) {
      uint32_t bits = 0u;
#pragma unroll 16
      for (int j = 0; j < 32; j++) {    // solutions beyond n are not valid
        const float4 b = S.sol[32 * w + j];
        const int bm = __float_as_int(b.w);
        const bool b_feas = (bm & 2) != 0;
        // without branches: both feasible, both infeasible, or one of each
        const bool lt = b.x < a.x, eq = b.x == a.x, lt1 = b.y < a.y, le1 = b.y <= a.y;
        const bool par = (lt | eq) & le1 & (b.z <= a.z) & (lt | lt1 | (b.z < a.z));
        const bool less = lt | (eq & lt1);
        const bool same = a_feas ? par : less;
        const bool dom = ((a_feas == b_feas) ? same : b_feas) & ((bm & 1) != 0);
        bits |= static_cast<uint32_t>(dom) << j;
      }
      S.dom[w][me] = bits;              // a solution does not dominate itself
    }
  }
  __syncthreads();
  // fronts by peeling until `size` solutions are covered: a solution joins
  // the front when none of its dominators is left
  bool left = valid, chosen = false;
  int covered = 0;
  while (covered < size) {
    uint32_t hit = 0u;
    if (left)
      for (int w = 0; w < n_words; w++) hit |= S.dom[w][i] & S.left[w];
    const bool front = left && hit == 0u;
    int n_front;
    const int before = block_scan(S, front, &n_front);   // its barriers end the reads of `left`
    if (n_front == 0) break;
    // the last front needed is cut in ascending index
    if (front) {
      left = false;
      chosen = covered + before < size;
    }
    const uint64_t lm = __ballot(left);
    if ((i & 31) == 0) S.left[i >> 5] = static_cast<uint32_t>(lm >> (i & 32));
    covered += n_front;
    __syncthreads();
  }
  int n_sel;
  const int pos = block_scan(S, chosen, &n_sel);
  if (chosen) sel_out[pos] = S.who[pos] = i;
  if (i == 0) *n_sel_out = n_sel;
  const int k_eff = min(k, n_sel);
  const int m = n_sel == 0 ? 0 : min(n_sel, (2 * n_sel + k - 1) / k);
  for (int j = i; j <= k; j += kSelThreads) clu_off[j] = min(j, k_eff) * m;
  if (n_sel == 0) {
    if (in) cluster_of[i] = -1;
    return;
  }
  // normalisation over the selection (exact minima and maxima)
  double me[3];
#pragma unroll
  for (int q = 0; q < 3; q++) {
    double lo, hi;
    int dummy;
    const double v = static_cast<double>(o[q]);
    block_argmin(S, chosen ? v : INFINITY, 0, lo, dummy);
    block_argmin(S, chosen ? -v : INFINITY, 0, hi, dummy);
    hi = -hi;
    me[q] = hi > lo ? (v - lo) / (hi - lo) : 0.0;
    S.norm[q][i] = me[q];
    if (chosen) S.sel[q][pos] = me[q];
  }
  __syncthreads();
  // leaders: smallest first objective, then farthest points
  double kk;
  int first;
  block_argmin(S, chosen ? me[0] : INFINITY, chosen ? i : 0x7fffffff, kk, first);
  if (i == 0) S.leader[0] = first;
  double lead[3] = {S.norm[0][first], S.norm[1][first], S.norm[2][first]};
  double nearest = chosen ? dist3(me, lead) : 0.0;
  // cluster of every valid solution: the nearest leader, ties to the lower
  int best = 0;
  double best_d = dist3(me, lead);
  for (int j = 1; j < k_eff; j++) {
    int nxt;
    block_argmin(S, chosen ? -nearest : INFINITY, chosen ? i : 0x7fffffff, kk, nxt);
    if (i == 0) S.leader[j] = nxt;
    const double ln[3] = {S.norm[0][nxt], S.norm[1][nxt], S.norm[2][nxt]};
    const double d = dist3(me, ln);
    if (chosen && d < nearest) nearest = d;
    if (d < best_d) {
      best_d = d;
      best = j;
    }
  }
  if (in) cluster_of[i] = valid ? best : -1;
  __syncthreads();
  // members of each cluster: the m nearest selected solutions, ascending
  // index; `group` clusters per pass, thread i taking selected solution q of
  // cluster j0 + g
  const int group = max(1, kSelThreads / n_sel), g = i / n_sel, q = i - g * n_sel;
  for (int j0 = 0; j0 < k_eff; j0 += group) {
    const bool mine = g < group && j0 + g < k_eff;
    double dme = 0.0;
    if (mine) {
      const int L = S.leader[j0 + g];
      const double ln[3] = {S.norm[0][L], S.norm[1][L], S.norm[2][L]};
      const double mq[3] = {S.sel[0][q], S.sel[1][q], S.sel[2][q]};
      dme = dist3(mq, ln);
      S.key[i] = dme;
    }
    __syncthreads();
    int closer = 0;
    if (mine) {
      const double* keys = &S.key[g * n_sel];
#pragma unroll 8
      for (int r = 0; r < n_sel; r++) {
        const double dq = keys[r];
        closer += (dq < dme || (dq == dme && r < q)) ? 1 : 0;
      }
    }
    const bool member = mine && closer < m;
    int cnt;
    // exactly m members by the (distance, index) order in every cluster of
    // the pass; the bound keeps every write inside cluster j's m slots
    const int at = block_scan(S, member, &cnt) - g * m;
    if (member && at >= 0 && at < m) clu_members[(j0 + g) * m + at] = S.who[q];
  }
}

}  // namespace accept
}  // namespace morea

using namespace morea;

namespace {

morea_status accept_fail(morea_status code, const char* msg) {
  set_error(msg);
  return code;
}

}  // namespace

extern "C" morea_status morea_select_clusters(const float* obj, const uint8_t* flags, const float* severity,
                                              int32_t n_pop, int32_t size, int32_t k, float guidance_max,
                                              int32_t* selection, int32_t* n_selected, int32_t* clu_off,
                                              int32_t* clu_members, int32_t members_cap, int32_t* cluster_of,
                                              void* stream) {
  if (n_pop < 1 || n_pop > accept::kSelThreads || size < 0 || k < 1 || isnan(guidance_max))
    return accept_fail(MOREA_EINVAL, "need 1 <= n_pop <= 1024, size >= 0, k >= 1, guidance_max not NaN");
  if (!obj || !flags || !severity || !selection || !n_selected || !clu_off || !clu_members || !cluster_of)
    return accept_fail(MOREA_EINVAL, "NULL argument");
  const int64_t s = std::min<int64_t>(size, n_pop);
  if (static_cast<int64_t>(members_cap) < k * ((2 * s + k - 1) / k))
    return accept_fail(MOREA_ERANGE, "members_cap below k * ceil(2 min(size, n_pop) / k)");
  {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return accept_fail(MOREA_EDEVICE, hipGetErrorString(e));
  }
  hipLaunchKernelGGL(accept::k_select, dim3(1), dim3(accept::kSelThreads), 0, static_cast<hipStream_t>(stream),
                     n_pop, static_cast<int>(s), k, guidance_max, obj, flags, severity, selection, n_selected, clu_off,
                     clu_members, cluster_of);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    char buf[256];
    snprintf(buf, sizeof(buf), "selection kernel: %s", hipGetErrorString(e));
    set_error(buf);
    return MOREA_EDEVICE;
  }
  return MOREA_OK;
}

extern "C" morea_status morea_accept_partial(morea_problem* p, float* parent_pts, int32_t n_parents,
                                             void* parent_cache, int32_t n_evals, const int32_t* eval_parent,
                                             const int32_t* eval_group, const float* new_coords,
                                             const float* child_obj, const uint8_t* child_flags,
                                             const float* child_sev, float* parent_obj, uint8_t* parent_flags,
                                             float* parent_sev, uint32_t* parent_counts, const float* archive_obj,
                                             int32_t n_archive, float guidance_max, uint8_t* accepted,
                                             void* stream) {
  if (!p) return accept_fail(MOREA_EINVAL, "problem is NULL");
  if (n_evals < 0 || n_parents < 1 || n_archive < 0)
    return accept_fail(MOREA_EINVAL, "need n_evals >= 0, n_parents >= 1, n_archive >= 0");
  if (isnan(guidance_max)) return accept_fail(MOREA_EINVAL, "guidance_max is NaN");
  if (n_evals == 0) return MOREA_OK;
  if (!parent_pts || !parent_cache || !eval_parent || !eval_group || !new_coords || !child_obj || !child_flags ||
      !child_sev || !parent_obj || !parent_flags || !parent_sev || !parent_counts || !accepted ||
      (n_archive > 0 && !archive_obj))
    return accept_fail(MOREA_EINVAL, "NULL argument");
  if (reinterpret_cast<uintptr_t>(parent_cache) % 16 != 0)
    return accept_fail(MOREA_EINVAL, "parent_cache must be 16-byte aligned");
  // the records and offsets of the partial evaluation live in the library's
  // workspace: they must be those of this evaluation list
  const void* key[5] = {parent_pts, parent_cache, eval_parent, eval_group, new_coords};
  if (!p->last_partial || memcmp(key, p->last_key, sizeof(key)) != 0 || p->last_n[0] != n_parents ||
      p->last_n[1] != n_evals)
    return accept_fail(MOREA_ESTATE, "acceptance must follow morea_eval_partial of the same evaluations");
  {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return accept_fail(MOREA_EDEVICE, hipGetErrorString(e));
  }
  const ProblemView& P = p->view;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(accept::k_decide, dim3((n_evals + accept::kBlock - 1) / accept::kBlock), dim3(accept::kBlock),
                     0, s, n_evals, n_parents, p->n_groups, eval_parent, eval_group, child_obj, child_flags,
                     child_sev, parent_obj, parent_flags, parent_sev, archive_obj, n_archive, guidance_max, accepted);
  Record* rec = static_cast<Record*>(parent_cache);
  Totals* tot = reinterpret_cast<Totals*>(static_cast<char*>(parent_cache) +
                                          static_cast<size_t>(n_parents) * P.n_tets * 2 * sizeof(Record));
  constexpr int per_block = accept::kBlock / kWave;
  hipLaunchKernelGGL(accept::k_write_back, dim3((n_evals + per_block - 1) / per_block), dim3(accept::kBlock), 0, s,
                     n_evals, n_parents, p->n_groups, P.n_points, P.n_tets, eval_parent, eval_group, accepted,
                     p->d_row_off, p->d_item_off, p->d_grp_off, p->d_grp_pts, p->d_dep_off, p->d_dep_tet,
                     new_coords, reinterpret_cast<const uint4*>(p->d_partial_records), parent_pts,
                     reinterpret_cast<uint4*>(rec));
  hipError_t e = hipGetLastError();
  if (e == hipSuccess)
    e = launch_finalize(P, parent_pts, n_parents, rec, parent_obj, parent_flags, parent_sev, parent_counts, tot, s);
  if (e != hipSuccess) {
    char buf[256];
    snprintf(buf, sizeof(buf), "acceptance kernels: %s", hipGetErrorString(e));
    set_error(buf);
    return MOREA_EDEVICE;
  }
  return MOREA_OK;
}
