// Elitist archive of the optimizer (Sec. 3: non-dominated solutions kept
// across generations in an archive of fixed capacity, 2000 in App. C's
// parameter listing; Sec. 4.3.2: with adaptive steering on, only guidance
// values up to 1.5 times the archive's best are kept, which purges the
// archive when steering starts) and the adaptation of the distribution
// multipliers of optimal mixing.
//
// Definitions where the paper defers to its references on elitist archiving
// and on MO-RV-GOMEA:
//   members are feasible solutions (valid, no fold, finite objectives and
//     severity) in slots; each carries an insertion stamp that orders them;
//     a free slot has stamp -1 and the objective vector (inf, inf, inf),
//     which dominates nothing, so the acceptance may read every slot;
//   an update's candidates are the members in stamp order, then the feasible
//     offers in index order, less every candidate whose guidance value is
//     above the steering bound; a candidate stays unless another candidate
//     Pareto-dominates it or an earlier one has the same objective vector;
//   above capacity the stayers are thinned by boxes: per objective the range
//     [lo, hi] of the stayers is cut into L equal boxes (FP64, contraction
//     off: box = min(L - 1, floor(((v - lo) / (hi - lo)) * L)), 0 where
//     hi == lo); L is found by a binary search over [1, min(capacity, 1024)]
//     for a resolution whose occupied boxes number at most the capacity, and
//     each occupied box keeps its earliest candidate;
//   members that do not stay free their slots; staying offers fill the free
//     slots in ascending slot order, in offer order, with the next stamps;
//   distribution multipliers (adaptive variance scaling, reduced): a
//     (cluster, element) improves in a generation when a kept child sampled
//     from it belongs to a parent that then entered the archive; on
//     improvement the no-improvement stretch resets and c = max(c, 1) / 0.9
//     (at most 10); otherwise, when c <= 1 the stretch grows, and when c > 1
//     or the stretch has reached 25, c = 0.9 c; a c below 1 whose stretch is
//     under 25 is reset to 1.
//
// The update is two kernels.  The domination tests (members against the
// offers, since members are mutually non-dominated and distinct; offers
// against every candidate) take one wave per candidate over the whole chip
// and leave their verdicts in the archive itself: a member that does not stay
// has its stamp replaced by kGone, an offer's verdict goes to `inserted`.
// Then one block of 1,024 threads, a candidate's values in its thread's
// registers, counts the boxes of each resolution in a hash table in LDS (the
// number of different keys does not depend on the order of insertion; the
// earliest candidate of a box is the smallest order value written to its
// entry, a member's stamp and slot or, above all stamps, the offer's index:
// no two alike, whatever the caller's stamps) and hands out the slots by block
// prefixes.
#include <math.h>
#include <stdio.h>

#include "morea_internal.h"

namespace morea {
namespace archive {

constexpr int kThreads = 1024;
constexpr int kMax = 4096;                 // members + offers per update
constexpr int kPer = kMax / kThreads;      // slots per thread
constexpr int kMaxLevels = 1024;           // boxes per objective (10-bit fields of a key)
constexpr uint32_t kNoKey = 0xffffffffu;
constexpr int kGone = INT32_MIN;           // stamp of a member that leaves, between the two kernels
constexpr int kTable = 8192;               // hash entries: at most half full
constexpr int kChunk = 8;                  // 64-candidate loads in flight per wave

// without branches, so that the loads behind the arguments go out together
__device__ __forceinline__ bool pareto(float a0, float a1, float a2, float b0, float b1, float b2) {
  return (a0 <= b0) & (a1 <= b1) & (a2 <= b2) & ((a0 < b0) | (a1 < b1) | (a2 < b2));
}

struct Shared {
  uint32_t key[kTable];              // box keys present
  unsigned long long order[kTable];  // smallest order value of the box
  int free_slot[kMax];       // free slots in ascending order
  int wsum[kThreads / 64];
  float wmin[kThreads / 64];
  float wmax[kThreads / 64];
};

// Exclusive prefix over the block of one value per thread; *total gets the sum.
__device__ int block_excl(Shared& S, int v, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) S.wsum[w] = x;
  __syncthreads();
  int before = 0, all = 0;
  for (int k = 0; k < kThreads / 64; k++) {
    const int s = S.wsum[k];
    before += k < w ? s : 0;
    all += s;
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

__device__ float block_min(Shared& S, float v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = fminf(v, __shfl_xor(v, d, 64));
  if ((threadIdx.x & 63) == 0) S.wmin[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = INFINITY;
  for (int k = 0; k < kThreads / 64; k++) r = fminf(r, S.wmin[k]);
  __syncthreads();
  return r;
}

__device__ float block_max(Shared& S, float v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
  if ((threadIdx.x & 63) == 0) S.wmax[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = -INFINITY;
  for (int k = 0; k < kThreads / 64; k++) r = fmaxf(r, S.wmax[k]);
  __syncthreads();
  return r;
}

// Box along one axis of a value at the fraction t of the range.
__device__ __forceinline__ int box_of(double t, int L) {
#pragma clang fp contract(off)
  const int b = static_cast<int>(floor(t * static_cast<double>(L)));
  return b < L - 1 ? b : L - 1;
}

struct Offers {
  const float* obj;
  const uint8_t* flags;
  const float* sev;
  int n;
};

__device__ __forceinline__ bool feasible(const float b[3], unsigned flags, float sev) {
  const bool f0 = isfinite(b[0]), f1 = isfinite(b[1]), f2 = isfinite(b[2]), fs = isfinite(sev);
  return (flags == 0) & f0 & f1 & f2 & fs;
}

// Verdicts of the domination tests, one wave per candidate: slots 0 .. cap - 1,
// then the offers.  Bound: latency (the arrays were written on another XCD, so
// the first reads miss its L2; a wave has 8 x 64 candidates in flight);
// capacity 2000 and 512 offers: 9 us on the whole chip (16 us when each
// step's tests waited for a flag byte), most of the 415 us that the one block
// took which did it before.
__global__ __launch_bounds__(256) void k_dominate(Offers F, float gmax, int cap, const float* arc_obj,
                                                int* arc_stamp, uint8_t* inserted) {
  const int x = __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x * 4 + (threadIdx.x >> 6)));
  const int lane = threadIdx.x & 63;
  if (x >= cap + F.n) return;
  const int me = x - cap;                                  // offer index, negative for a member
  float a[3];
  bool ok;
  if (me < 0) {
    if (arc_stamp[x] < 0) return;
    for (int o = 0; o < 3; o++) a[o] = arc_obj[3 * x + o];
    ok = !(a[2] > gmax);
  } else {
    for (int o = 0; o < 3; o++) a[o] = F.obj[3 * me + o];
    ok = feasible(a, F.flags[me], F.sev[me]) && !(a[2] > gmax);
    for (int y0 = 0; y0 < cap && ok; y0 += 64 * kChunk) {
      bool beaten = false;
#pragma unroll
      for (int q = 0; q < kChunk; q++) {
        const int y = min(y0 + 64 * q + lane, cap - 1);     // a slot read twice changes nothing
        const int st = arc_stamp[y];
        const float b0 = arc_obj[3 * y], b1 = arc_obj[3 * y + 1], b2 = arc_obj[3 * y + 2];
        // a member marked as gone meanwhile is a candidate all the same
        const bool par = pareto(b0, b1, b2, a[0], a[1], a[2]);
        const bool twin = (b0 == a[0]) & (b1 == a[1]) & (b2 == a[2]);
        beaten |= ((st >= 0) | (st == kGone)) & !(b2 > gmax) & (par | twin);
      }
      ok = __ballot(beaten) == 0;
    }
  }
  for (int y0 = 0; y0 < F.n && ok; y0 += 64 * kChunk) {
    bool beaten = false;
    float b[kChunk][3], sv[kChunk];
    unsigned fl[kChunk];
#pragma unroll
    for (int q = 0; q < kChunk; q++) {     // every load of the step before the first test
      const int y = min(y0 + 64 * q + lane, F.n - 1);
      for (int o = 0; o < 3; o++) b[q][o] = F.obj[3 * y + o];
      sv[q] = F.sev[y];
      fl[q] = F.flags[y];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < kChunk; q++) {
      const int y = min(y0 + 64 * q + lane, F.n - 1);
      const bool feas = feasible(b[q], fl[q], sv[q]), par = pareto(b[q][0], b[q][1], b[q][2], a[0], a[1], a[2]);
      const bool twin = (y < me) & (b[q][0] == a[0]) & (b[q][1] == a[1]) & (b[q][2] == a[2]);
      beaten |= feas & (y != me) & !(b[q][2] > gmax) & (par | twin);
    }
    ok = __ballot(beaten) == 0;
  }
  if (lane != 0) return;
  if (me >= 0)
    inserted[me] = ok ? 1 : 0;
  else if (!ok)
    arc_stamp[x] = kGone;
}

// Entry of `key`, inserted when it is new (*fresh counts insertions).
__device__ __forceinline__ int table_entry(Shared& S, uint32_t key, int* fresh) {
  int h = static_cast<int>((key * 2654435761u) >> 19);
  static_assert(kTable == 1 << 13, "hash width");
  for (;;) {
    const uint32_t old = atomicCAS(&S.key[h], kNoKey, key);
    if (old == kNoKey) *fresh += 1;
    if (old == kNoKey || old == key) return h;
    h = (h + 1) & (kTable - 1);
  }
}

// Thinning and slots.  One block: 11 passes over the box resolutions when
// the capacity is exceeded (a pass is a cleared table and one insertion a
// stayer instead of a bitonic sort of 78 steps), otherwise four prefixes, 6 us.
__global__ __launch_bounds__(kThreads) void k_update(int n_off, const float* __restrict__ offer_obj, int cap,
                                                     float* __restrict__ arc_obj, int* __restrict__ arc_stamp,
                                                     int* __restrict__ arc_state, float* __restrict__ best_out,
                                                     uint8_t* __restrict__ inserted, int* __restrict__ slot_of) {
  __shared__ Shared S;
  const int t = threadIdx.x;
  const int next = arc_state[1];
  // candidates of this thread: slots t, t + 1024, .. and offer t
  bool held[kPer], stay[kPer + 1];
  float v[kPer + 1][3];
  unsigned long long order[kPer + 1];
  int n_mine = 0;
#pragma unroll
  for (int j = 0; j < kPer; j++) {
    const int s = t + j * kThreads;
    const int st = s < cap ? arc_stamp[s] : -1;
    held[j] = st >= 0 || st == kGone;
    stay[j] = st >= 0;
    order[j] = static_cast<unsigned long long>(static_cast<uint32_t>(st)) << 32 | static_cast<uint32_t>(s);
#pragma unroll
    for (int o = 0; o < 3; o++) v[j][o] = stay[j] ? arc_obj[3 * s + o] : 0.f;
  }
  stay[kPer] = t < n_off && inserted[t] != 0;
  order[kPer] = (0x80000000ull + t) << 32;      // after every member
#pragma unroll
  for (int o = 0; o < 3; o++) v[kPer][o] = stay[kPer] ? offer_obj[3 * t + o] : 0.f;
#pragma unroll
  for (int j = 0; j <= kPer; j++) n_mine += stay[j] ? 1 : 0;
  int n_stay;
  block_excl(S, n_mine, &n_stay);
  // ---- thinning by boxes above capacity
  int levels = 0;
  if (n_stay > cap) {
    double at[kPer + 1][3];     // place in the stayers' range, per objective
#pragma unroll
    for (int o = 0; o < 3; o++) {
      float mn = INFINITY, mx = -INFINITY;
#pragma unroll
      for (int j = 0; j <= kPer; j++) {
        mn = stay[j] ? fminf(mn, v[j][o]) : mn;
        mx = stay[j] ? fmaxf(mx, v[j][o]) : mx;
      }
      const double lo = block_min(S, mn), hi = block_max(S, mx);
#pragma unroll
      for (int j = 0; j <= kPer; j++) at[j][o] = hi > lo ? (static_cast<double>(v[j][o]) - lo) / (hi - lo) : 0.0;
    }
    int a = 1, b = cap < kMaxLevels ? cap : kMaxLevels;
    // the last pass (a == b) takes the boxes' earliest candidates
    for (;;) {
      const int L = a < b ? (a + b + 1) / 2 : a;
#pragma unroll
      for (int q = 0; q < kTable / kThreads; q++) {
        S.key[t + q * kThreads] = kNoKey;
        if (a == b) S.order[t + q * kThreads] = ~0ull;
      }
      __syncthreads();
      int fresh = 0, entry[kPer + 1];
#pragma unroll
      for (int j = 0; j <= kPer; j++) {
        entry[j] = 0;
        if (!stay[j]) continue;
        const uint32_t key = static_cast<uint32_t>(box_of(at[j][0], L)) |
                             static_cast<uint32_t>(box_of(at[j][1], L)) << 10 |
                             static_cast<uint32_t>(box_of(at[j][2], L)) << 20;
        entry[j] = table_entry(S, key, &fresh);
        if (a == b) atomicMin(&S.order[entry[j]], order[j]);
      }
      int cnt;
      block_excl(S, fresh, &cnt);    // its barriers also end the table's use
      if (a == b) {
        levels = a;
        n_mine = 0;
#pragma unroll
        for (int j = 0; j <= kPer; j++) {
          stay[j] = stay[j] && S.order[entry[j]] == order[j];
          n_mine += stay[j] ? 1 : 0;
        }
        break;
      }
      if (cnt <= cap) a = L;
      else b = L - 1;
    }
    block_excl(S, n_mine, &n_stay);
  }
  // ---- members that do not stay free their slots; the free slots in order
  int n_free = 0;
#pragma unroll
  for (int j = 0; j < kPer; j++) {
    const int s = t + j * kThreads;
    if (held[j] && !stay[j]) {
      arc_stamp[s] = -1;
      arc_obj[3 * s] = INFINITY;
      arc_obj[3 * s + 1] = INFINITY;
      arc_obj[3 * s + 2] = INFINITY;
    }
    if (j * kThreads >= cap) continue;          // uniform: no slots in this pass
    const bool is_free = s < cap && !stay[j];
    int cnt;
    const int r = n_free + block_excl(S, is_free ? 1 : 0, &cnt);
    if (is_free) S.free_slot[r] = s;
    n_free += cnt;
  }
  // ---- staying offers take them in index order
  int n_new;
  const int r = block_excl(S, stay[kPer] ? 1 : 0, &n_new);   // its barriers publish the free slots
  if (t < n_off) {
    int slot = -1;
    if (stay[kPer]) {
      slot = S.free_slot[r];
      arc_obj[3 * slot] = v[kPer][0];
      arc_obj[3 * slot + 1] = v[kPer][1];
      arc_obj[3 * slot + 2] = v[kPer][2];
      arc_stamp[slot] = next + r;
    }
    inserted[t] = stay[kPer] ? 1 : 0;
    slot_of[t] = slot;
  }
  // best guidance among the members after the update
  float g = INFINITY;
#pragma unroll
  for (int j = 0; j <= kPer; j++) g = stay[j] ? fminf(g, v[j][2]) : g;
  g = block_min(S, g);
  if (t == 0) {
    arc_state[0] = n_stay;
    arc_state[1] = next + n_new;
    arc_state[2] = levels;
    arc_state[3] = 0;
    best_out[0] = g;
  }
}

// Points of the offers that entered the archive, into their slots.
__global__ void k_copy_points(int n_off, int per, const float* __restrict__ offer_pts,
                              const int* __restrict__ slot_of, float* __restrict__ arc_pts) {
  const int i = blockIdx.x;
  const int s = slot_of[i];
  if (s < 0) return;
  const float* src = offer_pts + static_cast<size_t>(i) * per;
  float* dst = arc_pts + static_cast<size_t>(s) * per;
  for (int q = threadIdx.x; q < per; q += blockDim.x) dst[q] = src[q];
}

__global__ void k_clear(int cap, float* __restrict__ arc_obj, int* __restrict__ arc_stamp,
                        int* __restrict__ arc_state, float* __restrict__ best_out) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < cap) {
    arc_stamp[s] = -1;
    arc_obj[3 * s] = INFINITY;
    arc_obj[3 * s + 1] = INFINITY;
    arc_obj[3 * s + 2] = INFINITY;
  }
  if (s < 4) arc_state[s] = 0;
  if (s == 0) best_out[0] = INFINITY;
}

// Improvements of one batch: a kept child whose parent entered the archive
// marks its (cluster, element).
__global__ void k_mark(int n_evals, int n_parents, int n_clusters, int n_groups, const int* __restrict__ eval_parent,
                       const int* __restrict__ eval_group, const int* __restrict__ eval_cluster,
                       const uint8_t* __restrict__ accepted, const uint8_t* __restrict__ parent_inserted,
                       uint8_t* __restrict__ improved) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_evals || !accepted[e]) return;
  const int p = eval_parent[e], g = eval_group[e], c = eval_cluster[e];
  if (p < 0 || p >= n_parents || g < 0 || g >= n_groups || c < 0 || c >= n_clusters) return;
  if (parent_inserted[p]) improved[static_cast<size_t>(c) * n_groups + g] = 1;
}

__global__ void k_adapt(int n, uint8_t* __restrict__ improved, float* __restrict__ mult, int* __restrict__ nis) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  float c = mult[q];
  int s = nis[q];
  if (improved[q]) {
    s = 0;
    c = fminf(fmaxf(c, 1.f) / 0.9f, 10.f);
  } else {
    if (c <= 1.f) s += 1;
    if (c > 1.f || s >= 25) c = 0.9f * c;
    else if (c < 1.f) c = 1.f;
  }
  mult[q] = c;
  nis[q] = s;
  improved[q] = 0;
}

}  // namespace archive
}  // namespace morea

using namespace morea;

namespace {

morea_status arc_fail(morea_status code, const char* msg) {
  set_error(msg);
  return code;
}

morea_status arc_launched(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return MOREA_OK;
  char buf[256];
  snprintf(buf, sizeof(buf), "%s: %s", what, hipGetErrorString(e));
  set_error(buf);
  return MOREA_EDEVICE;
}

morea_status arc_pending() {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return MOREA_OK;
  set_error(hipGetErrorString(e));
  return MOREA_EDEVICE;
}

}  // namespace

extern "C" morea_status morea_archive_clear(int32_t capacity, float* arc_obj, int32_t* arc_stamp,
                                            int32_t* arc_state, float* best_guidance, void* stream) {
  if (capacity < 1 || capacity > archive::kMax) return arc_fail(MOREA_EINVAL, "need 1 <= capacity <= 4096");
  if (!arc_obj || !arc_stamp || !arc_state || !best_guidance) return arc_fail(MOREA_EINVAL, "NULL argument");
  if (morea_status st = arc_pending()) return st;
  hipLaunchKernelGGL(archive::k_clear, dim3((capacity + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream),
                     capacity, arc_obj, arc_stamp, arc_state, best_guidance);
  return arc_launched("archive clear kernel");
}

extern "C" morea_status morea_archive_update(int32_t n_offers, const float* offer_obj, const uint8_t* offer_flags,
                                             const float* offer_sev, const float* offer_pts, int32_t n_points,
                                             float guidance_max, int32_t capacity, float* arc_obj,
                                             int32_t* arc_stamp, float* arc_pts, int32_t* arc_state,
                                             float* best_guidance, uint8_t* inserted, int32_t* slot_of,
                                             void* stream) {
  if (capacity < 1 || n_offers < 0 || n_offers > archive::kThreads ||
      static_cast<int64_t>(capacity) + n_offers > archive::kMax)
    return arc_fail(MOREA_ERANGE, "need capacity >= 1, 0 <= n_offers <= 1024, capacity + n_offers <= 4096");
  if (isnan(guidance_max)) return arc_fail(MOREA_EINVAL, "guidance_max is NaN");
  if (!arc_obj || !arc_stamp || !arc_state || !best_guidance || (n_offers > 0 && (!offer_obj || !offer_flags ||
      !offer_sev || !inserted || !slot_of)))
    return arc_fail(MOREA_EINVAL, "NULL argument");
  if ((offer_pts == nullptr) != (arc_pts == nullptr) || (arc_pts && n_points < 1))
    return arc_fail(MOREA_EINVAL, "offer_pts and arc_pts: both NULL, or both set with n_points >= 1");
  if (morea_status st = arc_pending()) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // slot_of is needed by the point copy even when the caller does not want it
  const archive::Offers offers{offer_obj, offer_flags, offer_sev, n_offers};
  hipLaunchKernelGGL(archive::k_dominate, dim3((capacity + n_offers + 3) / 4), dim3(256), 0, s, offers, guidance_max,
                     capacity, arc_obj, arc_stamp, inserted);
  hipLaunchKernelGGL(archive::k_update, dim3(1), dim3(archive::kThreads), 0, s, n_offers, offer_obj, capacity,
                     arc_obj, arc_stamp, arc_state, best_guidance, inserted, slot_of);
  if (morea_status st = arc_launched("archive update kernel")) return st;
  if (arc_pts && n_offers > 0) {
    hipLaunchKernelGGL(archive::k_copy_points, dim3(n_offers), dim3(256), 0, s, n_offers, 6 * n_points, offer_pts,
                       slot_of, arc_pts);
    return arc_launched("archive point copy kernel");
  }
  return MOREA_OK;
}

extern "C" morea_status morea_mark_improvements(int32_t n_evals, const int32_t* eval_parent,
                                                const int32_t* eval_group, const int32_t* eval_cluster,
                                                const uint8_t* accepted, int32_t n_parents,
                                                const uint8_t* parent_inserted, int32_t n_clusters,
                                                int32_t n_groups, uint8_t* improved, void* stream) {
  if (n_evals < 0 || n_parents < 1 || n_clusters < 1 || n_groups < 1)
    return arc_fail(MOREA_EINVAL, "need n_evals >= 0 and n_parents, n_clusters, n_groups >= 1");
  if (n_evals == 0) return MOREA_OK;
  if (!eval_parent || !eval_group || !eval_cluster || !accepted || !parent_inserted || !improved)
    return arc_fail(MOREA_EINVAL, "NULL argument");
  if (morea_status st = arc_pending()) return st;
  hipLaunchKernelGGL(archive::k_mark, dim3((n_evals + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream),
                     n_evals, n_parents, n_clusters, n_groups, eval_parent, eval_group, eval_cluster, accepted,
                     parent_inserted, improved);
  return arc_launched("improvement marking kernel");
}

extern "C" morea_status morea_adapt_multipliers(int32_t n_clusters, int32_t n_groups, uint8_t* improved,
                                                float* mult, int32_t* no_improvement, void* stream) {
  if (n_clusters < 1 || n_groups < 1) return arc_fail(MOREA_EINVAL, "need n_clusters, n_groups >= 1");
  if (!improved || !mult || !no_improvement) return arc_fail(MOREA_EINVAL, "NULL argument");
  if (morea_status st = arc_pending()) return st;
  const int n = n_clusters * n_groups;
  hipLaunchKernelGGL(archive::k_adapt, dim3((n + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream), n,
                     improved, mult, no_improvement);
  return arc_launched("multiplier adaptation kernel");
}
