// Deformation vector fields of one candidate, rasterized from its two meshes
// (Sec. 5.4 compares registrations through a forward DVF on the source grid
// and an inverse DVF on the target grid).  A voxel centre p of tet t of the
// sampled mesh (the centres of the evaluation: exact signed volumes, a centre
// on a face belonging to the tet that holds p + (e, e^2, e^3)) gets q - p,
// q its barycentric image in the other mesh.  A centre covered by several
// tets (a folded mesh) takes the tet of smallest index, a centre covered by
// none the displacement 0; a tet with a vertex coordinate that is not finite
// or has |x| >= 512 voxels is skipped.
//
// One pass over the (direction, tet) pairs: 64 rows of the tet's box at a
// time, one per lane, whose x-intervals are solved exactly from the four face
// planes; the voxels of the rows then go to the lanes in order.  Every
// covering tet lowers the centre's owner to its index, counts itself when it
// is not the first, and writes its displacement; where a centre is covered
// once that is the result, and a last pass over the voxels completes the
// counts and writes the others (0 for a centre in no tet, the owner's
// displacement for one in several).  The displacement is the FP64
// barycentric image rounded once to FP32.
//
// The same exact point location gives the point-based guidance error of the
// paper's prior work, which Sec. 4.1.3 replaces by the continuous form: every
// point c of C_s is located in the source mesh (smallest tet index if
// several), mapped to the target mesh through its barycentric coordinates,
// and its squared distance to the nearest point of the set's C_t taken; the
// value is the mean over all points of all sets (sets weighted |C_i| / |G|);
// points in no tet are left out and counted.
#include <math.h>
#include <stdio.h>

#include <algorithm>
#include <mutex>

#include "morea_internal.h"
#include "morea_raster.h"

namespace morea {
namespace dvf {

typedef __int128 i128;

__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 6 x signed volume (exact in 128 bits for any coordinates below 2^21)
__device__ __forceinline__ i128 vol6(const int64_t a[3], const int64_t b[3], const int64_t c[3], const int64_t d[3]) {
  const i128 u0 = b[0] - a[0], u1 = b[1] - a[1], u2 = b[2] - a[2];
  const i128 v0 = c[0] - a[0], v1 = c[1] - a[1], v2 = c[2] - a[2];
  const i128 w0 = d[0] - a[0], w1 = d[1] - a[1], w2 = d[2] - a[2];
  return u0 * (v1 * w2 - v2 * w1) - u1 * (v0 * w2 - v2 * w0) + u2 * (v0 * w1 - v1 * w0);
}

// Face value of vertex i (the volume with vertex i replaced by p), oriented
// positive inside.
__device__ __forceinline__ i128 face(const int64_t v[4][3], int i, const int64_t p[3], int sgn) {
  const int64_t* q0 = i == 0 ? p : v[0];
  const int64_t* q1 = i == 1 ? p : v[1];
  const int64_t* q2 = i == 2 ? p : v[2];
  const int64_t* q3 = i == 3 ? p : v[3];
  const i128 s = vol6(q0, q1, q2, q3);
  return sgn > 0 ? s : -s;
}

// Inside test with the tie rule: on a face plane the sign of the face value
// at p + (e, e^2, e^3) decides, i.e. the first nonzero component of its
// gradient (the change for a unit step along x, then y, then z).
__device__ __forceinline__ bool inside(const int64_t v[4][3], int sgn, const int64_t p[3], i128 val[4]) {
  bool in = true;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    val[i] = face(v, i, p, sgn);
    if (val[i] < 0) in = false;
  }
  if (!in) return false;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    if (val[i] != 0) continue;
    int sgrad = 0;
    for (int k = 0; k < 3 && sgrad == 0; k++) {
      int64_t pk[3] = {p[0], p[1], p[2]};
      pk[k] += 1;
      const i128 g = face(v, i, pk, sgn) - val[i];
      sgrad = (g > 0) - (g < 0);
    }
    if (sgrad <= 0) return false;
  }
  return true;
}

constexpr int kNoOwner = 0x7fffffff;
constexpr int kClearPer = 4;   // voxels per thread, a block's width apart

__global__ __launch_bounds__(256) void k_dvf_clear(size_t n, int* owner, uint32_t* cover) {
  const size_t first = static_cast<size_t>(blockIdx.x) * (256 * kClearPer) + threadIdx.x;
#pragma unroll
  for (int q = 0; q < kClearPer; q++) {
    const size_t i = first + 256 * q;
    if (i < n) {
      owner[i] = kNoOwner;
      cover[i] = 0u;
    }
  }
}

// Face planes of a tet about the box corner lo: for voxel lo + (j, y, z) the
// value s_i = A_i j + PY_i y + PZ_i z + B_i is 6 |V| times the barycentric
// coordinate of vertex i, an exact integer; T is double for extents up to
// 2^16 units (every sum below 2^53) and int64 otherwise.  lex_i: a centre on
// face i belongs to the tet (the first nonzero component of the inward normal
// is positive).
template <typename T>
struct Planes {
  T A[4], PY[4], PZ[4], B[4];
  int lex[4];
};

template <typename T>
__device__ __forceinline__ Planes<T> tet_planes(const int own[4][3], const int lo[3], int sgn) {
  Planes<T> P;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int b = i == 0 ? 1 : 0, u0 = i == 0 ? 2 : (i == 1 ? 2 : (i == 2 ? 3 : 1)),
              w0 = i == 0 ? 3 : (i == 1 ? 3 : (i == 2 ? 1 : 2));
    T u[3], w[3], o[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
      u[k] = static_cast<T>(own[u0][k] - own[b][k]);
      w[k] = static_cast<T>(own[w0][k] - own[b][k]);
      o[k] = static_cast<T>(1024 * lo[k] - own[b][k]);
    }
    const T f = static_cast<T>(i == 0 ? -sgn : sgn);
    const T x = f * (u[1] * w[2] - u[2] * w[1]), y = f * (u[2] * w[0] - u[0] * w[2]),
            z = f * (u[0] * w[1] - u[1] * w[0]);
    P.lex[i] = (x > 0 || (x == 0 && (y > 0 || (y == 0 && z > 0)))) ? 1 : 0;
    P.A[i] = x * 1024;
    P.PY[i] = y * 1024;
    P.PZ[i] = z * 1024;
    P.B[i] = x * o[0] + y * o[1] + z * o[2];
  }
  return P;
}

// Snapped vertices of tet t in the sampled mesh d and in the other one;
// false when a coordinate is invalid.
__device__ __forceinline__ bool load_tet(const ProblemView& P, const float* cand, int d, int t, int own[4][3],
                                         int oth[4][3]) {
  const int4 tv = P.tets[t];
  const int vs[4] = {tv.x, tv.y, tv.z, tv.w};
  bool ok = true;
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int k = 0; k < 3; k++) {
      const float x = cand[(d * 3 + k) * P.n_points + vs[i]], y = cand[((1 - d) * 3 + k) * P.n_points + vs[i]];
      const bool fine = fabsf(x) < kCoordLimit && fabsf(y) < kCoordLimit;
      ok = ok && fine;
      own[i][k] = fine ? static_cast<int>(rintf(x * kFixOne)) : 0;
      oth[i][k] = fine ? static_cast<int>(rintf(y * kFixOne)) : 0;
    }
  return ok;
}

__device__ __forceinline__ int64_t det6(const int v[4][3]) {   // |coordinates| < 2^19: below 2^63
  const int64_t a0 = v[1][0] - v[0][0], a1 = v[1][1] - v[0][1], a2 = v[1][2] - v[0][2];
  const int64_t b0 = v[2][0] - v[0][0], b1 = v[2][1] - v[0][1], b2 = v[2][2] - v[0][2];
  const int64_t c0 = v[3][0] - v[0][0], c1 = v[3][1] - v[0][1], c2 = v[3][2] - v[0][2];
  return a0 * (b1 * c2 - b2 * c1) - a1 * (b0 * c2 - b2 * c0) + a2 * (b0 * c1 - b1 * c0);
}

// Displacement of a voxel from the face values of vertices 1..3 there.
__device__ __forceinline__ void displacement(const double val[3], double inv_absD, const int oth[4][3],
                                             const int pv[3], float out[3]) {
#pragma unroll
  for (int a = 0; a < 3; a++) {
    double q = static_cast<double>(oth[0][a]);
#pragma unroll
    for (int i = 0; i < 3; i++) q += val[i] * inv_absD * static_cast<double>(oth[i + 1][a] - oth[0][a]);
    out[a] = static_cast<float>(q * (1.0 / 1024.0) - pv[a]);
  }
}

struct __attribute__((aligned(4))) F3 {
  float v[3];
};

// Rows [64 (part + k parts), ..) of a tet's box.  `mark` is 64 words of LDS
// of the wave.
template <typename T>
__device__ __forceinline__ void raster_rows(const ProblemView& P, const int own[4][3], const int oth[4][3], int t,
                                            int64_t D, const int lo[3], const int ext[3], int part, int parts,
                                            int* mark, int* owner, uint32_t* cover, float* out) {
  const int lane = lane_id();
  const Planes<T> pl = tet_planes<T>(own, lo, D > 0 ? 1 : -1);
  const double inv_absD = 1.0 / static_cast<double>(D > 0 ? D : -D);
  double invA[4];
  int kind[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    kind[i] = (pl.A[i] > 0) - (pl.A[i] < 0);
    // an estimate (clip_face corrects the row's end by the exact value)
    const double a = static_cast<double>(pl.A[i]), r = __builtin_amdgcn_rcp(a);
    invA[i] = kind[i] != 0 ? fma(fma(-a, r, 1.0), r, r) : 0.0;
  }
  const int rows = ext[1] * ext[2];
  int tag = 0;
  for (int rb = 64 * part; rb < rows; rb += 64 * parts) {
    const int r = rb + lane, zr = r / ext[1], yr = r - zr * ext[1];
    int js = 0, je = r < rows ? ext[0] - 1 : -1;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const T b = pl.PY[i] * yr + pl.PZ[i] * zr + pl.B[i] + pl.lex[i];
      clip_face<T>(kind[i], pl.A[i], invA[i], b, ext[0] - 1, js, je);
    }
    const int len = max(0, je - js + 1);
    // the voxels of the 64 rows form one stream; `at` is the row's first
    int at = len;
    at += __builtin_amdgcn_update_dpp(0, at, 0x111, 0xf, 0xf, false);   // within rows of 16 lanes: shifts by 1, 2,
    at += __builtin_amdgcn_update_dpp(0, at, 0x112, 0xf, 0xf, false);   // 4 and 8
    at += __builtin_amdgcn_update_dpp(0, at, 0x114, 0xf, 0xf, false);
    at += __builtin_amdgcn_update_dpp(0, at, 0x118, 0xf, 0xf, false);
    at += __builtin_amdgcn_update_dpp(0, at, 0x142, 0xa, 0xf, false);   // lane 15 -> rows 1, 3
    at += __builtin_amdgcn_update_dpp(0, at, 0x143, 0xc, 0xf, false);   // lane 31 -> rows 2, 3
    const int total = __builtin_amdgcn_readlane(at, 63);
    at -= len;
    const int packed = js | yr << 10 | zr << 20;
    for (int s = 0; s < total; s += 64) {
      // row of voxel s + lane: the last non-empty one that starts at or
      // before it -- one that starts inside the batch marks its place there
      tag += 64;
      if (len > 0 && at > s && at < s + 64) mark[at - s] = tag + lane;
      const int first = __builtin_ctzll(__ballot(len > 0 && at <= s && at + len > s));
      wave_sync();
      const int mk = mark[lane];
      const uint64_t starts = __ballot(mk >= tag);
      wave_sync();
      const uint64_t upto = starts & (~0ull >> (63 - lane));
      const int src = upto ? 63 - __builtin_clzll(upto) : lane;
      const int marked = __shfl(mk, src, 64) & 63;
      const int row = upto ? marked : first;
      const int u = s + lane, w = __shfl(packed, row, 64), u0 = __shfl(at, row, 64);
      if (u >= total) continue;
      const int j = (w & 1023) + u - u0, y = (w >> 10) & 1023, z = w >> 20;
      double val[3];
#pragma unroll
      for (int i = 0; i < 3; i++)
        val[i] = static_cast<double>(pl.A[i + 1] * j + pl.PY[i + 1] * y + pl.PZ[i + 1] * z + pl.B[i + 1]);
      const int pv[3] = {lo[0] + j, lo[1] + y, lo[2] + z};
      const size_t v = (static_cast<size_t>(pv[2]) * P.ny + pv[1]) * P.nx + pv[0];
      F3 o;
      displacement(val, inv_absD, oth, pv, o.v);
      *reinterpret_cast<F3*>(out + 3 * v) = o;
      if (atomicMin(&owner[v], t) != kNoOwner) atomicAdd(&cover[v], 1u);
    }
  }
}

// One wave per (direction, tet, part of its rows).  Bound: the atomics on the
// owners, one request per row of a tet (128x128x96 voxels, 3,402 tets: 52 us,
// 27 of them without any atomic or store; with the count as a second atomic
// per voxel 72), then a wave's chain of loads, spans and batches.  Testing
// every voxel of the boxes in 128-bit integers, twice, took 536 + 576 us.
__global__ __launch_bounds__(256) void k_dvf(ProblemView P, const float* cand, int parts, int* owner,
                                           uint32_t* cover, float* fwd, float* inv) {
  __shared__ int marks[4][64];
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  marks[wave][lane_id()] = 0;
  const int64_t w = static_cast<int64_t>(blockIdx.x) * 4 + wave;
  const int64_t item = w / parts;
  if (item >= 2 * static_cast<int64_t>(P.n_tets)) return;
  const int part = static_cast<int>(w - item * parts);
  const int d = item >= P.n_tets, t = static_cast<int>(item - (d ? P.n_tets : 0));
  // lane l < 24: mesh (l < 12 ? sampled : other), vertex (l % 12) / 3, axis l % 3
  const int lane = lane_id();
  const int4 tv = P.tets[t];
  float x = 0.f;
  if (lane < 24) {
    const int i = (lane % 12) / 3, k = lane % 3;
    const int pt = i == 0 ? tv.x : (i == 1 ? tv.y : (i == 2 ? tv.z : tv.w));
    const int mesh = lane < 12 ? d : 1 - d;
    x = cand[(mesh * 3 + k) * P.n_points + pt];
  }
  if (__ballot(lane < 24 && !(fabsf(x) < kCoordLimit)) != 0ull) return;
  const int fix = lane < 24 ? static_cast<int>(rintf(x * kFixOne)) : 0;
  int own[4][3], oth[4][3];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int k = 0; k < 3; k++) {
      own[i][k] = __builtin_amdgcn_readlane(fix, 3 * i + k);
      oth[i][k] = __builtin_amdgcn_readlane(fix, 12 + 3 * i + k);
    }
  const int64_t D = det6(own);
  if (D == 0) return;
  const int dims[3] = {P.nx, P.ny, P.nz};
  int lo[3], ext[3], wide = 0;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int mn = min(min(own[0][k], own[1][k]), min(own[2][k], own[3][k]));
    const int mx = max(max(own[0][k], own[1][k]), max(own[2][k], own[3][k]));
    wide = max(wide, mx - mn);
    lo[k] = max((mn + 1023) >> 10, 0);                        // ceil(mn / 1024), floor(mx / 1024)
    ext[k] = min(mx >> 10, dims[k] - 1) - lo[k] + 1;
  }
  if (ext[0] <= 0 || ext[1] <= 0 || ext[2] <= 0) return;
  const size_t V = static_cast<size_t>(P.nx) * P.ny * P.nz;
  int* ow = owner + d * V;
  uint32_t* cv = cover + d * V;
  float* out = d == 0 ? fwd : inv;
  if (wide <= kFastExtent)
    raster_rows<double>(P, own, oth, t, D, lo, ext, part, parts, marks[wave], ow, cv, out);
  else
    raster_rows<long long>(P, own, oth, t, D, lo, ext, part, parts, marks[wave], ow, cv, out);
}

// The counts, and the centres covered by no tet or by several (one thread per
// centre; `cover` holds the covering tets beyond the first).
__global__ __launch_bounds__(256) void k_dvf_rest(ProblemView P, const float* cand, const int* owner,
                                                uint32_t* cover, float* fwd, float* inv) {
  const size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
  const size_t V = static_cast<size_t>(P.nx) * P.ny * P.nz;
  if (i >= 2 * V) return;
  const int t = owner[i];
  const uint32_t c = t == kNoOwner ? 0u : cover[i] + 1u;
  if (c != 0u) cover[i] = c;
  if (c == 1u) return;
  const int d = i >= V;
  const size_t v = i - (d ? V : 0);
  float o[3] = {0.f, 0.f, 0.f};
  if (c > 1u) {
    const int pv[3] = {static_cast<int>(v % P.nx), static_cast<int>(v / P.nx % P.ny),
                       static_cast<int>(v / (static_cast<size_t>(P.nx) * P.ny))};
    int own[4][3], oth[4][3];
    load_tet(P, cand, d, t, own, oth);
    const int64_t D = det6(own);
    const Planes<long long> pl = tet_planes<long long>(own, pv, D > 0 ? 1 : -1);
    const double val[3] = {static_cast<double>(pl.B[1]), static_cast<double>(pl.B[2]),
                           static_cast<double>(pl.B[3])};
    displacement(val, 1.0 / static_cast<double>(D > 0 ? D : -D), oth, pv, o);
  }
  float* out = (d ? inv : fwd) + 3 * v;
  out[0] = o[0];
  out[1] = o[1];
  out[2] = o[2];
}

// Point-based guidance: one block of 4 waves per candidate; wave w takes the
// source guidance points w, w + 4, ... in order and sums their squared
// distances in FP64; the 4 sums are added in wave order.
__global__ __launch_bounds__(256) void k_point_guidance(ProblemView P, const float* pts, const int* off_s,
                                                      const int* fix_s, const int* off_t, const int* fix_t,
                                                      float* f, int* unmapped) {
  extern __shared__ int X[];                 // [2][n][3] snapped coordinates
  __shared__ double wsum[4];
  __shared__ int wcnt[4], wun[4], bad;
  const int n = P.n_points, c = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)), lane = lane_id();
  const float* cp = pts + static_cast<size_t>(c) * 6 * n;
  if (threadIdx.x == 0) bad = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < 6 * n; i += blockDim.x) {
    const int m = i / (3 * n), a = (i / n) % 3, v = i % n;
    const float x = cp[i];
    if (!(fabsf(x) < kCoordLimit)) bad = 1;
    X[(m * n + v) * 3 + a] = fabsf(x) < kCoordLimit ? static_cast<int>(rintf(x * kFixOne)) : 0;
  }
  __syncthreads();
  if (bad) {
    if (threadIdx.x == 0) {
      f[c] = __builtin_nanf("");
      unmapped[c] = 0;
    }
    return;
  }
  const int G = P.n_sets > 0 ? off_s[P.n_sets] : 0;
  double sum = 0.0;
  int cnt = 0, un = 0;
  for (int g = wave; g < G; g += 4) {
    int s = 0;
    while (off_s[s + 1] <= g) s++;
    const int64_t cpt[3] = {fix_s[3 * g], fix_s[3 * g + 1], fix_s[3 * g + 2]};
    // the smallest tet of the source mesh that holds the point
    int hit_t = -1;
    for (int base = 0; base < P.n_tets && hit_t < 0; base += 64) {
      const int t = base + lane;
      bool hit = false;
      if (t < P.n_tets) {
        const int4 tv = P.tets[t];
        const int vi[4] = {tv.x, tv.y, tv.z, tv.w};
        int64_t own[4][3];
        bool in_box = true;
#pragma unroll
        for (int k = 0; k < 3; k++) {
          int64_t mn = INT64_MAX, mx = INT64_MIN;
#pragma unroll
          for (int i = 0; i < 4; i++) {
            own[i][k] = X[3 * vi[i] + k];
            mn = min(mn, own[i][k]);
            mx = max(mx, own[i][k]);
          }
          in_box = in_box && cpt[k] >= mn && cpt[k] <= mx;
        }
        if (in_box) {
          const i128 D = vol6(own[0], own[1], own[2], own[3]);
          i128 val[4];
          hit = D != 0 && inside(own, D > 0 ? 1 : -1, cpt, val);
        }
      }
      const uint64_t m = __ballot(hit);
      if (m != 0ull) hit_t = base + __builtin_ctzll(m);
    }
    if (hit_t < 0) {
      un += 1;
      continue;
    }
    // its image in the target mesh (every lane, the same tet)
    const int4 tv = P.tets[hit_t];
    const int vi[4] = {tv.x, tv.y, tv.z, tv.w};
    int64_t own[4][3], oth[4][3];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int k = 0; k < 3; k++) {
        own[i][k] = X[3 * vi[i] + k];
        oth[i][k] = X[3 * (n + vi[i]) + k];
      }
    const i128 D = vol6(own[0], own[1], own[2], own[3]);
    i128 val[4];
    (void)inside(own, D > 0 ? 1 : -1, cpt, val);
    const double inv_absD = 1.0 / static_cast<double>(D > 0 ? D : -D);
    double q[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
      double qa = static_cast<double>(oth[0][a]);
#pragma unroll
      for (int i = 1; i < 4; i++)
        qa += static_cast<double>(val[i]) * inv_absD * static_cast<double>(oth[i][a] - oth[0][a]);
      q[a] = qa * (1.0 / 1024.0);
    }
    // nearest point of the set's C_t
    double best = INFINITY;
    for (int k = off_t[s] + lane; k < off_t[s + 1]; k += 64) {
      double d2 = 0.0;
#pragma unroll
      for (int a = 0; a < 3; a++) {
        const double diff = q[a] - static_cast<double>(fix_t[3 * k + a]) * (1.0 / 1024.0);
        d2 = fma(diff, diff, d2);
      }
      best = fmin(best, d2);
    }
    for (int dd = 32; dd >= 1; dd >>= 1) best = fmin(best, __shfl_xor(best, dd, 64));
    sum += best;
    cnt += 1;
  }
  if (lane == 0) {
    wsum[wave] = sum;
    wcnt[wave] = cnt;
    wun[wave] = un;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double total = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
    const int nn = wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
    f[c] = nn > 0 ? static_cast<float>(total / nn) : __builtin_nanf("");
    unmapped[c] = wun[0] + wun[1] + wun[2] + wun[3];
  }
}

}  // namespace dvf
}  // namespace morea

using namespace morea;

namespace morea {
namespace dvf {

// Owner workspace of the allocation-free DVF entry point: one int32 per
// voxel centre of both grids, 16 MiB, so grids of at most 2,097,152 voxels.
// Every GPU the library runs on holds its own copy until the process ends;
// calls on one GPU share it (calls that overlap on one GPU race), and every
// call clears the part it uses with a kernel first.
constexpr size_t kScratchInts = static_cast<size_t>(1) << 22;
static __device__ __align__(256) int32_t scratch[kScratchInts];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
int32_t* g_scratch[kMaxDevices] = {};

}  // namespace dvf

// Device address of the scratch array on the current device (looked up once
// per device, with that device current).  The array's name is only a
// host-side stand-in: kernels get this address.
morea_status static_scratch_init(int device) {
  if (device < 0 || device >= dvf::kMaxDevices) {
    set_error("device index beyond the scratch table");
    return MOREA_EINVAL;
  }
  std::lock_guard<std::mutex> lock(dvf::g_scratch_mu);
  if (dvf::g_scratch[device]) return MOREA_OK;
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(dvf::scratch));
  if (e != hipSuccess || !ptr) {
    char buf[256];
    snprintf(buf, sizeof(buf), "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
    set_error(buf);
    return MOREA_EDEVICE;
  }
  dvf::g_scratch[device] = static_cast<int32_t*>(ptr);
  return MOREA_OK;
}

}  // namespace morea

namespace {

morea_status launch_dvf(morea_problem* p, const float* cand, float* fwd, float* inv, uint32_t* cover, int32_t* work,
                        hipStream_t s) {
  const ProblemView& P = p->view;
  const size_t V = static_cast<size_t>(P.nx) * P.ny * P.nz;
  // one wave per 512 voxels of an average tet, so that a mesh of a few large
  // tets fills the chip too (a wave takes about 10 us for its set-up and as
  // long for 512 voxels); parts beyond a tet's rows return at once
  const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(256, static_cast<int64_t>(V) / P.n_tets / 512));
  const int64_t waves = 2 * static_cast<int64_t>(P.n_tets) * parts;
  hipLaunchKernelGGL(dvf::k_dvf_clear, dim3(static_cast<unsigned>((2 * V + 256 * dvf::kClearPer - 1) / (256 * dvf::kClearPer))),
                     dim3(256), 0, s, 2 * V, work, cover);
  hipLaunchKernelGGL(dvf::k_dvf, dim3(static_cast<unsigned>((waves + 3) / 4)), dim3(256), 0, s, P, cand,
                     static_cast<int>(parts), work, cover, fwd, inv);
  hipLaunchKernelGGL(dvf::k_dvf_rest, dim3(static_cast<unsigned>((2 * V + 255) / 256)), dim3(256), 0, s, P, cand,
                     work, cover, fwd, inv);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    char buf[256];
    snprintf(buf, sizeof(buf), "DVF rasterization: %s", hipGetErrorString(e));
    set_error(buf);
    return MOREA_EDEVICE;
  }
  return MOREA_OK;
}

}  // namespace

extern "C" morea_status morea_rasterize_dvf_static(morea_problem* p, const float* cand, float* fwd, float* inv,
                                                   uint32_t* cover, void* stream) {
  if (!p || !cand || !fwd || !inv || !cover) {
    set_error("NULL argument");
    return MOREA_EINVAL;
  }
  const ProblemView& P = p->view;
  const size_t V = static_cast<size_t>(P.nx) * P.ny * P.nz;
  if (2 * V > dvf::kScratchInts) {
    char buf[160];
    snprintf(buf, sizeof(buf), "allocation-free DVF: %zu voxels per grid exceed the scratch limit of %zu", V,
             dvf::kScratchInts / 2);
    set_error(buf);
    return MOREA_ERANGE;
  }
  {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
      set_error(hipGetErrorString(e));
      return MOREA_EDEVICE;
    }
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    set_error("hipGetDevice failed");
    return MOREA_EDEVICE;
  }
  if (dev < 0 || dev >= dvf::kMaxDevices || !dvf::g_scratch[dev]) {
    // first call on this device (problems created on it normally did this)
    if (morea_status st = static_scratch_init(dev)) return st;
  }
  return launch_dvf(p, cand, fwd, inv, cover, dvf::g_scratch[dev], static_cast<hipStream_t>(stream));
}

extern "C" morea_status morea_rasterize_dvf(morea_problem* p, const float* cand, float* fwd, float* inv,
                                            uint32_t* cover, int32_t* work, void* stream) {
  if (!p || !cand || !fwd || !inv || !cover || !work) {
    set_error("NULL argument");
    return MOREA_EINVAL;
  }
  {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
      set_error(hipGetErrorString(e));
      return MOREA_EDEVICE;
    }
  }
  return launch_dvf(p, cand, fwd, inv, cover, work, static_cast<hipStream_t>(stream));
}

extern "C" morea_status morea_point_guidance(morea_problem* p, const float* pts, int32_t pop, float* f,
                                             int32_t* unmapped, void* stream) {
  if (!p || pop < 0) {
    set_error("bad argument");
    return MOREA_EINVAL;
  }
  if (pop == 0) return MOREA_OK;
  if (!pts || !f || !unmapped) {
    set_error("NULL argument");
    return MOREA_EINVAL;
  }
  const ProblemView& P = p->view;
  if (P.n_points > 6144) {
    set_error("point-based guidance keeps a candidate in LDS: at most 6144 points per mesh");
    return MOREA_ERANGE;
  }
  {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
      set_error(hipGetErrorString(e));
      return MOREA_EDEVICE;
    }
  }
  const size_t lds = sizeof(int) * 6 * static_cast<size_t>(P.n_points);
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(dvf::k_point_guidance),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  if (e == hipSuccess) {
    hipLaunchKernelGGL(dvf::k_point_guidance, dim3(pop), dim3(256), lds, static_cast<hipStream_t>(stream), P, pts,
                       p->d_set_off[0], p->d_set_fix[0], p->d_set_off[1], p->d_set_fix[1], f, unmapped);
    e = hipGetLastError();
  }
  if (e != hipSuccess) {
    char buf[256];
    snprintf(buf, sizeof(buf), "point-based guidance: %s", hipGetErrorString(e));
    set_error(buf);
    return MOREA_EDEVICE;
  }
  return MOREA_OK;
}
