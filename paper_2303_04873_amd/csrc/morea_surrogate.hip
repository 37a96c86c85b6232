// Learned pre-screen of offspring: a per-tetrahedron multilayer perceptron
// 23 -> 128 -> 128 -> 1 (ReLU) that predicts how an offspring's mean
// intensity term of a tet (the sum of h over the tet's samples in both
// directions divided by their number, Sec. 4.1.2) differs from its parent's,
// from how the tet's vertices moved away from the parent's, the tet's region
// statistics, the parent's exact term and samples of the target image.
// Trained on records produced by the exact evaluator for offspring and
// parents; a batch of offspring is ranked by the parent's exact terms plus
// the predicted changes before only the best are evaluated exactly.  The
// surrogate has no counterpart in the paper; it sits in front of the exact
// evaluation, which stays the judge of every selected candidate.
//
// Dense layers run on the matrix cores with BF16 operands and FP32
// accumulation; the pre-screen and the training on v_mfma_f32_32x32x16_bf16
// (layouts below), explicit rows' predictions on v_mfma_f32_32x32x8_bf16, one
// 64-lane wave per tile of 32 rows: lane l holds row (A) / column (B) l % 32 and the k-quad 4 * (l / 32);
// accumulator element r of lane l is row 8 (r / 4) + 4 (l / 32) + r % 4,
// column l % 32.  Master weights, gradients and the Adam state are FP32.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <random>
#include <string>
#include <vector>

#include "morea_internal.h"
#include "morea_workspace.h"

namespace morea {
namespace surr {

constexpr int kIn = 23, kInPad = 24, kHid = 128;
constexpr int oW1 = 0, oB1 = oW1 + kHid * kIn, oW2 = oB1 + kHid, oB2 = oW2 + kHid * kHid,
              oW3 = oB2 + kHid, oB3 = oW3 + kHid, kParams = oB3 + 1;   // 19,713
constexpr int kRowTile = 32;
constexpr int kGradTiles = 20;            // 16 tiles of W2, 4 of W1

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef unsigned short bf16;

__device__ __forceinline__ bf16 f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return static_cast<bf16>(u >> 16);
}
__device__ __forceinline__ float bf2f(bf16 b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }
__device__ __forceinline__ s4 ld4(const bf16* p) { return *reinterpret_cast<const s4*>(p); }
__device__ __forceinline__ f16v mma(s4 a, s4 b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int acc_row(int r, int kh) { return 8 * (r >> 2) + 4 * kh + (r & 3); }
__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Weights staged in LDS by every block that runs the network.
struct alignas(16) NetLds {
  bf16 w1[kHid][kInPad];   // W1[j][k], k padded with zeros
  bf16 w2[kHid][kHid];     // W2[j][k]
  float b1[kHid], b2[kHid], w3[kHid];
  float b3;
};

// Per-wave tile buffers.  For inference the output reduction reuses the
// layer-1 activations' space (dead once layer 2 has consumed them).
typedef float RedTile[kRowTile][kRowTile + 1];
struct alignas(16) TileLds {
  bf16 x[kRowTile][kInPad];
  union {
    bf16 h1[kRowTile][kHid];
    RedTile red;
  };
  float y[kRowTile];
};

__device__ void load_net(NetLds* N, const bf16* w1b, const bf16* w2b, const float* params) {
  for (int i = threadIdx.x; i < kHid * kInPad; i += blockDim.x) (&N->w1[0][0])[i] = w1b[i];
  for (int i = threadIdx.x; i < kHid * kHid / 4; i += blockDim.x)
    reinterpret_cast<s4*>(&N->w2[0][0])[i] = reinterpret_cast<const s4*>(w2b)[i];
  for (int i = threadIdx.x; i < kHid; i += blockDim.x) {
    N->b1[i] = params[oB1 + i];
    N->b2[i] = params[oB2 + i];
    N->w3[i] = params[oW3 + i];
  }
  if (threadIdx.x == 0) N->b3 = params[oB3];
}

// max(v, 0) as the median of v, 0 and +inf (given by inf_reg): one instruction
// where fmaxf of a matrix result takes two, the first to quieten a NaN.  0 for
// a NaN, as fmaxf.
__device__ __forceinline__ float inf_reg() {
  float inf;
  asm("s_mov_b32 %0, 0x7f800000" : "=s"(inf));
  return inf;
}

__device__ __forceinline__ float relu(float v, float inf) { return __builtin_amdgcn_fmed3f(v, 0.f, inf); }

// Forward pass of one tile of 32 rows (T->x filled).  Leaves relu(z1) in
// T->h1 (BF16) unless `red` overlays it, returns the layer-2
// pre-activations (4 column tiles) in z2 and writes y to T->y.
__device__ void tile_forward(const NetLds* N, TileLds* T, RedTile& red, f16v z2[4]) {
  const int lane = lane_id(), i = lane & 31, kh = lane >> 5;
#pragma unroll
  for (int n = 0; n < 4; n++) {
    f16v acc = {};
#pragma unroll
    for (int s = 0; s < kInPad / 8; s++)
      acc = mma(ld4(&T->x[i][8 * s + 4 * kh]), ld4(&N->w1[32 * n + i][8 * s + 4 * kh]), acc);
    const float bias = N->b1[32 * n + i];
#pragma unroll
    for (int r = 0; r < 16; r++) T->h1[acc_row(r, kh)][32 * n + i] = f2bf(fmaxf(acc[r] + bias, 0.f));
  }
  wave_sync();
  float part[16];
#pragma unroll
  for (int r = 0; r < 16; r++) part[r] = 0.f;
#pragma unroll
  for (int n = 0; n < 4; n++) {
    f16v acc = {};
#pragma unroll
    for (int s = 0; s < kHid / 8; s++)
      acc = mma(ld4(&T->h1[i][8 * s + 4 * kh]), ld4(&N->w2[32 * n + i][8 * s + 4 * kh]), acc);
    const float bias = N->b2[32 * n + i], w = N->w3[32 * n + i];
#pragma unroll
    for (int r = 0; r < 16; r++) {
      acc[r] += bias;
      part[r] = fmaf(fmaxf(acc[r], 0.f), w, part[r]);
    }
    z2[n] = acc;
  }
  // y[row] = sum over the 128 columns: this lane holds column i of 16 rows
  wave_sync();
#pragma unroll
  for (int r = 0; r < 16; r++) red[acc_row(r, kh)][i] = part[r];
  wave_sync();
  if (lane < kRowTile) {
    float y = N->b3;
    for (int c = 0; c < kRowTile; c++) y += red[lane][c];
    T->y[lane] = y;
  }
  wave_sync();
}

// ------------------------------------------------------------- features

// Features of (offspring, tet), relative to the offspring's parent (whose
// exact evaluation is known: its per-tet records are in its cache):
//   0..11  the move of the tet's 4 target-mesh vertices from the parent's,
//          (T_v - T_parent,v) / 0.5 voxel (the scale of the offspring's
//          perturbation, well resolved in BF16);
//   12..14 estimates of the change of the tet's mean intensity term, each
//          the mean of h = (I_s(x) - I_t(y))^2 over a fixed set of points of
//          the tet, x and y at the same barycentric coordinates in the
//          offspring's source and target tets, minus the same mean for the
//          parent: over the 4 vertices, the 6 edge midpoints, and 16
//          interior points (Halton points in barycentric form); divided by
//          h_scale;
//   15..21 the first 7 of the tet's 8 source-region statistics, the 7th
//          (the mean of (I_s - I_t)^2) divided by h_scale;
//   22     the parent's exact mean intensity term of the tet, (h_S + h_T) /
//          (n_S + n_T) from its records (0 without samples), divided by
//          h_scale.
// h_scale is the mean of (I_s - I_t)^2 over the grid's voxels (1 when that is
// 0), so that the h-valued features and the targets are of order 1.  Image
// values are trilinear interpolants at the point clamped into the image box,
// so every feature is continuous in the vertex positions.
constexpr float kRelScale = 2.0f;
constexpr int kHalton = 16;

// The parents of a batch of offspring: points [n][2][3][n_points], per-tet
// records of their full evaluation [n][n_tets][2], the parent of each
// offspring.
struct Parents {
  const float* pts;
  const Record* rec;
  const int* of;
  int n;
};

// Trilinear interpolant at (x, y, z) clamped into [0, n - 1] on each axis,
// from a quad copy `q` of a padded image (entry e holds FP32 voxel e of the
// padded volume, voxel e + 1 minus it, voxel e + px, voxel e + px + 1 minus that, voxel (i, j, k) at
// (k + 1) pxy + (j + 1) px + i + 1), so a sample reads two aligned 16-byte
// entries instead of eight scattered values.  The cell is the one below the
// point; at n - 1 its upper corner is on the zero border, with weight 0.
// With kBig false
// the copy is below 4 GiB: one 32-bit byte offset serves both loads, from two
// scalar base addresses (dimensions are at most 1,024, so 24-bit products do).
template <bool kBig>
__device__ __forceinline__ float sample_clamped(const ProblemView& P, const float4* q, float x, float y, float z) {
  // the median is the clamp (also of a NaN, which becomes 0)
  const float p0 = __builtin_amdgcn_fmed3f(x, 0.f, static_cast<float>(P.nx - 1));
  const float p1 = __builtin_amdgcn_fmed3f(y, 0.f, static_cast<float>(P.ny - 1));
  const float p2 = __builtin_amdgcn_fmed3f(z, 0.f, static_cast<float>(P.nz - 1));
  const unsigned c0 = static_cast<unsigned>(p0), c1 = static_cast<unsigned>(p1), c2 = static_cast<unsigned>(p2);
  const float f0 = __builtin_amdgcn_fractf(p0), f1 = __builtin_amdgcn_fractf(p1), f2 = __builtin_amdgcn_fractf(p2);
  const float4 *lo = q + (P.pxy + P.px + 1), *hi = lo + P.pxy;
  float4 b, b1;
  if constexpr (kBig) {
    const size_t e = static_cast<size_t>(c2) * P.pxy + static_cast<size_t>(c1) * P.px + c0;
    b = lo[e];
    b1 = hi[e];
  } else {
    const uint32_t off = (__umul24(c2, P.pxy) + (__umul24(c1, P.px) + c0)) << 4;
    b = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(lo) + off);
    b1 = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(hi) + off);
  }
  const float x00 = fmaf(f0, b.y, b.x), x10 = fmaf(f0, b.w, b.z);
  const float x01 = fmaf(f0, b1.y, b1.x), x11 = fmaf(f0, b1.w, b1.z);
  const float y0 = fmaf(f1, x10 - x00, x00), y1 = fmaf(f1, x11 - x01, x01);
  return fmaf(f2, y1 - y0, y0);
}

// A tet's vertices in one candidate: mesh 0 (source) or 1 (target).
__device__ __forceinline__ void tet_vertices(const ProblemView& P, const float* cand, int tet, int mesh,
                                             float d[4][3]) {
  const int4 tv = P.tets[tet];
  const int vs[4] = {tv.x, tv.y, tv.z, tv.w};
#pragma unroll
  for (int v = 0; v < 4; v++)
#pragma unroll
    for (int a = 0; a < 3; a++) d[v][a] = cand[(3 * mesh + a) * P.n_points + vs[v]];
}

// A tet as its last vertex and the edges from it to the other three.
struct Edges {
  float v[3], e[3][3];
};

__device__ __forceinline__ Edges edges(const float d[4][3]) {
  Edges t;
#pragma unroll
  for (int a = 0; a < 3; a++) {
    t.v[a] = d[3][a];
#pragma unroll
    for (int k = 0; k < 3; k++) t.e[k][a] = d[k][a] - d[3][a];
  }
  return t;
}

// h at a source and a target position: (I_s(x) - I_t(y))^2.
template <bool kBig>
__device__ __forceinline__ float h_at(const ProblemView& P, const float4* img_s, const float4* img_t,
                                      const float x[3], const float y[3]) {
  const float d = sample_clamped<kBig>(P, img_s, x[0], x[1], x[2]) - sample_clamped<kBig>(P, img_t, y[0], y[1], y[2]);
  return d * d;
}

// h at the midpoint of an edge from its ends' positions (the same bits
// whichever end comes first).
template <bool kBig>
__device__ __forceinline__ float h_mid(const ProblemView& P, const float4* img_s, const float4* img_t,
                                       const float xa[3], const float xb[3], const float ya[3], const float yb[3]) {
  float x[3], y[3];
#pragma unroll
  for (int a = 0; a < 3; a++) {
    x[a] = (xa[a] + xb[a]) * 0.5f;
    y[a] = (ya[a] + yb[a]) * 0.5f;
  }
  return h_at<kBig>(P, img_s, img_t, x, y);
}

// The points of a tet behind the estimated changes, as barycentric
// coordinates `bary`: its 4 vertices, the edge midpoints (0,1) (0,2) (0,3)
// (1,2) (1,3) (2,3), then kHalton interior points from kInner on.
constexpr int kInner = 10, kPoints = kInner + kHalton;

// Sum of h at N points of a tet, in order, one at a time.
template <bool kBig, int N>
__device__ __forceinline__ float point_run(const ProblemView& P, const float4* img_s, const float4* img_t,
                                           const Edges& S, const Edges& T, const float4* bary) {
  float sum = 0.f;
#pragma unroll 1
  for (int q = 0; q < N; q++) {
    const float4 l = bary[q];
    float x[3], y[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
      x[a] = fmaf(l.z, S.e[2][a], fmaf(l.y, S.e[1][a], fmaf(l.x, S.e[0][a], S.v[a])));
      y[a] = fmaf(l.z, T.e[2][a], fmaf(l.y, T.e[1][a], fmaf(l.x, T.e[0][a], T.v[a])));
    }
    sum += h_at<kBig>(P, img_s, img_t, x, y);
  }
  return sum;
}

// Mean of h over the interior points (`inner`) of a tet with vertices s
// (source) and t (target).
template <bool kBig>
__device__ __forceinline__ float interior_mean(const ProblemView& P, const float4* img_s, const float4* img_t,
                                               const float s[4][3], const float t[4][3], const float4* inner) {
  return point_run<kBig, kHalton>(P, img_s, img_t, edges(s), edges(t), inner) * (1.f / kHalton);
}

// Means from the values at the 4 vertices and at the 6 midpoints.
__device__ __forceinline__ void corner_means(const float hv[4], const float he[6], float m[3]) {
  m[0] = (((hv[0] + hv[1]) + hv[2]) + hv[3]) * 0.25f;
  m[1] = (((((he[0] + he[1]) + he[2]) + he[3]) + he[4]) + he[5]) * (1.f / 6.f);
}

// Means of h over the three point sets: m[0] the vertices, m[1] the edge
// midpoints, m[2] the interior points.
template <bool kBig>
__device__ __forceinline__ void point_means(const ProblemView& P, const float4* img_s, const float4* img_t,
                                            const float s[4][3], const float t[4][3], const float4* bary, float m[3]) {
  const Edges S = edges(s), T = edges(t);
  m[0] = point_run<kBig, 4>(P, img_s, img_t, S, T, bary) * 0.25f;
  m[1] = point_run<kBig, 6>(P, img_s, img_t, S, T, bary + 4) * (1.f / 6.f);
  m[2] = point_run<kBig, kHalton>(P, img_s, img_t, S, T, bary + kInner) * (1.f / kHalton);
}

// |signed volume| (voxel^3): the expected samples of the tet in its direction.
__device__ __forceinline__ float tet_volume(const float d[4][3]) {
  float e[3][3];
#pragma unroll
  for (int k = 0; k < 3; k++)
#pragma unroll
    for (int a = 0; a < 3; a++) e[k][a] = d[k + 1][a] - d[0][a];
  const float det = e[0][0] * (e[1][1] * e[2][2] - e[1][2] * e[2][1]) -
                    e[0][1] * (e[1][0] * e[2][2] - e[1][2] * e[2][0]) +
                    e[0][2] * (e[1][0] * e[2][1] - e[1][1] * e[2][0]);
  return fabsf(det) * (1.f / 6.f);
}

// Mean intensity term per sample of a tet over both directions, from its
// two records.
__device__ __forceinline__ float tet_mean_h(const Record* rec, int tet) {
  const Record a = rec[2 * static_cast<size_t>(tet)], b = rec[2 * static_cast<size_t>(tet) + 1];
  const uint32_t n = a.n + b.n;
  return n ? (a.h + b.h) / static_cast<float>(n) : 0.f;
}

// Value of stored voxel e of image `which` as FP32 (0 beyond the volume).
template <int ST>
__device__ __forceinline__ float stored_voxel(const ProblemView& P, int which, size_t e) {
  if (e >= P.pvox) return 0.f;
  if constexpr (ST == kF32) {
    return static_cast<const float*>(P.img[which])[e];
  } else if constexpr (ST == kBF16) {
    return bf2f(static_cast<const bf16*>(P.img[which])[e]);
  } else {
    return static_cast<float>(static_cast<const _Float16*>(P.img[which])[e]);
  }
}

// Quad copy of image `which` (0 source, 1 target; any storage) as FP32: entry
// e holds padded voxel e, the difference of e + 1 to it, voxel e + px, the
// difference of e + px + 1 to that (one fused multiply-add per x interpolation).
template <int ST>
__global__ void k_image_quads(ProblemView P, int which, float4* out) {
  const size_t e = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= P.pvox) return;
  const float a = stored_voxel<ST>(P, which, e), b = stored_voxel<ST>(P, which, e + P.px);
  out[e] = make_float4(a, stored_voxel<ST>(P, which, e + 1) - a, b, stored_voxel<ST>(P, which, e + P.px + 1) - b);
}

template <int ST>
__global__ void k_tet_stats(ProblemView P, const float* ref, float* stats, int* counts, float inv_mean) {
  const int tet = blockIdx.x;
  const int lane = threadIdx.x;
  const int4 tv = P.tets[tet];
  const int vs[4] = {tv.x, tv.y, tv.z, tv.w};
  double v[4][3];
  for (int i = 0; i < 4; i++)
    for (int a = 0; a < 3; a++) v[i][a] = rint(static_cast<double>(ref[3 * vs[i] + a]) * 1024.0);
  double e[3][3];
  for (int i = 0; i < 3; i++)
    for (int a = 0; a < 3; a++) e[i][a] = v[i + 1][a] - v[0][a];
  const double det = e[0][0] * (e[1][1] * e[2][2] - e[1][2] * e[2][1]) -
                     e[0][1] * (e[1][0] * e[2][2] - e[1][2] * e[2][0]) +
                     e[0][2] * (e[1][0] * e[2][1] - e[1][1] * e[2][0]);
  const double sg = det > 0 ? 1.0 : -1.0;
  // inward face normals n_i and a vertex r_i on each face (face i omits v_i)
  double n[4][3], r[4][3];
  for (int i = 0; i < 4; i++) {
    const int b0 = i == 0 ? 1 : 0, u0 = i == 0 ? 2 : (i == 1 ? 2 : (i == 2 ? 3 : 1)),
              w0 = i == 0 ? 3 : (i == 1 ? 3 : (i == 2 ? 1 : 2));
    double u[3], w[3];
    for (int a = 0; a < 3; a++) {
      r[i][a] = v[b0][a];
      u[a] = v[u0][a] - v[b0][a];
      w[a] = v[w0][a] - v[b0][a];
    }
    const double f = (i == 0 ? -sg : sg);
    n[i][0] = f * (u[1] * w[2] - u[2] * w[1]);
    n[i][1] = f * (u[2] * w[0] - u[0] * w[2]);
    n[i][2] = f * (u[0] * w[1] - u[1] * w[0]);
  }
  int lo[3], hi[3];
  const int dims[3] = {P.nx, P.ny, P.nz};
  for (int a = 0; a < 3; a++) {
    double mn = v[0][a], mx = v[0][a];
    for (int i = 1; i < 4; i++) {
      mn = fmin(mn, v[i][a]);
      mx = fmax(mx, v[i][a]);
    }
    lo[a] = max(0, static_cast<int>(ceil(mn / 1024.0)));
    hi[a] = min(dims[a] - 1, static_cast<int>(floor(mx / 1024.0)));
  }
  const int wx = max(0, hi[0] - lo[0] + 1), wy = max(0, hi[1] - lo[1] + 1), wz = max(0, hi[2] - lo[2] + 1);
  const long long nbox = det != 0.0 ? static_cast<long long>(wx) * wy * wz : 0;
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};   // n, Is, Is^2, fg_s, It, It^2, fg_t, (Is-It)^2
  for (long long q = lane; q < nbox; q += 64) {
    const int x = lo[0] + static_cast<int>(q % wx), y = lo[1] + static_cast<int>((q / wx) % wy),
              z = lo[2] + static_cast<int>(q / (static_cast<long long>(wx) * wy));
    const double p[3] = {x * 1024.0, y * 1024.0, z * 1024.0};
    bool in = true;
    for (int i = 0; i < 4 && in; i++) {
      const double val = n[i][0] * (p[0] - r[i][0]) + n[i][1] * (p[1] - r[i][1]) + n[i][2] * (p[2] - r[i][2]);
      if (val < 0) in = false;
      else if (val == 0)
        in = n[i][0] > 0 || (n[i][0] == 0 && (n[i][1] > 0 || (n[i][1] == 0 && n[i][2] > 0)));
    }
    if (!in) continue;
    const int vi = (z + 1) * P.pxy + (y + 1) * P.px + x + 1;   // padded volumes
    float is, it;
    if constexpr (ST == kF32) {
      is = static_cast<const float*>(P.img[0])[vi];
      it = static_cast<const float*>(P.img[1])[vi];
    } else if constexpr (ST == kBF16) {
      is = bf2f(static_cast<const bf16*>(P.img[0])[vi]);
      it = bf2f(static_cast<const bf16*>(P.img[1])[vi]);
    } else {
      is = static_cast<float>(static_cast<const _Float16*>(P.img[0])[vi]);
      it = static_cast<float>(static_cast<const _Float16*>(P.img[1])[vi]);
    }
    s[0] += 1.f;
    s[1] += is;
    s[2] += is * is;
    s[3] += is > 0.f;
    s[4] += it;
    s[5] += it * it;
    s[6] += it > 0.f;
    s[7] += (is - it) * (is - it);
  }
  for (int k = 0; k < 8; k++)
    for (int d = 32; d >= 1; d >>= 1) s[k] += __shfl_xor(s[k], d, 64);
  if (lane == 0) {
    const float cnt = s[0], inv_n = cnt > 0.f ? 1.f / cnt : 0.f;
    const float ms = s[1] * inv_n, mt = s[4] * inv_n;
    float* o = stats + 8 * tet;
    o[0] = ms;
    o[1] = sqrtf(fmaxf(s[2] * inv_n - ms * ms, 0.f));
    o[2] = s[3] * inv_n;
    o[3] = mt;
    o[4] = sqrtf(fmaxf(s[5] * inv_n - mt * mt, 0.f));
    o[5] = s[6] * inv_n;
    o[6] = s[7] * inv_n;
    o[7] = cnt * inv_mean;
    counts[tet] = static_cast<int>(cnt);
  }
}

// Images and constants the features read.
struct FeatureInputs {
  const float4* img_s;  // quad copies of the two images
  const float4* img_t;
  const float4* bary;   // [kPoints] points of a tet, barycentric
  const float* stats;   // [n_tets][8]
  float h_scale;
  float inv_h;          // 1 / h_scale
};

// One thread per (offspring, tet) row: the 23 features in order.  Threads in
// tet-major order, so that the threads in flight read the same part of the
// images.
template <bool kBig>
__global__ void k_features(ProblemView P, const float* pts, Parents Q, FeatureInputs F, int pop, float* feats) {
  const long long r = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (r >= static_cast<long long>(pop) * P.n_tets) return;
  const int tet = static_cast<int>(r / pop), cand = static_cast<int>(r % pop);
  float* o = feats + (static_cast<size_t>(cand) * P.n_tets + tet) * kIn;
  const int par = Q.of[cand];
  if (par < 0 || par >= Q.n) {   // no parent: the row has no features
    for (int k = 0; k < kIn; k++) o[k] = __builtin_nanf("");
    return;
  }
  const float* cp = pts + static_cast<size_t>(cand) * 6 * P.n_points;
  const float* pp = Q.pts + static_cast<size_t>(par) * 6 * P.n_points;
  float d[4][3], dp[4][3];
  tet_vertices(P, cp, tet, 1, d);
  tet_vertices(P, pp, tet, 1, dp);
#pragma unroll
  for (int v = 0; v < 4; v++)
#pragma unroll
    for (int a = 0; a < 3; a++) o[3 * v + a] = (d[v][a] - dp[v][a]) * kRelScale;
  float mc[3], mp[3];
  float sv[4][3];
  tet_vertices(P, cp, tet, 0, sv);
  point_means<kBig>(P, F.img_s, F.img_t, sv, d, F.bary, mc);
  tet_vertices(P, pp, tet, 0, sv);
  point_means<kBig>(P, F.img_s, F.img_t, sv, dp, F.bary, mp);
#pragma unroll
  for (int k = 0; k < 3; k++) o[12 + k] = (mc[k] - mp[k]) * F.inv_h;
#pragma unroll
  for (int k = 0; k < 6; k++) o[15 + k] = F.stats[8 * tet + k];
  o[21] = F.stats[8 * tet + 6] * F.inv_h;
  o[22] = tet_mean_h(Q.rec + static_cast<size_t>(par) * P.n_tets * 2, tet) * F.inv_h;
}

// Target of (offspring, tet): its mean intensity term minus its parent's
// (both from their caches' records), divided by h_scale; NaN without a valid
// parent.
__global__ void k_targets(const Record* rec, int n_tets, int rows, Parents Q, float inv_h, float* t) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  const int cand = r / n_tets, tet = r - cand * n_tets;
  const int par = Q.of[cand];
  if (par < 0 || par >= Q.n) {
    t[r] = __builtin_nanf("");
    return;
  }
  t[r] = (tet_mean_h(rec + static_cast<size_t>(cand) * n_tets * 2, tet) -
          tet_mean_h(Q.rec + static_cast<size_t>(par) * n_tets * 2, tet)) * inv_h;
}

// Coordinates by columns, so that lanes on consecutive candidates read
// consecutive words (as [cand][6][n_points] every lane of such a load lies in
// a line of its own): out [n_points][C][n] of candidates first .. first + n - 1
// of pts, rows 0..5 the coordinates (source x y z, target x y z) and, with
// C = 9, rows 6..8 the target's coordinates minus the parent's
// (unspecified without a valid parent).  Tiles of 64 candidates by 32 points.
constexpr int kColCands = 64, kColPoints = 32;
constexpr size_t kColBytes = size_t{256} << 20;   // of columns at a time (at least 64 candidates)

template <int C>
__global__ __launch_bounds__(256) void k_columns(const float* pts, int first, int n, int n_points, Parents Q,
                                                 float* out) {
  __shared__ float tile[C == 9 ? 2 : 1][kColPoints][kColCands + 1];
  const int c0 = blockIdx.y * kColCands, c = blockIdx.z;
  const size_t p0 = static_cast<size_t>(blockIdx.x) * kColPoints;
  const int pl = threadIdx.x & 31, cl = threadIdx.x >> 5;
  const size_t p = p0 + pl;
  // unconditional loads (clamped; unused beyond the edges), all in flight
  const size_t pc = min(p, static_cast<size_t>(n_points) - 1);
  float v[kColCands / 8], w[kColCands / 8];
#pragma unroll
  for (int q = 0; q < kColCands / 8; q++)
    v[q] = pts[((static_cast<size_t>(first) + min(c0 + cl + 8 * q, n - 1)) * 6 + c) * n_points + pc];
  if constexpr (C == 9)
    if (c >= 3) {
      int par[kColCands / 8];
#pragma unroll
      for (int q = 0; q < kColCands / 8; q++) par[q] = Q.of[static_cast<size_t>(first) + min(c0 + cl + 8 * q, n - 1)];
#pragma unroll
      for (int q = 0; q < kColCands / 8; q++) {
        const bool ok = par[q] >= 0 && par[q] < Q.n;
        w[q] = v[q];
        if (Q.n > 0) w[q] = Q.pts[(static_cast<size_t>(ok ? par[q] : 0) * 6 + c) * n_points + pc];
        if (!ok) w[q] = v[q];
      }
#pragma unroll
      for (int q = 0; q < kColCands / 8; q++) tile[1][pl][cl + 8 * q] = v[q] - w[q];
    }
#pragma unroll
  for (int q = 0; q < kColCands / 8; q++) tile[0][pl][cl + 8 * q] = v[q];
  __syncthreads();
  const int ol = threadIdx.x & 63, pr = threadIdx.x >> 6;
  if (c0 + ol >= n) return;
  for (int r = pr; r < kColPoints && p0 + r < static_cast<size_t>(n_points); r += 4) {
    float* o = out + ((p0 + r) * C + c) * n + c0 + ol;
    o[0] = tile[0][r][ol];
    if constexpr (C == 9)
      if (c >= 3) o[static_cast<size_t>(3) * n] = tile[1][r][ol];
  }
}

// A tet's vertices in candidate `cand` of a column array of n candidates,
// rows row .. row + 2 of C (scalar addresses plus one 32-bit byte offset where
// the tet is the same for the wave: a column is below 2^32 bytes).
template <int C>
__device__ __forceinline__ void column_vertices(const float* cols, const int4 tv, int row, int n, unsigned cand,
                                                float d[4][3]) {
  const int vs[4] = {tv.x, tv.y, tv.z, tv.w};
  unsigned off = 4u * cand;
  asm volatile("" : "+v"(off));   // kept as 32 bits, not widened ahead of a loop
#pragma unroll
  for (int v = 0; v < 4; v++)
#pragma unroll
    for (int a = 0; a < 3; a++) {
      const float* col = cols + (static_cast<size_t>(vs[v]) * C + row + a) * n;
      d[v][a] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(col) + off);
    }
}

// h at every mesh point and edge midpoint of n candidates given by columns
// (C rows a point): out [n_points + n_edges][n].  The tets around a point or an
// edge share its value: in the 800-point mesh 3,402 tets read 34,020 values, of
// which 5,415 differ.  A wave takes a point or an edge of 64 candidates; bound
// by the columns it reads (4,096 offspring: 125 us with every candidate's
// items on all XCDs, 103 us with each XCD's own).
template <bool kBig, int C>
__global__ __launch_bounds__(256) void k_shared_points(ProblemView P, const float* cols, int n, const int2* edge_ends,
                                                       int n_edges, FeatureInputs F, float* out) {
  const unsigned item_blocks = (static_cast<unsigned>(P.n_points) + n_edges + 3) / 4, groups = (n + 63u) / 64;
  unsigned ib, group;
  if (groups >= 8) {
    // blocks go to the 8 XCDs in turn: each takes its own candidates, whose
    // columns its L2 holds
    const unsigned q = blockIdx.x / 8;
    ib = q % item_blocks;
    group = q / item_blocks * 8 + blockIdx.x % 8;
  } else {
    ib = blockIdx.x / groups;
    group = blockIdx.x % groups;
  }
  const int item = __builtin_amdgcn_readfirstlane(static_cast<int>(ib * 4 + (threadIdx.x >> 6)));
  const unsigned cand = group * 64 + (threadIdx.x & 63);
  if (item >= P.n_points + n_edges || cand >= static_cast<unsigned>(n)) return;
  int a = item, b = item;
  if (item >= P.n_points) {
    const int2 e = edge_ends[item - P.n_points];
    a = __builtin_amdgcn_readfirstlane(e.x);
    b = __builtin_amdgcn_readfirstlane(e.y);
  }
  float va[6], vb[6];
#pragma unroll
  for (int k = 0; k < 6; k++) {
    va[k] = cols[(static_cast<size_t>(a) * C + k) * n + cand];
    vb[k] = cols[(static_cast<size_t>(b) * C + k) * n + cand];
  }
  // a point's two ends are itself: (v + v) / 2 = v
  out[static_cast<size_t>(item) * n + cand] = h_mid<kBig>(P, F.img_s, F.img_t, va, vb, va + 3, vb + 3);
}

// The values of a tet's vertices and edges in candidate `cand`, as means.
__device__ __forceinline__ void shared_means(const float* hs, int n_points, const int4 tv, const int te[6], int n,
                                             unsigned cand, float m[3]) {
  const int vs[4] = {tv.x, tv.y, tv.z, tv.w};
  unsigned off = 4u * cand;
  asm volatile("" : "+v"(off));   // kept as 32 bits, not widened ahead of a loop
  float hv[4], he[6];
#pragma unroll
  for (int k = 0; k < 4; k++)
    hv[k] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(hs + static_cast<size_t>(vs[k]) * n) + off);
#pragma unroll
  for (int k = 0; k < 6; k++)
    he[k] = *reinterpret_cast<const float*>(
        reinterpret_cast<const char*>(hs + (static_cast<size_t>(n_points) + te[k]) * n) + off);
  corner_means(hv, he, m);
}

// Point means and mean intensity term of every (parent, tet) of parents
// first .. first + n - 1, whose coordinates are given by columns and whose
// shared points' values by hs: out [parent][n_tets] (m0, m1, m2, term).
// Threads in tet-major order, so that the threads in flight read the same part
// of the images.
template <bool kBig>
__global__ void k_parent_means(ProblemView P, const float* cols, const float* hs, const int* tet_edges, int first,
                               int n, const Record* rec, FeatureInputs F, float4* out) {
  const long long r = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (r >= static_cast<long long>(n) * P.n_tets) return;
  const int tet = static_cast<int>(r / n), cand = static_cast<int>(r % n);
  const int4 tv = P.tets[tet];
  float S[4][3], T[4][3], m[3];
  column_vertices<6>(cols, tv, 0, n, cand, S);
  column_vertices<6>(cols, tv, 3, n, cand, T);
  int te[6];
#pragma unroll
  for (int k = 0; k < 6; k++) te[k] = tet_edges[8 * static_cast<size_t>(tet) + k];
  shared_means(hs, P.n_points, tv, te, n, cand, m);
  m[2] = interior_mean<kBig>(P, F.img_s, F.img_t, S, T, F.bary + kInner);
  const size_t par = static_cast<size_t>(first) + cand;
  out[par * P.n_tets + tet] = make_float4(m[0], m[1], m[2], tet_mean_h(rec + par * P.n_tets * 2, tet));
}

// ------------------------------------------------------------ prescreen
// The pre-screen runs both dense layers transposed, Z^T = W X^T, on
// v_mfma_f32_32x32x16_bf16 (BF16 operands, FP32 accumulation): the weights
// are the A operand (lane l: output unit 32 n + l % 32, k = 8 (l / 32) .. +7
// of a 16-wide slice), the tets the B operand (lane l: tet l % 32 of the
// tile, the same k range), and the accumulator of lane l holds tet l % 32
// and units 8 (r / 4) + 4 (l / 32) + r % 4 of the output tile (r = 0..15).
// Accumulators r = 8 g .. 8 g + 7 of layer 1 are therefore, after bias, ReLU
// and BF16 rounding, one 16-wide k-slice of layer 2's B operand, in the unit
// order  slot kk of lane half h -> unit 4 h + kk (kk < 4), 8 + 4 h + kk - 4
// (kk >= 4)  within the slice; W2's columns are stored in that order, so no
// activation passes through LDS.  Layer 1's bias rides on constant features
// (features 23..25 = 1, W1 columns 23..25 = b1 split into three BF16 terms
// that sum to it in the FP32 accumulator); layer 2's accumulators start at b2.
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned u4v __attribute__((ext_vector_type(4)));
typedef int i4v __attribute__((ext_vector_type(4)));
typedef int i8v __attribute__((ext_vector_type(8)));

// Read-only for the kernel and the same for a wave: scalar loads.
typedef const __attribute__((address_space(4))) i4v* TetPtr;
typedef const __attribute__((address_space(4))) float* StatPtr;
typedef const __attribute__((address_space(4))) i8v* TetEdgePtr;

constexpr int kPreIn = 32;                 // features padded: 23 + three constant 1s + zeros
constexpr int kPreCands = 64;              // offspring per pre-screen wave: two tiles of the network
constexpr int kPreWaves = 8;               // per block
constexpr int kMaxTetRun = 8;              // tets per pre-screen work item, or 4, 2, 1
// Work items that fill the card: 512 blocks of 8 waves.  With fewer, runs are
// shorter (a wave's tets are a serial chain): 4 offspring of 3,402 tets took
// 128 us in runs of 8 and take 79 in runs of 1; 64 of 384 tets 85 and 55 us.
constexpr int kPreItems = 4096;
constexpr int kW1Row = kPreIn + 8;         // LDS row strides padded against bank conflicts
constexpr int kW2Row = kHid + 8;

// A score's numerator and denominator are added in one order, whatever the
// length of the runs, so that a score does not depend on the size of the call:
// a tree over 8 tets at a time (aligned, tets beyond the last adding zero), of
// which a run of 8, 4, 2 or 1 is a part, then chains over those eights.
constexpr int kSumLevels = 4;
static_assert(1 << (kSumLevels - 1) == kMaxTetRun, "a run's tree");

__device__ __forceinline__ float2 add2(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }

struct alignas(16) PreLds {
  bf16 w1[kHid][kW1Row];   // W1 | b1 (three terms) | 0
  bf16 w2[kHid][kW2Row];   // W2, columns permuted per 16-wide slice
  float b2[kHid];
  float w3[kHid];
  float4 bary[kHalton];
  float2 sum[kSumLevels][64 * kPreWaves];   // per thread: sums of 1, 2, 4, 8 tets of the run
};

// Slot of unit u of a 16-wide slice in that order.
__device__ __forceinline__ int unit_slot(int u) {
  return u < 8 ? 8 * (u >> 2) + (u & 3) : 8 * ((u - 8) >> 2) + 4 + (u & 3);
}

__device__ __forceinline__ bf8 ld8(const bf16* p) { return *reinterpret_cast<const bf8*>(p); }

typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float fl2 __attribute__((ext_vector_type(2)));

// Eight values rounded to BF16 (nearest even, two per instruction).
__device__ __forceinline__ bf8 pack8(const float v[8]) {
  u4v w;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const fl2 p = {v[2 * q], v[2 * q + 1]};
    w[q] = __builtin_bit_cast(unsigned, __builtin_convertvector(p, bf2));
  }
  return __builtin_bit_cast(bf8, w);
}

// The network's output without its last bias for a tile of 32 rows whose
// features are the B operands xb0 (k = 0..15) and xb1 (16..31): this lane's
// share of the units, to be added to that of lane ^ 32.
__device__ __forceinline__ float net_tile(const PreLds& N, const bf8 xb0, const bf8 xb1, int i, int h, float inf) {
  // layer 1: 4 output tiles of 32 units, K = 32 (two slices)
  bf8 hb[8];
#pragma unroll
  for (int n = 0; n < 4; n++) {
    f16v z = {};
    z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld8(&N.w1[32 * n + i][8 * h]), xb0, z, 0, 0, 0);
    z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld8(&N.w1[32 * n + i][16 + 8 * h]), xb1, z, 0, 0, 0);
    float v0[8], v1[8];
#pragma unroll
    for (int r = 0; r < 8; r++) {
      v0[r] = relu(z[r], inf);
      v1[r] = relu(z[8 + r], inf);
    }
    hb[2 * n] = pack8(v0);
    hb[2 * n + 1] = pack8(v1);
  }
  // layer 2 (K = 128, eight slices) and the output layer
  float part = 0.f;
#pragma unroll 1
  for (int n = 0; n < 4; n++) {
    f16v z;
#pragma unroll
    for (int r = 0; r < 16; r++) z[r] = N.b2[32 * n + 8 * (r >> 2) + 4 * h + (r & 3)];
#pragma unroll
    for (int sl = 0; sl < 8; sl++)
      z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld8(&N.w2[32 * n + i][16 * sl + 8 * h]), hb[sl], z, 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 16; r++) part = fmaf(relu(z[r], inf), N.w3[32 * n + 8 * (r >> 2) + 4 * h + (r & 3)], part);
  }
  return part;
}

// Upper half of a and lower half of b exchanged.
__device__ __forceinline__ void swap_halves(unsigned& a, unsigned& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

// Score of each offspring: the predicted intensity objective,
// sum_tet (parent_tet + h_scale pred_tet) w_tet / sum_tet w_tet with
// parent_tet the parent's exact mean term (FP32, from its records), pred_tet
// the network's predicted change (in units of h_scale) and w_tet the
// offspring's |volume| of the tet's source plus that of its target (voxel^3,
// the samples the tet contributes in the two directions).  A wave takes a run
// of tets of 64 offspring, one offspring per lane: it samples the images and
// forms the features, which half-wave exchanges turn into the B operands of
// two tiles of the network.
//
// What bounds it: the 64 gathers of a tet's 16 interior points in two images
// (about 30 cycles of a CU's L1 each, from how far apart 64 offspring lie) of
// 111 loads, and the 1,770 vector instructions around them, 61% of the issue
// slots.
// 128x128x96 (3,402 tets), 4,096 offspring: 3,390 us with coordinates read as
// stored (a line per lane for each of 36 words), half a tet's points per half
// wave and 3 waves per SIMD; 1,580 us with coordinates by columns (k_columns,
// 43 us); 1,275 us with 4 waves per SIMD (blocks of 8: the weights' 46 KiB of
// LDS allow two) and one-instruction ReLUs; 1,140 us with both points and
// coordinates of 64 offspring per load and quads of differences; 930 us as it
// stands, the vertices' and midpoints' values taken from k_shared_points (103
// us, and 155 -> 118 us in k_parent_means).
template <bool kBig>
__global__ __launch_bounds__(64 * kPreWaves, 4) void k_prescreen(ProblemView P, const float* cols, const float* hs,
                                                                 const int* tet_edges,
                                                                 const int* parent_of, int n_parents,
                                                                 FeatureInputs F, const float4* pmeans,
                                                                 const float* params, const bf16* w1b,
                                                                 const bf16* w2b, int n, int tet_run,
                                                                 float2* partial, int stride) {
  __shared__ PreLds N;
  constexpr int kThreads = 64 * kPreWaves;
#pragma unroll
  for (int e0 = 0; e0 < kHid * kPreIn / 4; e0 += kThreads) {
    const int e = e0 + threadIdx.x, j = e / (kPreIn / 4), k0 = e % (kPreIn / 4) * 4;
    const s4 zero = {0, 0, 0, 0};
    *reinterpret_cast<s4*>(&N.w1[j][k0]) = k0 < kInPad ? ld4(w1b + j * kInPad + k0) : zero;
  }
#pragma unroll
  for (int e0 = 0; e0 < kHid * kHid / 4; e0 += kThreads) {
    const int e = e0 + threadIdx.x, j = e / (kHid / 4), k0 = e % (kHid / 4) * 4;
    // four units of a slice are four slots in a row
    *reinterpret_cast<s4*>(&N.w2[j][(k0 & ~15) + unit_slot(k0 & 15)]) = ld4(w2b + j * kHid + k0);
  }
  if (threadIdx.x < kHalton) N.bary[threadIdx.x] = F.bary[kInner + threadIdx.x];
  float b1 = 0.f;
  if (threadIdx.x < kHid) {
    b1 = params[oB1 + threadIdx.x];
    N.b2[threadIdx.x] = params[oB2 + threadIdx.x];
    N.w3[threadIdx.x] = params[oW3 + threadIdx.x];
  }
  const float b3 = params[oB3], inf = inf_reg();
  __syncthreads();
  if (threadIdx.x < kHid) {
    // b1 = hi + mid + lo, three BF16 terms carrying its 24-bit mantissa
    const bf16 hi = f2bf(b1), mid = f2bf(b1 - bf2f(hi)), lo = f2bf(b1 - bf2f(hi) - bf2f(mid));
    N.w1[threadIdx.x][kIn] = hi;
    N.w1[threadIdx.x][kIn + 1] = mid;
    N.w1[threadIdx.x][kIn + 2] = lo;
  }
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = lane_id(), i = lane & 31, h = lane >> 5;
  const int n_groups = (n + kPreCands - 1) / kPreCands;
  const int n_runs = (P.n_tets + tet_run - 1) / tet_run;
  const long long n_items = static_cast<long long>(n_runs) * n_groups;
  const long long n_waves = static_cast<long long>(gridDim.x) * kPreWaves;
  const TetPtr tets = (TetPtr)P.tets;
  const StatPtr stats = (StatPtr)F.stats;
  const TetEdgePtr edge_ids = (TetEdgePtr)tet_edges;
  // work items (run of tets, group of 64 offspring), run-major, one per wave
  // at a time: the lanes of a wave read nearly the same image positions and
  // the waves in flight share a few runs of tets
  for (long long w = static_cast<long long>(blockIdx.x) * kPreWaves + wave; w < n_items; w += n_waves) {
    const int run = __builtin_amdgcn_readfirstlane(static_cast<int>(w / n_groups));
    const int grp = __builtin_amdgcn_readfirstlane(static_cast<int>(w % n_groups));
    const int cand = grp * kPreCands + lane;
    const int par = cand < n ? parent_of[cand] : -1;
    const bool ok = par >= 0 && par < n_parents;   // no parent: scored by the reduction
    if (__ballot(ok) == 0) {
      if (cand < n) partial[static_cast<size_t>(run) * stride + cand] = make_float2(0.f, 0.f);
      continue;
    }
    const unsigned col = cand < n ? cand : 0;
    const float4* pmr = pmeans + static_cast<size_t>(ok ? par : 0) * P.n_tets;
    const int t_end = min(P.n_tets, (run + 1) * tet_run);
    for (int tet = run * tet_run; tet < t_end; tet++) {
      const i4v tq = tets[tet];
      const int4 tv = make_int4(tq.x, tq.y, tq.z, tq.w);
      const float4 pm = pmr[tet];
      // features in order: 12 vertex moves, 3 estimated changes, 7
      // statistics, the parent's mean term, three constant 1s for the terms
      // of b1, zeros
      float f[4][8];
      float wt;
      {
        float rel[4][3];
        column_vertices<9>(cols, tv, 6, n, col, rel);
#pragma unroll
        for (int k = 0; k < 12; k++) f[k / 8][k % 8] = rel[k / 3][k % 3] * kRelScale;
      }
      const bf8 x0 = pack8(f[0]);
      {
        float sv[4][3], d[4][3], m[3];
        column_vertices<9>(cols, tv, 0, n, col, sv);
        column_vertices<9>(cols, tv, 3, n, col, d);
        wt = tet_volume(sv) + tet_volume(d);
        asm volatile("" : "+v"(wt));   // here, or the vertices stay in registers through the network
        const i8v eq = edge_ids[tet];
        const int te[6] = {eq[0], eq[1], eq[2], eq[3], eq[4], eq[5]};
        shared_means(hs, P.n_points, tv, te, n, col, m);
        m[2] = interior_mean<kBig>(P, F.img_s, F.img_t, sv, d, N.bary);
        f[1][4] = (m[0] - pm.x) * F.inv_h;
        f[1][5] = (m[1] - pm.y) * F.inv_h;
        f[1][6] = (m[2] - pm.z) * F.inv_h;
      }
      const StatPtr st = stats + 8 * static_cast<size_t>(tet);
      f[1][7] = st[0];
#pragma unroll
      for (int k = 0; k < 5; k++) f[2][k] = st[1 + k];
      f[2][5] = st[6] * F.inv_h;
      f[2][6] = pm.w * F.inv_h;
      f[2][7] = f[3][0] = f[3][1] = 1.f;
#pragma unroll
      for (int k = 2; k < 8; k++) f[3][k] = 0.f;
      // lane l of a B operand holds row l % 32 and 8 of 16 k values by its
      // half: with the halves of features 0..7 and 8..15 exchanged, the
      // former are the first slice of offspring 0..31, the latter that of
      // offspring 32..63; likewise 16..23 and 24..31 the second slice
      u4v a = __builtin_bit_cast(u4v, x0), b = __builtin_bit_cast(u4v, pack8(f[1]));
      u4v c = __builtin_bit_cast(u4v, pack8(f[2])), e = __builtin_bit_cast(u4v, pack8(f[3]));
#pragma unroll
      for (int q = 0; q < 4; q++) {
        unsigned u = a[q], v = b[q];
        swap_halves(u, v);
        a[q] = u;
        b[q] = v;
        u = c[q];
        v = e[q];
        swap_halves(u, v);
        c[q] = u;
        e[q] = v;
      }
      float y0 = net_tile(N, __builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, c), i, h, inf);
      float y1 = net_tile(N, __builtin_bit_cast(bf8, b), __builtin_bit_cast(bf8, e), i, h, inf);
      unsigned s0 = __float_as_uint(y0), s1 = __float_as_uint(y1);
      swap_halves(s0, s1);   // both shares of this lane's own offspring
      const float y = __uint_as_float(s0) + __uint_as_float(s1) + b3;
      // the parent's exact term plus the predicted change, weighted by the
      // offspring's expected samples of the tet
      const float term = fmaf(y, F.h_scale, pm.w);
      {
#pragma clang fp contract(off)
        float2 x = make_float2(wt * term, wt);
        int lv = 0;
        for (int q = tet - run * tet_run; q & 1; q >>= 1) x = add2(N.sum[lv++][threadIdx.x], x);
        N.sum[lv][threadIdx.x] = x;
      }
    }
    float2 x = make_float2(0.f, 0.f);
    for (int lv = 0; lv < kSumLevels; lv++)
      if (((t_end - run * tet_run) >> lv) & 1) x = add2(N.sum[lv][threadIdx.x], x);
    if (cand < n) partial[static_cast<size_t>(run) * stride + cand] = x;
  }
}

// Scores from the per-(run, offspring) partial sums, kRuns runs to 8 tets: 16
// threads an offspring take a share of the eights each, in order (a single
// chain of 426 loads took 106 us for 4,096 offspring, bound by their latency),
// then the shares in order.
constexpr int kScoreGroups = 16;

// Sum of the first `have` runs of an eight (the others add zero).
template <int kRuns>
__device__ __forceinline__ float2 eight_sum(const float2* at, int stride, int have) {
  float2 v[kRuns];
#pragma unroll
  for (int q = 0; q < kRuns; q++) v[q] = q < have ? at[static_cast<size_t>(q) * stride] : make_float2(0.f, 0.f);
#pragma unroll
  for (int d = 1; d < kRuns; d *= 2)
#pragma unroll
    for (int q = 0; q < kRuns; q += 2 * d) v[q] = add2(v[q], v[q + d]);
  return v[0];
}

template <int kRuns>
__global__ __launch_bounds__(64 * kScoreGroups) void k_prescreen_reduce(const float2* partial, int n_runs, int pop,
                                                                       Parents Q, float* score) {
  __shared__ float2 s_sum[kScoreGroups][64];
  const int col = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int cand = blockIdx.x * 64 + col;
  const int n_eights = (n_runs + kRuns - 1) / kRuns;
  const int per = (n_eights + kScoreGroups - 1) / kScoreGroups, t1 = min(n_eights, (grp + 1) * per);
  const int whole = min(t1, n_runs / kRuns);
  float2 a = make_float2(0.f, 0.f);
  if (cand < pop) {
    const float2* at = partial + static_cast<size_t>(grp) * per * kRuns * pop + cand;
    int t = grp * per;
#pragma unroll 8 / kRuns + (kRuns > 4)
    for (; t < whole; t++, at += static_cast<size_t>(kRuns) * pop) a = add2(a, eight_sum<kRuns>(at, pop, kRuns));
    if (t < t1) a = add2(a, eight_sum<kRuns>(at, pop, n_runs - t * kRuns));
  }
  s_sum[grp][col] = a;
  __syncthreads();
  if (grp != 0 || cand >= pop) return;
  for (int q = 1; q < kScoreGroups; q++) a = add2(a, s_sum[q][col]);
  const int par = Q.of[cand];
  // no parent: never preferred
  score[cand] = par < 0 || par >= Q.n ? INFINITY : (a.y > 0.f ? a.x / a.y : 0.f);
}

// Predictions for explicit feature rows (one wave per 32 rows).
__global__ __launch_bounds__(256) void k_predict_rows(const float* X, int n, const bf16* w1b,
                                                       const bf16* w2b, const float* params, float* y) {
  __shared__ NetLds N;
  __shared__ TileLds Tl[4];
  load_net(&N, w1b, w2b, params);
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = lane_id(), i = lane & 31, kh = lane >> 5;
  const int row0 = (blockIdx.x * 4 + wave) * kRowTile;
  if (row0 >= n) return;
  TileLds* T = &Tl[wave];
  const bool valid = row0 + i < n;
  for (int k = kh * 12; k < (kh ? kInPad : 12); k++)
    T->x[i][k] = f2bf(valid && k < kIn ? X[static_cast<size_t>(row0 + i) * kIn + k] : 0.f);
  wave_sync();
  f16v z2[4];
  tile_forward(&N, T, T->red, z2);
  if (lane < kRowTile && row0 + lane < n) y[row0 + lane] = T->y[lane];
}

// ------------------------------------------------------------- training
// Loss and gradients of a batch in one kernel: a block of 4 waves takes 128
// rows at a time, a wave 32 of them, through the forward pass, the backward
// pass and the weight gradients, whose sums stay in accumulators over all the
// block's rows.  v_mfma_f32_32x32x16 has the same lane and k layout for both
// operands, so each product can be formed in either orientation from the
// same fragments:
//   z^T = W x^T  (lane = row, registers = units): relu(z1^T) is at once the
//     other operand of layer 2, dz2^T that of the backward product, and the
//     output layer sums over a lane's own registers;
//   z = x W^T    (lane = unit, registers = rows): the contraction over rows
//     of dW = dz^T h reads dz and h as they stand in the accumulators.
// Both orientations are computed (the matrix cores have the time), so nothing
// is transposed and no activation goes to memory; h1 and dz2 pass through LDS
// as whole fragments, because wave w sums rows 32 w .. of dW2 over the rows of
// all four waves (64 accumulators a wave; all of dW2 in every wave would take
// 256 and spill).  The k slots of an accumulator used as an operand are in
// the order of unit_slot, so W2 and its transpose are stored in that order.
//
// Bound: 154 KB of LDS (both orders of W2 and the fragments) leave one block
// on a compute unit, one wave on a SIMD, so it is the chain of a block's
// steps (152 MFMAs of 32 cycles and as long reading fragments) after loading
// the weights: 8.3 us per 32,768 rows after 15 us.  65,536 rows: 32 us in a
// kernel trace, then 4.8 us to add the blocks' sums; a batch's loss and
// gradients went from 723 to 31 us, 35 in calls that a host issues one by one
// (activations through memory, 320 waves for the weight gradients,
// and one thread adding 2,048 partial sums per bias took 175 + 76 + 476 us).
constexpr int kPartTiles = kGradTiles * 1024;              // entries of dW2 (16 tiles) and dW1 (4)
constexpr int kPartSums = 3 * kHid + 2;                    // dw3, db2, db1, db3, loss
constexpr int kPart = (kPartTiles + kPartSums + 63) / 64 * 64;   // floats per block
constexpr int kTrainWaves = 4;
constexpr int kTrainBlocks = 256;                          // one per compute unit
constexpr int kXRow = kRowTile + 8;

struct alignas(16) TrainLds {
  bf16 w1[kHid][kW1Row];                   // W1[j][k], zeros beyond the features
  union {
    struct {
      bf16 w2[kHid][kW2Row];               // W2[j][slot of k]
      bf16 w2t[kHid][kW2Row];              // its transpose: [k][slot of j]
    };
    float sums[kTrainWaves][kPartSums];    // after the last rows
  };
  float b1[kHid], b2[kHid], w3[kHid];
  bf16 x[kTrainWaves][kRowTile][kXRow];    // rows, features padded with zeros
  float dy[kTrainWaves][kRowTile];
  union {
    struct {                               // fragments [wave][2 tile + slice][lane]
      u4v h[kTrainWaves][8][64], d[kTrainWaves][8][64];
    };
    float dw1[kTrainWaves][4 * 1024];      // after the last rows
  };
};
static_assert(sizeof(TrainLds) <= 160 * 1024, "one block's LDS");

// Accumulators 8 g .. 8 g + 7 as one operand fragment (rounded to BF16).
__device__ __forceinline__ bf8 pack_acc(const f16v& z, int g) {
  u4v w;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const fl2 v = {z[8 * g + 2 * q], z[8 * g + 2 * q + 1]};
    w[q] = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf2));
  }
  return __builtin_bit_cast(bf8, w);
}

__device__ __forceinline__ f16v mma16(bf8 a, bf8 b, f16v c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// The 16 values of v[32 n ..] at the rows of lane half h's accumulators.
__device__ __forceinline__ f16v acc_rows(const float* v, int h) {
  f16v r;
#pragma unroll
  for (int g = 0; g < 4; g++) {
    const float4 q = *reinterpret_cast<const float4*>(v + 8 * g + 4 * h);
    r[4 * g] = q.x;
    r[4 * g + 1] = q.y;
    r[4 * g + 2] = q.z;
    r[4 * g + 3] = q.w;
  }
  return r;
}

__global__ __launch_bounds__(64 * kTrainWaves, 1) void k_train(const float* X, const float* t, int n,
                                                              const bf16* w1b, const bf16* w2b, const float* params,
                                                              float* part) {
  __shared__ TrainLds S;
  const float inf = inf_reg();
  constexpr int kThreads = 64 * kTrainWaves;
#pragma unroll
  for (int e0 = 0; e0 < kHid * kPreIn / 4; e0 += kThreads) {
    const int e = e0 + threadIdx.x, j = e / (kPreIn / 4), k0 = e % (kPreIn / 4) * 4;
    const s4 zero = {0, 0, 0, 0};
    *reinterpret_cast<s4*>(&S.w1[j][k0]) = k0 < kInPad ? ld4(w1b + j * kInPad + k0) : zero;
  }
#pragma unroll
  for (int e0 = 0; e0 < kHid * kHid / 4; e0 += kThreads) {
    // consecutive lanes take consecutive j: the transposed stores fill whole
    // LDS rows (consecutive k would be 16 lanes to a bank)
    const int e = e0 + threadIdx.x, j = e % kHid, k0 = e / kHid * 4;
    const s4 w = ld4(w2b + j * kHid + k0);
    // four units of a slice are four slots in a row
    *reinterpret_cast<s4*>(&S.w2[j][(k0 & ~15) + unit_slot(k0 & 15)]) = w;
#pragma unroll
    for (int q = 0; q < 4; q++) S.w2t[k0 + q][(j & ~15) + unit_slot(j & 15)] = static_cast<bf16>(w[q]);
  }
  if (threadIdx.x < kHid) {
    S.b1[threadIdx.x] = params[oB1 + threadIdx.x];
    S.b2[threadIdx.x] = params[oB2 + threadIdx.x];
    S.w3[threadIdx.x] = params[oW3 + threadIdx.x];
  }
  const float b3 = params[oB3];
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  int lane = lane_id(), i = lane & 31, h = lane >> 5;
  bf16 (*xs)[kXRow] = S.x[wave];
  for (int q = lane; q < kRowTile * kXRow; q += 64) xs[0][q] = 0;
  const float two_n = 2.f / static_cast<float>(n);
  f16v dw2[4], dw1[4];
#pragma unroll
  for (int a = 0; a < 4; a++) dw1[a] = dw2[a] = f16v{};
  float gw3[4] = {}, gb2[4] = {}, gb1[4] = {}, gb3 = 0.f, loss = 0.f;
  const int step = gridDim.x * kTrainWaves * kRowTile;
  for (int first = blockIdx.x * kTrainWaves * kRowTile; first < n; first += step) {
    // opaque lane indices: the weight fragments are read from LDS where they
    // are used, not kept in 288 registers over the steps
    asm volatile("" : "+v"(i), "+v"(h), "+v"(lane));
    const int row0 = first + wave * kRowTile, rows = min(kRowTile, n - row0);   // rows <= 0: none
    // all loads of the tile in flight together (clamped to the batch)
    constexpr int kLoads = (kRowTile * kIn + 63) / 64;
    const size_t x0 = static_cast<size_t>(row0) * kIn, x_last = static_cast<size_t>(n) * kIn - 1;
    float xv[kLoads];
#pragma unroll
    for (int q = 0; q < kLoads; q++) xv[q] = X[min(x0 + 64 * q + lane, x_last)];
    const float target = t[min(row0 + i, n - 1)];
    __syncthreads();   // the weights (first step) or the last step's fragments are done with
#pragma unroll
    for (int q0 = 0; q0 < kLoads; q0++) {
      const int q = 64 * q0 + lane;
      if (q < kRowTile * kIn) xs[q / kIn][q % kIn] = f2bf(q < rows * kIn ? xv[q0] : 0.f);
    }
    wave_sync();
    // the rows as an operand: lane = row, features 16 s + 8 h + 0..7, and
    // transposed: lane = feature, the rows in accumulator order
    bf8 xb[2], xu[2];
#pragma unroll
    for (int s = 0; s < 2; s++) {
      xb[s] = ld8(&xs[i][16 * s + 8 * h]);
      u4v w;
#pragma unroll
      for (int k = 0; k < 8; k += 2) {
        const int r = 16 * s + (k < 4 ? 4 * h + k : 8 + 4 * h + k - 4);
        w[k / 2] = static_cast<unsigned>(xs[r][i]) | static_cast<unsigned>(xs[r + 1][i]) << 16;
      }
      xu[s] = __builtin_bit_cast(bf8, w);
    }
    // layer 1 in both orientations
    bf8 ht[8];
    u4v hu[8];
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const bf8 w0 = ld8(&S.w1[32 * a + i][8 * h]), w1 = ld8(&S.w1[32 * a + i][16 + 8 * h]);
      f16v z = acc_rows(S.b1 + 32 * a, h), u;
      const float bias = S.b1[32 * a + i];
#pragma unroll
      for (int r = 0; r < 16; r++) u[r] = bias;
      z = mma16(w1, xb[1], mma16(w0, xb[0], z));
      u = mma16(xb[1], w1, mma16(xb[0], w0, u));
#pragma unroll
      for (int r = 0; r < 16; r++) {
        z[r] = relu(z[r], inf);
        u[r] = relu(u[r], inf);
      }
#pragma unroll
      for (int g = 0; g < 2; g++) {
        ht[2 * a + g] = pack_acc(z, g);
        hu[2 * a + g] = __builtin_bit_cast(u4v, pack_acc(u, g));
        S.h[wave][2 * a + g][lane] = hu[2 * a + g];
      }
    }
    // layer 2 in both orientations; the output and its gradient
    f16v zt[4], zu[4];
    float y = 0.f;
#pragma unroll
    for (int a = 0; a < 4; a++) {
      zt[a] = acc_rows(S.b2 + 32 * a, h);
      const float bias = S.b2[32 * a + i];
#pragma unroll
      for (int r = 0; r < 16; r++) zu[a][r] = bias;
#pragma unroll
      for (int sl = 0; sl < 8; sl++) {
        const bf8 w = ld8(&S.w2[32 * a + i][16 * sl + 8 * h]);
        zt[a] = mma16(w, ht[sl], zt[a]);
        zu[a] = mma16(ht[sl], w, zu[a]);
      }
      const f16v w3 = acc_rows(S.w3 + 32 * a, h);
#pragma unroll
      for (int r = 0; r < 16; r++) y = fmaf(relu(zt[a][r], inf), w3[r], y);
    }
    y += __shfl_xor(y, 32, 64) + b3;
    const float diff = i < rows ? y - target : 0.f;
    const float dy = diff * two_n;
    if (h == 0) {
      S.dy[wave][i] = dy;
      loss = fmaf(diff, diff, loss);
      gb3 += dy;
    }
    wave_sync();
    // dz2 in both orientations, dw3 and db2
    const f16v dyr = acc_rows(S.dy[wave], h);
    bf8 dt[8];
#pragma unroll
    for (int a = 0; a < 4; a++) {
      const f16v w3r = acc_rows(S.w3 + 32 * a, h);
      const float w3 = S.w3[32 * a + i];
#pragma unroll
      for (int r = 0; r < 16; r++) {
        zt[a][r] = zt[a][r] > 0.f ? dy * w3r[r] : 0.f;
        const float z = zu[a][r], dz = z > 0.f ? dyr[r] * w3 : 0.f;
        gw3[a] = fmaf(dyr[r], relu(z, inf), gw3[a]);
        gb2[a] += dz;
        zu[a][r] = dz;
      }
#pragma unroll
      for (int g = 0; g < 2; g++) {
        dt[2 * a + g] = pack_acc(zt[a], g);
        S.d[wave][2 * a + g][lane] = __builtin_bit_cast(u4v, pack_acc(zu[a], g));
      }
    }
    // layer 1 backward: dh1 = dz2 W2, db1 and this wave's share of dW1
#pragma unroll
    for (int a = 0; a < 4; a++) {
      f16v z = {};
#pragma unroll
      for (int sl = 0; sl < 8; sl++) z = mma16(dt[sl], ld8(&S.w2t[32 * a + i][16 * sl + 8 * h]), z);
#pragma unroll
      for (int r = 0; r < 16; r++) {
        // relu'(z1): h1 is not negative, so any set bit means z1 > 0
        const unsigned hb = hu[2 * a + r / 8][r % 8 / 2];
        z[r] = ((r & 1) ? hb >> 16 : hb & 0xffffu) ? z[r] : 0.f;
        gb1[a] += z[r];
      }
      dw1[a] = mma16(pack_acc(z, 1), xu[1], mma16(pack_acc(z, 0), xu[0], dw1[a]));
    }
    __syncthreads();
    // rows 32 wave .. of dW2 over the block's 128 rows
#pragma unroll
    for (int v = 0; v < kTrainWaves; v++)
#pragma unroll
      for (int g = 0; g < 2; g++) {
        const bf8 d = __builtin_bit_cast(bf8, S.d[v][2 * wave + g][lane]);
#pragma unroll
        for (int b = 0; b < 4; b++) dw2[b] = mma16(d, __builtin_bit_cast(bf8, S.h[v][2 * b + g][lane]), dw2[b]);
      }
  }
  // the block's sums: lane halves, then waves in order
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 4; a++) {
    gw3[a] += __shfl_xor(gw3[a], 32, 64);
    gb2[a] += __shfl_xor(gb2[a], 32, 64);
    gb1[a] += __shfl_xor(gb1[a], 32, 64);
    if (h == 0) {
      S.sums[wave][32 * a + i] = gw3[a];
      S.sums[wave][kHid + 32 * a + i] = gb2[a];
      S.sums[wave][2 * kHid + 32 * a + i] = gb1[a];
    }
  }
  for (int d = 16; d >= 1; d >>= 1) {
    gb3 += __shfl_xor(gb3, d, 64);
    loss += __shfl_xor(loss, d, 64);
  }
  if (lane == 0) {
    S.sums[wave][3 * kHid] = gb3;
    S.sums[wave][3 * kHid + 1] = loss;
  }
  float* out = part + static_cast<size_t>(blockIdx.x) * kPart;
#pragma unroll
  for (int a = 0; a < 4; a++)
#pragma unroll
    for (int r = 0; r < 16; r++) {
      out[((4 * wave + a) * 16 + r) * 64 + lane] = dw2[a][r];
      S.dw1[wave][(a * 16 + r) * 64 + lane] = dw1[a][r];
    }
  __syncthreads();
#pragma unroll
  for (int e0 = 0; e0 < 4 * 1024; e0 += kThreads) {
    const int e = e0 + threadIdx.x;
    out[16 * 1024 + e] = ((S.dw1[0][e] + S.dw1[1][e]) + S.dw1[2][e]) + S.dw1[3][e];
  }
  for (int e = threadIdx.x; e < kPart - kPartTiles; e += kThreads)
    out[kPartTiles + e] = e < kPartSums ? ((S.sums[0][e] + S.sums[1][e]) + S.sums[2][e]) + S.sums[3][e] : 0.f;
}

// Parameter of entry e of a block's partial sums, -1 for none, -2 the loss.
__device__ __forceinline__ int part_param(int e) {
  if (e < kPartTiles) {
    const int q = e >> 10, r = (e >> 6) & 15, i = e & 31, h = (e >> 5) & 1;
    const int row = acc_row(r, h);
    if (q < 16) return oW2 + (32 * (q / 4) + row) * kHid + 32 * (q % 4) + i;
    return i < kIn ? oW1 + (32 * (q - 16) + row) * kIn + i : -1;
  }
  e -= kPartTiles;
  if (e < kHid) return oW3 + e;
  if (e < 2 * kHid) return oB2 + e - kHid;
  if (e < 3 * kHid) return oB1 + e - 2 * kHid;
  return e == 3 * kHid ? oB3 : (e == 3 * kHid + 1 ? -2 : -1);
}

// Gradient of every parameter from the blocks' partial sums (16 groups of
// partials side by side, then the groups in order: a fixed order, and 16
// chains instead of one, since a thread's sum is bound by the latency of its
// loads), then either the Adam update (FP32 master, BF16 copies refreshed) or
// a copy of the gradient to `grad_out`.
constexpr int kSumGroups = 16;

__global__ __launch_bounds__(64 * kSumGroups) void k_reduce_update(const float* part, int n_parts, float* params,
                                                                  float* m, float* v, bf16* w1b, bf16* w2b, float lr,
                                                                  float c1, float c2, float* grad_out,
                                                                  float* loss_out, int n) {
  __shared__ float s_sum[kSumGroups][64];
  const int col = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + col;
  const int per = (n_parts + kSumGroups - 1) / kSumGroups;
  const int b1_ = min(n_parts, (grp + 1) * per);
  float g = 0.f;
#pragma unroll 4
  for (int b = grp * per; b < b1_; b++) g += part[static_cast<size_t>(b) * kPart + e];
  s_sum[grp][col] = g;
  __syncthreads();
  if (grp != 0) return;
  for (int q = 1; q < kSumGroups; q++) g += s_sum[q][col];
  const int p = part_param(e);
  if (p == -2 && loss_out) *loss_out = g / static_cast<float>(n);
  if (p < 0) return;
  if (grad_out) {
    grad_out[p] = g;
    return;
  }
  const float b1 = 0.9f, b2 = 0.999f;
  const float mm = b1 * m[p] + (1.f - b1) * g;
  const float vv = b2 * v[p] + (1.f - b2) * g * g;
  m[p] = mm;
  v[p] = vv;
  const float w = params[p] - lr * (mm * c1) / (sqrtf(vv * c2) + 1e-8f);
  params[p] = w;
  if (p < oB1) {
    const int j = (p - oW1) / kIn, k = (p - oW1) % kIn;
    w1b[j * kInPad + k] = f2bf(w);
  } else if (p >= oW2 && p < oB2) {
    w2b[p - oW2] = f2bf(w);
  }
}

__global__ void k_refresh_bf16(const float* params, bf16* w1b, bf16* w2b) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < kHid * kInPad) {
    const int j = q / kInPad, k = q % kInPad;
    w1b[q] = k < kIn ? f2bf(params[oW1 + j * kIn + k]) : static_cast<bf16>(0);
  }
  if (q < kHid * kHid) w2b[q] = f2bf(params[oW2 + q]);
}

// --------------------------------------------------------- selection

// Indices of the k lowest scores (ties: lower index first), one block,
// bitonic sort of (score, index) pairs in LDS; n <= 8192.
__global__ __launch_bounds__(1024) void k_select(const float* score, int n, int k, int* idx_out) {
  __shared__ float key[8192];
  __shared__ int val[8192];
  int m = 1;
  while (m < n) m <<= 1;
  for (int q = threadIdx.x; q < m; q += blockDim.x) {
    key[q] = q < n ? score[q] : INFINITY;
    val[q] = q;
  }
  __syncthreads();
  for (int size = 2; size <= m; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int q = threadIdx.x; q < m; q += blockDim.x) {
        const int o = q ^ stride;
        if (o > q) {
          const bool up = (q & size) == 0;
          const float a = key[q], b = key[o];
          const int ia = val[q], ib = val[o];
          const bool greater = (a > b) || (a == b && ia > ib) || (a != a && b == b);
          if (greater == up) {
            key[q] = b; key[o] = a;
            val[q] = ib; val[o] = ia;
          }
        }
      }
      __syncthreads();
    }
  for (int q = threadIdx.x; q < k; q += blockDim.x) idx_out[q] = val[q];
}

__global__ void k_gather(const float* pts, const int* idx, int k, int per_cand, float* out) {
  for (size_t q = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
       q < static_cast<size_t>(k) * per_cand; q += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const size_t c = q / per_cand, e = q % per_cand;
    out[q] = pts[static_cast<size_t>(idx[c]) * per_cand + e];
  }
}

}  // namespace surr
}  // namespace morea

using namespace morea;
using namespace morea::surr;

struct morea_surrogate {
  morea_problem* p = nullptr;
  int max_rows = 0;
  float* params = nullptr;
  float* adam_m = nullptr;
  float* adam_v = nullptr;
  bf16* w1b = nullptr;
  bf16* w2b = nullptr;
  float* stats = nullptr;
  int* counts = nullptr;
  float* ref = nullptr;
  float4* img_s = nullptr;  // quad copies of the source and target images
  float4* img_t = nullptr;
  float4* bary = nullptr;   // [kPoints] sample points of a tet, barycentric
  int n_edges = 0;          // edges of the mesh, each once
  int2* edge_ends = nullptr;   // [n_edges]
  int* tet_edges = nullptr;    // [n_tets][8] a tet's edges (0,1) (0,2) (0,3) (1,2) (1,3) (2,3), two unused
  float h_scale = 1.f;      // mean of (I_s - I_t)^2 over the grid (1 when 0)
  // pre-screen: the parents' point means, then the partial sums, columns and
  // shared points' values
  morea::Workspace work;
  float* part = nullptr;    // training: the blocks' partial sums
  int steps = 0;
  std::vector<void*> allocs;
};

namespace {
thread_local std::string s_error;
morea_status sfail(morea_status s, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  s_error = buf;
  morea::set_error(buf);
  return s;
}

template <typename T>
morea_status salloc(morea_surrogate* s, T** dst, size_t bytes) {
  void* d = nullptr;
  hipError_t e = hipMalloc(&d, bytes ? bytes : 4);
  if (e != hipSuccess) return sfail(MOREA_ENOMEM, "hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
  s->allocs.push_back(d);
  *dst = static_cast<T*>(d);
  return MOREA_OK;
}

morea_status sdev(hipError_t e, const char* what) {
  if (e == hipSuccess) return MOREA_OK;
  return sfail(MOREA_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

hipError_t launch_stats(morea_surrogate* s, const float* ref_dev) {
  const ProblemView& P = s->p->view;
  const float inv_mean = static_cast<float>(P.n_tets) / static_cast<float>(P.nx * P.ny * P.nz);
  switch (s->p->storage) {
    case kF32: hipLaunchKernelGGL(k_tet_stats<kF32>, dim3(P.n_tets), dim3(64), 0, 0, P, ref_dev, s->stats, s->counts, inv_mean); break;
    case kBF16: hipLaunchKernelGGL(k_tet_stats<kBF16>, dim3(P.n_tets), dim3(64), 0, 0, P, ref_dev, s->stats, s->counts, inv_mean); break;
    default: hipLaunchKernelGGL(k_tet_stats<kF16>, dim3(P.n_tets), dim3(64), 0, 0, P, ref_dev, s->stats, s->counts, inv_mean); break;
  }
  return hipGetLastError();
}

hipError_t launch_image_copies(morea_surrogate* s) {
  const ProblemView& P = s->p->view;
  const dim3 grid((P.pvox + 255) / 256);
  for (int which = 0; which < 2; which++) {
    float4* out = which ? s->img_t : s->img_s;
    switch (s->p->storage) {
      case kF32: hipLaunchKernelGGL(k_image_quads<kF32>, grid, dim3(256), 0, 0, P, which, out); break;
      case kBF16: hipLaunchKernelGGL(k_image_quads<kBF16>, grid, dim3(256), 0, 0, P, which, out); break;
      default: hipLaunchKernelGGL(k_image_quads<kF16>, grid, dim3(256), 0, 0, P, which, out); break;
    }
  }
  return hipGetLastError();
}

// Radical inverse of j in base b (van der Corput).
double radical_inverse(int j, int b) {
  double r = 0.0, f = 1.0 / b;
  for (; j > 0; j /= b, f /= b) r += f * (j % b);
  return r;
}

// A tet's sample points as barycentric coordinates: the vertices, the edge
// midpoints, then Halton points j = 1..16 in bases 2, 3, 5, each (u1, u2, u3)
// sorted into a <= b <= c and mapped to (a, b - a, c - b, 1 - c) (the spacings
// of sorted uniforms, uniform on the simplex).
std::vector<float4> sample_points() {
  std::vector<float4> out;
  float l[4];
  for (int v = 0; v < 4; v++) out.push_back(make_float4(v == 0, v == 1, v == 2, v == 3));
  for (int v = 0; v < 4; v++)
    for (int w = v + 1; w < 4; w++) {
      for (int k = 0; k < 4; k++) l[k] = k == v || k == w ? 0.5f : 0.f;
      out.push_back(make_float4(l[0], l[1], l[2], l[3]));
    }
  for (int j = 1; j <= kHalton; j++) {
    double u[3] = {radical_inverse(j, 2), radical_inverse(j, 3), radical_inverse(j, 5)};
    std::sort(u, u + 3);
    out.push_back(make_float4(static_cast<float>(u[0]), static_cast<float>(u[1] - u[0]),
                              static_cast<float>(u[2] - u[1]), static_cast<float>(1.0 - u[2])));
  }
  return out;
}

// The mesh's edges, each once, in ascending order of their ends, and the tets'.
void mesh_edges(const std::vector<int>& tets, std::vector<int2>& ends, std::vector<int>& of_tet) {
  const size_t n_tets = tets.size() / 4;
  std::vector<std::pair<std::pair<int, int>, size_t>> all;   // ends, place in of_tet
  all.reserve(6 * n_tets);
  for (size_t t = 0; t < n_tets; t++) {
    size_t k = 8 * t;
    for (int v = 0; v < 4; v++)
      for (int w = v + 1; w < 4; w++) all.push_back({std::minmax(tets[4 * t + v], tets[4 * t + w]), k++});
  }
  std::sort(all.begin(), all.end());
  of_tet.assign(8 * n_tets, 0);
  for (size_t i = 0; i < all.size(); i++) {
    if (i == 0 || all[i].first != all[i - 1].first) ends.push_back(make_int2(all[i].first.first, all[i].first.second));
    of_tet[all[i].second] = static_cast<int>(ends.size()) - 1;
  }
}

// Blocks of k_shared_points: 4 points or edges of 64 candidates each; from 8
// groups of candidates on, a multiple of 8 groups.
unsigned shared_blocks(size_t n_shared, int n) {
  const size_t groups = (static_cast<size_t>(n) + 63) / 64;
  return static_cast<unsigned>((n_shared + 3) / 4 * (groups >= 8 ? (groups + 7) / 8 * 8 : groups));
}

// The quad copies reach 4 GiB: sampled with 64-bit offsets.
bool big_quads(const ProblemView& P) { return P.pvox >= 1u << 28; }

FeatureInputs feature_inputs(const morea_surrogate* s) {
  return FeatureInputs{s->img_s, s->img_t, s->bary, s->stats, s->h_scale, 1.f / s->h_scale};
}

int train_blocks(int rows) {
  const int tiles = (rows + kRowTile - 1) / kRowTile;
  return std::min(kTrainBlocks, (tiles + kTrainWaves - 1) / kTrainWaves);
}

morea_status train_launch(morea_surrogate* s, const float* X, const float* t, int n, float lr,
                          float* grad_out, float* loss_out, hipStream_t st) {
  if (!s || !X || !t) return sfail(MOREA_EINVAL, "NULL argument");
  if (n < 1 || n > s->max_rows) return sfail(MOREA_ERANGE, "rows %d outside [1, %d]", n, s->max_rows);
  const int blocks = train_blocks(n);
  hipLaunchKernelGGL(k_train, dim3(blocks), dim3(64 * kTrainWaves), 0, st, X, t, n, s->w1b, s->w2b, s->params,
                     s->part);
  float c1 = 1.f, c2 = 1.f;
  if (!grad_out) {
    s->steps += 1;
    c1 = 1.f / (1.f - powf(0.9f, static_cast<float>(s->steps)));
    c2 = 1.f / (1.f - powf(0.999f, static_cast<float>(s->steps)));
  }
  hipLaunchKernelGGL(k_reduce_update, dim3(kPart / 64), dim3(64 * kSumGroups), 0, st, s->part, blocks,
                     s->params, s->adam_m, s->adam_v, s->w1b, s->w2b, lr, c1, c2, grad_out, loss_out, n);
  return sdev(hipGetLastError(), "training kernels");
}
}  // namespace

extern "C" {

int32_t morea_surrogate_num_params(void) { return kParams; }
int32_t morea_surrogate_num_features(void) { return kIn; }

morea_status morea_surrogate_create(morea_problem* p, int32_t max_rows, uint64_t seed,
                                    morea_surrogate** out) {
  if (!out) return sfail(MOREA_EINVAL, "out is NULL");
  *out = nullptr;
  if (!p) return sfail(MOREA_EINVAL, "problem is NULL");
  if (max_rows < 1 || max_rows > (1 << 24)) return sfail(MOREA_EINVAL, "max_rows %d outside [1, 2^24]", max_rows);
  morea_surrogate* s = new morea_surrogate();
  s->p = p;
  s->max_rows = max_rows;
  const int NT = p->view.n_tets;
  morea_status st = MOREA_OK;
  auto ok = [&](morea_status r) { if (st == MOREA_OK) st = r; return st == MOREA_OK; };
  ok(salloc(s, &s->params, sizeof(float) * kParams));
  ok(salloc(s, &s->adam_m, sizeof(float) * kParams));
  ok(salloc(s, &s->adam_v, sizeof(float) * kParams));
  ok(salloc(s, &s->w1b, sizeof(bf16) * kHid * kInPad));
  ok(salloc(s, &s->w2b, sizeof(bf16) * kHid * kHid));
  ok(salloc(s, &s->stats, sizeof(float) * 8 * NT));
  ok(salloc(s, &s->counts, sizeof(int) * NT));
  ok(salloc(s, &s->part, sizeof(float) * kPart * static_cast<size_t>(train_blocks(max_rows))));
  ok(salloc(s, &s->ref, sizeof(float) * 3 * p->view.n_points));
  ok(salloc(s, &s->img_s, sizeof(float4) * static_cast<size_t>(p->view.pvox)));
  ok(salloc(s, &s->img_t, sizeof(float4) * static_cast<size_t>(p->view.pvox)));
  ok(salloc(s, &s->bary, sizeof(float4) * kPoints));
  std::vector<int2> ends;
  std::vector<int> of_tet;
  mesh_edges(p->tets_host, ends, of_tet);
  s->n_edges = static_cast<int>(ends.size());
  ok(salloc(s, &s->edge_ends, sizeof(int2) * ends.size()));
  ok(salloc(s, &s->tet_edges, sizeof(int) * of_tet.size()));
  float* ref_dev = s->ref;
  if (st == MOREA_OK) {
    // He-normal initial weights, zero biases, from the given seed
    std::vector<float> h(kParams, 0.f);
    std::mt19937_64 rng(seed);
    std::normal_distribution<float> n1(0.f, sqrtf(2.f / kIn)), n2(0.f, sqrtf(2.f / kHid)), n3(0.f, sqrtf(1.f / kHid));
    for (int q = oW1; q < oB1; q++) h[q] = n1(rng);
    for (int q = oW2; q < oB2; q++) h[q] = n2(rng);
    for (int q = oW3; q < oB3; q++) h[q] = n3(rng);
    std::vector<float> z(kParams, 0.f);
    ok(sdev(hipMemcpy(s->params, h.data(), sizeof(float) * kParams, hipMemcpyHostToDevice), "upload"));
    ok(sdev(hipMemcpy(s->adam_m, z.data(), sizeof(float) * kParams, hipMemcpyHostToDevice), "upload"));
    ok(sdev(hipMemcpy(s->adam_v, z.data(), sizeof(float) * kParams, hipMemcpyHostToDevice), "upload"));
    ok(sdev(hipMemcpy(ref_dev, p->ref_host.data(), sizeof(float) * p->ref_host.size(), hipMemcpyHostToDevice), "upload"));
  }
  if (st == MOREA_OK) {
    hipLaunchKernelGGL(k_refresh_bf16, dim3((kHid * kHid + 255) / 256), dim3(256), 0, 0, s->params, s->w1b, s->w2b);
    ok(sdev(hipGetLastError(), "refresh"));
    ok(sdev(launch_stats(s, ref_dev), "tet statistics"));
    ok(sdev(launch_image_copies(s), "image copies"));
    const std::vector<float4> bary = sample_points();
    ok(sdev(hipMemcpy(s->bary, bary.data(), sizeof(float4) * kPoints, hipMemcpyHostToDevice), "upload"));
    ok(sdev(hipMemcpy(s->edge_ends, ends.data(), sizeof(int2) * ends.size(), hipMemcpyHostToDevice), "upload"));
    ok(sdev(hipMemcpy(s->tet_edges, of_tet.data(), sizeof(int) * of_tet.size(), hipMemcpyHostToDevice), "upload"));
    ok(sdev(hipDeviceSynchronize(), "surrogate set-up"));
  }
  if (st == MOREA_OK) {
    // h_scale: the count-weighted mean of the tets' mean (I_s - I_t)^2 (the
    // reference mesh tiles the grid, so this is the mean over its voxels)
    std::vector<float> hs(8 * static_cast<size_t>(NT));
    std::vector<int> hc(NT);
    ok(sdev(hipMemcpy(hs.data(), s->stats, sizeof(float) * hs.size(), hipMemcpyDeviceToHost), "copy"));
    ok(sdev(hipMemcpy(hc.data(), s->counts, sizeof(int) * hc.size(), hipMemcpyDeviceToHost), "copy"));
    double num = 0.0, den = 0.0;
    for (int t = 0; t < NT; t++) {
      num += static_cast<double>(hc[t]) * hs[8 * static_cast<size_t>(t) + 6];
      den += hc[t];
    }
    const double hsc = den > 0.0 ? num / den : 0.0;
    s->h_scale = hsc > 0.0 && std::isfinite(hsc) ? static_cast<float>(hsc) : 1.f;
  }
  if (st != MOREA_OK) {
    for (void* a : s->allocs) (void)hipFree(a);
    delete s;
    return st;
  }
  *out = s;
  return MOREA_OK;
}

void morea_surrogate_destroy(morea_surrogate* s) {
  if (!s) return;
  (void)hipDeviceSynchronize();
  for (void* a : s->allocs) (void)hipFree(a);
  if (s->work.data) (void)hipFree(s->work.data);
  delete s;
}

morea_status morea_surrogate_features(morea_surrogate* s, const float* pts, int32_t pop, const float* parent_pts,
                                      int32_t n_parents, const void* parent_cache, const int32_t* parent_of,
                                      float* feats, void* stream) {
  if (!s || pop < 0 || n_parents < 0) return sfail(MOREA_EINVAL, "bad argument");
  const long long rows = static_cast<long long>(pop) * s->p->view.n_tets;
  if (rows == 0) return MOREA_OK;
  if (!pts || !feats || !parent_of || (n_parents > 0 && (!parent_pts || !parent_cache)))
    return sfail(MOREA_EINVAL, "NULL argument");
  if (rows > (1LL << 31) / 4) return sfail(MOREA_ERANGE, "too many rows");
  const Parents Q{parent_pts, static_cast<const Record*>(parent_cache), parent_of, n_parents};
  const dim3 grid(static_cast<unsigned>((rows + 255) / 256));
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (big_quads(s->p->view))
    hipLaunchKernelGGL(k_features<true>, grid, dim3(256), 0, st, s->p->view, pts, Q, feature_inputs(s), pop, feats);
  else
    hipLaunchKernelGGL(k_features<false>, grid, dim3(256), 0, st, s->p->view, pts, Q, feature_inputs(s), pop, feats);
  return sdev(hipGetLastError(), "features");
}

morea_status morea_surrogate_targets(morea_surrogate* s, const void* cache, int32_t pop, const void* parent_cache,
                                     int32_t n_parents, const int32_t* parent_of, float* targets, void* stream) {
  if (!s || pop < 0 || n_parents < 0) return sfail(MOREA_EINVAL, "bad argument");
  const long long rows = static_cast<long long>(pop) * s->p->view.n_tets;
  if (rows == 0) return MOREA_OK;
  if (!cache || !targets || !parent_of || (n_parents > 0 && !parent_cache))
    return sfail(MOREA_EINVAL, "NULL argument");
  if (rows > (1LL << 31) - 256) return sfail(MOREA_ERANGE, "too many rows");
  const Parents Q{nullptr, static_cast<const Record*>(parent_cache), parent_of, n_parents};
  hipLaunchKernelGGL(k_targets, dim3(static_cast<unsigned>((rows + 255) / 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), static_cast<const Record*>(cache), s->p->view.n_tets,
                     static_cast<int>(rows), Q, 1.f / s->h_scale, targets);
  return sdev(hipGetLastError(), "targets");
}

morea_status morea_surrogate_train_step(morea_surrogate* s, const float* feats, const float* targets,
                                        int32_t n_rows, float lr, float* loss_out, void* stream) {
  return train_launch(s, feats, targets, n_rows, lr, nullptr, loss_out, static_cast<hipStream_t>(stream));
}

morea_status morea_surrogate_gradients(morea_surrogate* s, const float* feats, const float* targets,
                                       int32_t n_rows, float* grads, float* loss_out, void* stream) {
  if (!grads) return sfail(MOREA_EINVAL, "grads is NULL");
  return train_launch(s, feats, targets, n_rows, 0.f, grads, loss_out, static_cast<hipStream_t>(stream));
}

morea_status morea_surrogate_predict_rows(morea_surrogate* s, const float* feats, int32_t n_rows,
                                          float* pred, void* stream) {
  if (!s || !feats || !pred || n_rows < 0) return sfail(MOREA_EINVAL, "bad argument");
  if (n_rows == 0) return MOREA_OK;
  const int waves = (n_rows + kRowTile - 1) / kRowTile;
  hipLaunchKernelGGL(k_predict_rows, dim3((waves + 3) / 4), dim3(256), 0, static_cast<hipStream_t>(stream),
                     feats, n_rows, s->w1b, s->w2b, s->params, pred);
  return sdev(hipGetLastError(), "predict");
}

morea_status morea_surrogate_prescreen(morea_surrogate* s, const float* pts, int32_t pop, const float* parent_pts,
                                       int32_t n_parents, const void* parent_cache, const int32_t* parent_of,
                                       float* score, void* stream) {
  if (!s || pop < 0 || n_parents < 0) return sfail(MOREA_EINVAL, "bad argument");
  if (pop == 0) return MOREA_OK;
  if (!pts || !score || !parent_of || (n_parents > 0 && (!parent_pts || !parent_cache)))
    return sfail(MOREA_EINVAL, "NULL argument");
  const ProblemView& P = s->p->view;
  // tets per work item: as many as leave kPreItems items, a power of two up to kMaxTetRun
  const long long groups = (static_cast<long long>(pop) + kPreCands - 1) / kPreCands;
  int tet_run = 1;
  while (tet_run < kMaxTetRun && 2 * tet_run * kPreItems <= P.n_tets * groups) tet_run *= 2;
  const int n_runs = (P.n_tets + tet_run - 1) / tet_run;
  const size_t rows = static_cast<size_t>(n_parents) * P.n_tets;
  const size_t pm_bytes = (sizeof(float4) * rows + 255) / 256 * 256;
  const size_t part_bytes = (sizeof(float2) * static_cast<size_t>(n_runs) * pop + 255) / 256 * 256;
  // candidates laid out by columns at a time: all, unless that exceeds kColBytes
  const size_t col_bytes = 9 * sizeof(float) * static_cast<size_t>(P.n_points);
  const size_t n_shared = static_cast<size_t>(P.n_points) + s->n_edges;
  const size_t cand_bytes = col_bytes + sizeof(float) * n_shared;
  const size_t fits = std::max<size_t>(kPreCands, kColBytes / cand_bytes / kPreCands * kPreCands);
  const size_t all = static_cast<size_t>(std::max(pop, n_parents));
  hipError_t e = hipSuccess;
  size_t asked = 0;
  const size_t most = reserve_slab(
      s->work, pm_bytes + part_bytes, cand_bytes, kPreCands, std::min(fits, all),
      [&](size_t bytes) {
        void* d = nullptr;
        asked = bytes;
        e = hipMalloc(&d, bytes);
        if (e != hipSuccess) (void)hipGetLastError();
        return e == hipSuccess ? d : nullptr;
      },
      [](void* d) { (void)hipFree(d); });   // waits for the device
  if (most == 0) return sfail(MOREA_ENOMEM, "hipMalloc(%zu): %s", asked, hipGetErrorString(e));
  const int slab = static_cast<int>(most);
  char* work = static_cast<char*>(s->work.data);
  float4* pmeans = reinterpret_cast<float4*>(work);
  float2* partial = reinterpret_cast<float2*>(work + pm_bytes);
  float* cols = reinterpret_cast<float*>(work + pm_bytes + part_bytes);
  float* hs = cols + col_bytes / sizeof(float) * most;
  const hipStream_t st = static_cast<hipStream_t>(stream);
  const FeatureInputs F = feature_inputs(s);
  const Parents Q{parent_pts, static_cast<const Record*>(parent_cache), parent_of, n_parents};
  const unsigned col_tiles = static_cast<unsigned>((P.n_points + kColPoints - 1) / kColPoints);
  for (int first = 0; first < n_parents; first += slab) {
    const int n = std::min(slab, n_parents - first);
    hipLaunchKernelGGL(k_columns<6>, dim3(col_tiles, (n + kColCands - 1) / kColCands, 6), dim3(256), 0, st, parent_pts,
                       first, n, P.n_points, Q, cols);
    const dim3 grid(static_cast<unsigned>((static_cast<size_t>(n) * P.n_tets + 255) / 256));
    const dim3 shared_grid(shared_blocks(n_shared, n));
    if (big_quads(P)) {
      hipLaunchKernelGGL((k_shared_points<true, 6>), shared_grid, dim3(256), 0, st, P, cols, n, s->edge_ends,
                         s->n_edges, F, hs);
      hipLaunchKernelGGL(k_parent_means<true>, grid, dim3(256), 0, st, P, cols, hs, s->tet_edges, first, n, Q.rec, F,
                         pmeans);
    } else {
      hipLaunchKernelGGL((k_shared_points<false, 6>), shared_grid, dim3(256), 0, st, P, cols, n, s->edge_ends,
                         s->n_edges, F, hs);
      hipLaunchKernelGGL(k_parent_means<false>, grid, dim3(256), 0, st, P, cols, hs, s->tet_edges, first, n, Q.rec, F,
                         pmeans);
    }
  }
  for (int first = 0; first < pop; first += slab) {
    const int n = std::min(slab, pop - first);
    hipLaunchKernelGGL(k_columns<9>, dim3(col_tiles, (n + kColCands - 1) / kColCands, 6), dim3(256), 0, st, pts, first,
                       n, P.n_points, Q, cols);
    const long long items = static_cast<long long>(n_runs) * ((n + kPreCands - 1) / kPreCands);
    const dim3 grid(static_cast<unsigned>(std::min<long long>((items + kPreWaves - 1) / kPreWaves, kPreItems / kPreWaves)));
    const dim3 block(64 * kPreWaves);
    const dim3 shared_grid(shared_blocks(n_shared, n));
    if (big_quads(P)) {
      hipLaunchKernelGGL((k_shared_points<true, 9>), shared_grid, dim3(256), 0, st, P, cols, n, s->edge_ends,
                         s->n_edges, F, hs);
      hipLaunchKernelGGL(k_prescreen<true>, grid, block, 0, st, P, cols, hs, s->tet_edges, parent_of + first, n_parents,
                         F, pmeans, s->params, s->w1b, s->w2b, n, tet_run, partial + first, pop);
    } else {
      hipLaunchKernelGGL((k_shared_points<false, 9>), shared_grid, dim3(256), 0, st, P, cols, n, s->edge_ends,
                         s->n_edges, F, hs);
      hipLaunchKernelGGL(k_prescreen<false>, grid, block, 0, st, P, cols, hs, s->tet_edges, parent_of + first,
                         n_parents, F, pmeans, s->params, s->w1b, s->w2b, n, tet_run, partial + first, pop);
    }
  }
  const auto reduce = tet_run == 8 ? k_prescreen_reduce<1> : (tet_run == 4 ? k_prescreen_reduce<2> :
                      (tet_run == 2 ? k_prescreen_reduce<4> : k_prescreen_reduce<8>));
  hipLaunchKernelGGL(reduce, dim3((pop + 63) / 64), dim3(64 * kScoreGroups), 0, st, partial, n_runs, pop, Q, score);
  return sdev(hipGetLastError(), "prescreen");
}

morea_status morea_surrogate_select(const float* score, int32_t n, int32_t k, const float* pts,
                                    int32_t n_points, int32_t* idx_out, float* selected_pts, void* stream) {
  if (!score || !idx_out || n < 1 || n > 8192 || k < 1 || k > n)
    return sfail(MOREA_EINVAL, "need 1 <= k <= n <= 8192 and non-NULL arrays");
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_select, dim3(1), dim3(1024), 0, st, score, n, k, idx_out);
  if (pts && selected_pts) {
    const int per = 6 * n_points;
    hipLaunchKernelGGL(k_gather, dim3(1024), dim3(256), 0, st, pts, idx_out, k, per, selected_pts);
  }
  return sdev(hipGetLastError(), "select");
}

morea_status morea_surrogate_get_params(morea_surrogate* s, float* host_params) {
  if (!s || !host_params) return sfail(MOREA_EINVAL, "bad argument");
  return sdev(hipMemcpy(host_params, s->params, sizeof(float) * kParams, hipMemcpyDeviceToHost), "copy");
}

morea_status morea_surrogate_set_params(morea_surrogate* s, const float* host_params) {
  if (!s || !host_params) return sfail(MOREA_EINVAL, "bad argument");
  morea_status st = sdev(hipMemcpy(s->params, host_params, sizeof(float) * kParams, hipMemcpyHostToDevice), "copy");
  if (st != MOREA_OK) return st;
  hipLaunchKernelGGL(k_refresh_bf16, dim3((kHid * kHid + 255) / 256), dim3(256), 0, 0, s->params, s->w1b, s->w2b);
  st = sdev(hipGetLastError(), "refresh");
  if (st == MOREA_OK) st = sdev(hipDeviceSynchronize(), "set params");
  return st;
}

morea_status morea_surrogate_scale(const morea_surrogate* s, float* h_scale) {
  if (!s || !h_scale) return sfail(MOREA_EINVAL, "bad argument");
  *h_scale = s->h_scale;
  return MOREA_OK;
}

morea_status morea_surrogate_stats(morea_surrogate* s, float* host_stats, int32_t* host_counts) {
  if (!s || !host_stats) return sfail(MOREA_EINVAL, "bad argument");
  const int NT = s->p->view.n_tets;
  morea_status st = sdev(hipMemcpy(host_stats, s->stats, sizeof(float) * 8 * NT, hipMemcpyDeviceToHost), "copy");
  if (st == MOREA_OK && host_counts)
    st = sdev(hipMemcpy(host_counts, s->counts, sizeof(int) * NT, hipMemcpyDeviceToHost), "copy");
  return st;
}

}  // extern "C"
