// Sobol-sampled objective evaluation: the paper's own estimator of the
// intensity and guidance terms (App. A.2).  Each tet of each mesh is sampled
// at N random points spread uniformly through its barycentric coordinates,
// N = round(rate * volume); a point takes four numbers r_j of a Sobol
// sequence seeded from the tet's coordinates, lambda_j = -ln r_j / sum_k
// (-ln r_k), and is p = v_0 + sum_{i>=1} lambda_i (v_i - v_0) in the sampled
// tet and q = w_0 + sum_{i>=1} lambda_i (w_i - w_0) in the other mesh's
// tet.  h (Sec. 4.1.2) compares the trilinear values of the two images at p
// and q, with foreground decided on each stencil's exact support; the
// guidance term (Sec. 4.1.3) compares the two distance maps at p and q for
// the sets whose interpolated own distance is below the radius.  Magnitude
// and folds are those of the full evaluation (Sec. 4.1.1, App. A.4).
//
// The sequence: 4 dimensions with 32-bit direction numbers from the
// primitive polynomials 1, x + 1, x^2 + x + 1, x^3 + x + 1 (initial
// numbers (1), (1, 3), (1, 3, 1)), point n in natural order (the XOR of the
// direction numbers of the set bits of n), randomised by a digital shift of
// four words from a SplitMix64 hash of the seed, the direction and the
// tet's 12 fixed-point coordinates.  r_j = (2 floor(u_j / 2^9) + 1) 2^-24.
// -ln is the FP32 atanh series of ln m, m in [sqrt(1/2), sqrt(2)], to s^11.
// The points are formed in FP32 with explicit FMAs and correctly rounded
// divisions, contraction off: which trilinear corners a point's stencil
// supports depends on its bits, and these are the bits the definition
// fixes.
//
// One 64-lane wave per (candidate, tet); a block's waves take candidates of
// one tet where the images are staged; both directions in turn; sample n
// of a direction is taken by lane n % 64.  Since lane < 64, the Sobol
// integer of n = 64 k + lane is the XOR of that of the lane (per lane, once
// per item) and that of 64 k (wave-uniform, scalar, once per batch).
//
// What bounds it: the vector instructions, 243 lane instructions a point, and
// where the images are not staged in LDS the gathers, each lane in a cache line
// of its own (46 cycles of a CU for 64).  The instructions were 5,760 a wave (88%
// of the issue slots, 232 per point to form it and find its cell; now 3,510, 86%
// of the slots): the divisions are the correctly rounded ones without scaling
// for extreme operands, the logarithm is halved (the ratios do not change),
// which saves its scalings, and tets that stay in the grid's border cells take
// a path without bounds tests on which one cell serves the images and the
// distance maps, a row's two corners are one load and values are read only
// where both points are foreground.  128x128x96, population 128, rate 1: 4.11
// -> 2.90, 4.62 -> 3.34, 4.94 -> 3.67 ms (three images); with the images in LDS
// 2.82, 2.96, 3.12 ms.
// At six waves a SIMD the staged form spills 14 scalar registers into lanes of
// vector registers and 5 vector registers to scratch (24 bytes a lane, most of
// the 1.2 GB that a launch of 512 candidates writes, 2% of the copy rate), the
// other form 1 (none in the compiler's default schedule).
#include <math.h>
#include <stdio.h>

#include <type_traits>

#include "morea_internal.h"
#include "morea_sobol_point.h"

namespace morea {
namespace sobol {

constexpr int kMaxSamples = 1 << 20;          // per tet and direction
constexpr uint64_t kGolden = 0x9e3779b97f4a7c15ull;

struct DirTable {
  uint32_t v[4][32];
};

// Direction numbers V_j[b] = m_{b+1} 2^(31-b), m_k = m_{k-s} XOR
// (XOR over i = 1..s of c_i 2^i m_{k-i}) with c_i the coefficient of
// x^(s-i) of the degree-s primitive polynomial (c_s = 1).
constexpr DirTable make_directions() {
  DirTable t{};
  for (int b = 0; b < 32; b++) t.v[0][b] = 0x80000000u >> b;
  const uint32_t poly[3] = {0x3u, 0x7u, 0xbu};   // x + 1, x^2 + x + 1, x^3 + x + 1
  const int degree[3] = {1, 2, 3};
  const uint64_t first[3][3] = {{1, 0, 0}, {1, 3, 0}, {1, 3, 1}};
  for (int j = 0; j < 3; j++) {
    const int s = degree[j];
    uint64_t m[33] = {};
    for (int k = 1; k <= s; k++) m[k] = first[j][k - 1];
    for (int k = s + 1; k <= 32; k++) {
      uint64_t x = m[k - s];
      for (int i = 1; i <= s; i++)
        if ((poly[j] >> (s - i)) & 1u) x ^= m[k - i] << i;
      m[k] = x;
    }
    for (int b = 0; b < 32; b++) t.v[j + 1][b] = static_cast<uint32_t>(m[b + 1] << (31 - b));
  }
  return t;
}

// Bits 0..5 of the sample index, whose XOR is the lane's, and the XOR of the
// direction numbers of bits 6 .. 6 + c, by which the integer of 64 k changes
// when k + 1 ends in c zero bits.  r takes bits 9..31: shifted down by 8, the
// lowest bit cleared (the lane's words set it).
struct StepTable {
  uint32_t v[26][4];
};

constexpr DirTable kDirections = make_directions();

constexpr StepTable make_steps() {
  StepTable t{};
  for (int j = 0; j < 4; j++) {
    uint32_t x = 0;
    for (int c = 0; c < 26; c++) {
      x ^= kDirections.v[j][6 + c];
      t.v[c][j] = (x >> 8) & ~1u;
    }
  }
  return t;
}

__constant__ __attribute__((aligned(16))) StepTable kSteps = make_steps();

__device__ __forceinline__ uint64_t splitmix(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// Sum over the wave in lane 63: within rows of 16 lanes, then across them
// (DPP: no LDS round trips and no shuffle addresses kept in registers).
template <int ctrl, int rows>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rows, 0xf, false));
}

__device__ __forceinline__ float wave_sum_63(float v) {
  v += dpp<0x111, 0xf>(v);
  v += dpp<0x112, 0xf>(v);
  v += dpp<0x114, 0xf>(v);
  v += dpp<0x118, 0xf>(v);
  v += dpp<0x142, 0xa>(v);
  v += dpp<0x143, 0xc>(v);
  return v;
}

__device__ __forceinline__ double wave_sum_d(double v) {
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

template <int ST>
__device__ __forceinline__ float ld(const void* base, int idx) {
  if constexpr (ST == kF32) {
    return static_cast<const float*>(base)[idx];
  } else if constexpr (ST == kBF16) {
    return __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t*>(base)[idx]) << 16);
  } else {
    return static_cast<float>(static_cast<const _Float16*>(base)[idx]);
  }
}

// Trilinear value and exact-support foreground of an image (zero padding) at
// an FP32 point in grid coordinates.
template <int ST>
__device__ __forceinline__ float image_at(const ProblemView& P, const void* img, const uint16_t* cells, float x,
                                          float y, float z, bool& fg) {
  const float kx = floorf(x), ky = floorf(y), kz = floorf(z);
  const float fx = x - kx, fy = y - ky, fz = z - kz;
  const int ix = static_cast<int>(kx), iy = static_cast<int>(ky), iz = static_cast<int>(kz);
  fg = false;
  // both corners of an axis lie outside the grid when k <= -2 or k >= n
  if (kx < -1.f || ky < -1.f || kz < -1.f || ix > P.nx - 1 || iy > P.ny - 1 || iz > P.nz - 1) return 0.f;
  const int i0 = (iz + 1) * P.pxy + (iy + 1) * P.px + ix + 1;
  // a cell without a positive corner is background whatever the support
  const unsigned code = cells[i0];
  if (!(code & 1u)) return 0.f;
  const int i1 = i0 + P.pxy;
  const float c000 = ld<ST>(img, i0), c100 = ld<ST>(img, i0 + 1);
  const float c010 = ld<ST>(img, i0 + P.px), c110 = ld<ST>(img, i0 + P.px + 1);
  const float c001 = ld<ST>(img, i1), c101 = ld<ST>(img, i1 + 1);
  const float c011 = ld<ST>(img, i1 + P.px), c111 = ld<ST>(img, i1 + P.px + 1);
  if (code & 2u) {
    fg = true;    // every corner is positive, so is every supported one
  } else {
    const bool ux = fx > 0.f, uy = fy > 0.f, uz = fz > 0.f;
    const bool f0 = c000 > 0.f || (ux && c100 > 0.f) || (uy && c010 > 0.f) || (ux && uy && c110 > 0.f);
    const bool f1 = c001 > 0.f || (ux && c101 > 0.f) || (uy && c011 > 0.f) || (ux && uy && c111 > 0.f);
    fg = f0 || (uz && f1);
    if (!fg) return 0.f;
  }
  const float x00 = fmaf(fx, c100 - c000, c000), x10 = fmaf(fx, c110 - c010, c010);
  const float x01 = fmaf(fx, c101 - c001, c001), x11 = fmaf(fx, c111 - c011, c011);
  const float y0 = fmaf(fy, x10 - x00, x00), y1 = fmaf(fy, x11 - x01, x01);
  return fmaf(fz, y1 - y0, y0);
}

// Stencil of a distance map (edge clamping): the point clamped into
// [0, n - 1] per axis, the cell below it capped at n - 2 (at 0 for n = 1),
// its first padded element and fractions.
struct MapCell {
  int i0;
  float fx, fy, fz;
};

__device__ __forceinline__ MapCell map_cell(const ProblemView& P, float x, float y, float z) {
  const float cx = fminf(fmaxf(x, 0.f), static_cast<float>(P.nx - 1));
  const float cy = fminf(fmaxf(y, 0.f), static_cast<float>(P.ny - 1));
  const float cz = fminf(fmaxf(z, 0.f), static_cast<float>(P.nz - 1));
  const int ix = max(min(static_cast<int>(floorf(cx)), P.nx - 2), 0);
  const int iy = max(min(static_cast<int>(floorf(cy)), P.ny - 2), 0);
  const int iz = max(min(static_cast<int>(floorf(cz)), P.nz - 2), 0);
  return MapCell{(iz + 1) * P.pxy + (iy + 1) * P.px + ix + 1, cx - static_cast<float>(ix),
                 cy - static_cast<float>(iy), cz - static_cast<float>(iz)};
}

__device__ __forceinline__ float map_at(const ProblemView& P, const float* m, const MapCell& c) {
  const int i0 = c.i0, i1 = c.i0 + P.pxy;
  const float x00 = fmaf(c.fx, m[i0 + 1] - m[i0], m[i0]);
  const float x10 = fmaf(c.fx, m[i0 + P.px + 1] - m[i0 + P.px], m[i0 + P.px]);
  const float x01 = fmaf(c.fx, m[i1 + 1] - m[i1], m[i1]);
  const float x11 = fmaf(c.fx, m[i1 + P.px + 1] - m[i1 + P.px], m[i1 + P.px]);
  const float y0 = fmaf(c.fy, x10 - x00, x00), y1 = fmaf(c.fy, x11 - x01, x01);
  return fmaf(c.fz, y1 - y0, y0);
}

// Two consecutive stored values at any element, by one load.
struct __attribute__((aligned(4))) F2 {
  float a, b;
};
struct __attribute__((aligned(2))) H2 {
  uint16_t a, b;
};

template <int ST>
__device__ __forceinline__ void ld_pair(const void* base, uint32_t e, float& a, float& b) {
  if constexpr (ST == kF32) {
    const F2 v = *reinterpret_cast<const F2*>(static_cast<const char*>(base) + (e << 2));
    a = v.a;
    b = v.b;
  } else {
    const H2 v = *reinterpret_cast<const H2*>(static_cast<const char*>(base) + (e << 1));
    if constexpr (ST == kBF16) {
      a = __uint_as_float(static_cast<uint32_t>(v.a) << 16);
      b = __uint_as_float(static_cast<uint32_t>(v.b) << 16);
    } else {
      a = static_cast<float>(__builtin_bit_cast(_Float16, v.a));
      b = static_cast<float>(__builtin_bit_cast(_Float16, v.b));
    }
  }
}

template <int ST>
__device__ __forceinline__ const void* at(const void* base, int e) {
  return static_cast<const char*>(base) + static_cast<ptrdiff_t>(e) * (ST == kF32 ? 4 : 2);
}

// The cell of a point in [-1, n) per axis, from its padded lower corner
// element, and the point's fractions in it.  Image borders hold 0 and map
// borders repeat the nearest value, so both interpolate in this cell as the
// definitions have it (zero padding, edge clamping).
struct Cell {
  uint32_t e;
  float fx, fy, fz;
};

__device__ __forceinline__ int floor_int(float x) {
  int i;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(x));
  return i;
}

__device__ __forceinline__ Cell inner_cell(const ProblemView& P, const float p[3]) {
  Cell c;
  c.e = static_cast<uint32_t>(__mul24(floor_int(p[2]), P.pxy) + (__mul24(floor_int(p[1]), P.px) +
                                                                 (floor_int(p[0]) + (P.pxy + P.px + 1))));
  c.fx = __builtin_amdgcn_fractf(p[0]);
  c.fy = __builtin_amdgcn_fractf(p[1]);
  c.fz = __builtin_amdgcn_fractf(p[2]);
  return c;
}

// The 8 corners of a cell: v[2 r], v[2 r + 1] of row r = (0, 0), (1, 0),
// (0, 1), (1, 1) in (y, z).
template <int ST>
__device__ __forceinline__ void corners(const ProblemView& P, const void* base, uint32_t e, float v[8]) {
  ld_pair<ST>(base, e, v[0], v[1]);
  ld_pair<ST>(at<ST>(base, P.px), e, v[2], v[3]);
  ld_pair<ST>(at<ST>(base, P.pxy), e, v[4], v[5]);
  ld_pair<ST>(at<ST>(base, P.pxy + P.px), e, v[6], v[7]);
}

__device__ __forceinline__ float trilinear(const float v[8], const Cell& c) {
  const float x00 = fmaf(c.fx, v[1] - v[0], v[0]), x10 = fmaf(c.fx, v[3] - v[2], v[2]);
  const float x01 = fmaf(c.fx, v[5] - v[4], v[4]), x11 = fmaf(c.fx, v[7] - v[6], v[6]);
  const float y0 = fmaf(c.fy, x10 - x00, x00), y1 = fmaf(c.fy, x11 - x01, x01);
  return fmaf(c.fz, y1 - y0, y0);
}

// Whether a supported corner (nonzero weight) is positive.
__device__ __forceinline__ bool support(const float v[8], const Cell& c) {
  const bool ux = c.fx > 0.f, uy = c.fy > 0.f, uz = c.fz > 0.f;
  const bool f0 = v[0] > 0.f || (ux && v[1] > 0.f) || (uy && v[2] > 0.f) || (ux && uy && v[3] > 0.f);
  const bool f1 = v[4] > 0.f || (ux && v[5] > 0.f) || (uy && v[6] > 0.f) || (ux && uy && v[7] > 0.f);
  return f0 || (uz && f1);
}

// The terms of a point are rounded alike in every form (no contraction), so
// that a candidate's sums do not depend on the form, hence the population, it
// is evaluated in.

// The guidance term of the sets in `bits` at cells cp, cq, added to g.
__device__ __forceinline__ void map_terms(const ProblemView& P, unsigned bits, const float* map_own,
                                          const float* map_oth, const float* set_w, const Cell& cp, const Cell& cq,
                                          float& g) {
#pragma clang fp contract(off)
  for (int s = 0; s < P.n_sets; s++) {
    if ((bits >> s) & 1u) {
      float v[8];
      const size_t first = static_cast<size_t>(s) * P.pvox;
      corners<kF32>(P, map_own + first, cp.e, v);
      const float dn = trilinear(v, cp);
      if (dn < P.radius) {
        corners<kF32>(P, map_oth + first, cq.e, v);
        const float diff = dn - trilinear(v, cq);
        g = fmaf(set_w[s] * (P.radius - dn) * P.inv_radius, diff * diff, g);
      }
    }
  }
}

// h and g of a point p of the sampled tet and q of the other one, both in
// [-1, n) per axis, added to h and g.
template <int ST>
__device__ __forceinline__ void inner_sample(const ProblemView& P, const void* img_own, const void* img_oth,
                                             const uint16_t* cells_own, const uint16_t* cells_oth,
                                             const float* map_own, const float* map_oth, const float* set_w,
                                             const float p[3], const float q[3], float& h, float& g) {
#pragma clang fp contract(off)
  const Cell cp = inner_cell(P, p), cq = inner_cell(P, q);
  const unsigned kp = cells_own[cp.e], kq = cells_oth[cq.e];
  // with all weights nonzero a point is foreground where its cell has a
  // positive corner: h needs the values only where both points are
  const bool pa = (kp & 1u) != 0u, pb = (kq & 1u) != 0u;
  const bool flat = cp.fx * cp.fy * cp.fz * cq.fx * cq.fy * cq.fz == 0.f;
  if ((pa && pb) || (flat && (pa || pb))) {
    float u[8], v[8];
    corners<ST>(P, img_own, cp.e, u);
    corners<ST>(P, img_oth, cq.e, v);
    float a = trilinear(u, cp), b = trilinear(v, cq);
    bool fa = pa, fb = pb;
    if (__ballot(flat)) {
      asm volatile("");   // kept as a branch
      fa = support(u, cp);
      fb = support(v, cq);
      a = fa ? a : 0.f;
      b = fb ? b : 0.f;
    }
    const float d = a - b;
    h += fa != fb ? 1.f : d * d;
  } else {
    h += pa != pb ? 1.f : 0.f;
  }
  // sets within the radius at one of the cell's corners (if at none, the
  // interpolated distance is not below it either)
  const unsigned bits = kp >> 8;
  if (__ballot(bits != 0u)) map_terms(P, bits, map_own, map_oth, set_w, cp, cq, g);
}

// The boxes of the two images (0 source, 1 target) that a block's tets lie in:
// values as FP32 and the cells' band bytes, staged once for the block's
// candidates (their tets are one mesh tet, moved a little) and both
// directions.  Two blocks of 12 waves per CU (of 8 waves with more registers
// each: 14% longer).
//
// Staging has a fixed cost, a block's waves waiting for each other twice,
// which many samples in a block repay; and a block whose waves do not divide
// over the four SIMDs leaves some of them waiting, where the waves of the plain
// form fill them.  Plain against staged in us, 3,072 tets of cells of edge n,
// `per` waves a block, 60 candidates (per 12) or 22 (per 11):
//   per 12: n = 12, 432 samples a tet: 1,134 : 1,125; n = 14, 366: 1,071 : 1,053;
//           n = 15, 450: 1,281 : 1,176, 844: 2,182 : 1,686
//   per 11: n = 14, 457: 498 : 511; n = 15, 562: 602 : 581
// and as the quotient, n = 15: per 9, 562 samples: 0.98, 703: 1.07; per 8, 450:
// 0.98, 562: 1.08; per 7, 844: 1.10; per 4, 1,125: 0.99, 1,688: 1.10; per 3,
// 1,688: 0.99, 2,812: 1.08; per 2, 9,000: 0.81; per 1: 0.63.
// So from 4,900 samples of a block's candidates, times the share of the SIMDs'
// turns that its waves take, and from 3 waves on: over 925 sizes (1 to 128
// candidates, 173 to 10,900 samples) 0.3% slower than the better form of each.
// With fewer blocks than the chip holds the line is higher (384 tets, 12
// candidates, n = 14: 0.96 at 457 samples, 1.01 at 686); from n = 17 on the
// boxes do not fit.  128x128x96 with 3,402 tets, population 128: 2.90 -> 2.82,
// 3.34 -> 2.96 and 3.67 -> 3.12 ms (three images).
constexpr int kBlockWaves = 12;
constexpr int kBoxVoxels = 16256;
constexpr double kStageSamples = 4900.0;   // of a block's candidates
constexpr int kStageWaves = 3;

struct BoxLds {
  float v[kBoxVoxels];
  uint8_t band[kBoxVoxels];
  int lo[2][3], hi[2][3];   // padded cells of the waves' tets
  int points;               // samples of the block
  int found[2];             // bit 0: a positive value in the box, bits 8..15: its band bits
};
static_assert(sizeof(BoxLds) <= 81920, "two blocks per CU");

// One of them, in scalar registers.
struct Box {
  int first, sy, sz;   // element of the padded origin's cell in v / band, strides
};

__device__ __forceinline__ bool box_corners(const BoxLds& L, int e, float v[8], int sy, int sz) {
  const float *r0 = L.v + e, *r1 = r0 + sy, *r2 = r0 + sz, *r3 = r1 + sz;
  v[0] = r0[0];
  v[1] = r0[1];
  v[2] = r1[0];
  v[3] = r1[1];
  v[4] = r2[0];
  v[5] = r2[1];
  v[6] = r3[0];
  v[7] = r3[1];
  // a positive corner, by the words as integers (no NaN; -0 is negative)
  int top = __float_as_int(v[0]);
#pragma unroll
  for (int k = 1; k < 8; k++) top = max(top, __float_as_int(v[k]));
  return top > 0;
}

// h of inner points from the staged boxes, then g as inner_sample's.
__device__ __forceinline__ void staged_sample(const ProblemView& P, const BoxLds& L, const Box& bo, const Box& bt,
                                              bool any_fg, bool any_band, const float* map_own, const float* map_oth,
                                              const float* set_w, const float p[3], const float q[3], float& h,
                                              float& g) {
#pragma clang fp contract(off)
  const int px = floor_int(p[0]), py = floor_int(p[1]), pz = floor_int(p[2]);
  const int qx = floor_int(q[0]), qy = floor_int(q[1]), qz = floor_int(q[2]);
  const int ep = __mul24(pz, bo.sz) + (__mul24(py, bo.sy) + (px + bo.first));
  const int eq = __mul24(qz, bt.sz) + (__mul24(qy, bt.sy) + (qx + bt.first));
  const Cell cp{0u, __builtin_amdgcn_fractf(p[0]), __builtin_amdgcn_fractf(p[1]), __builtin_amdgcn_fractf(p[2])};
  const Cell cq{0u, __builtin_amdgcn_fractf(q[0]), __builtin_amdgcn_fractf(q[1]), __builtin_amdgcn_fractf(q[2])};
  if (any_fg) {
    float u[8], v[8];
    bool fa = box_corners(L, ep, u, bo.sy, bo.sz), fb = box_corners(L, eq, v, bt.sy, bt.sz);
    if (__ballot(fa || fb)) {
      float a = trilinear(u, cp), b = trilinear(v, cq);
      const bool flat = cp.fx * cp.fy * cp.fz * cq.fx * cq.fy * cq.fz == 0.f;
      if (__ballot(flat)) {
        asm volatile("");   // kept as a branch
        fa = support(u, cp);
        fb = support(v, cq);
        a = fa ? a : 0.f;
        b = fb ? b : 0.f;
      }
      const float d = a - b;
      h += fa != fb ? 1.f : d * d;
    }
  }
  if (any_band) {
    const unsigned bits = L.band[ep];
    if (__ballot(bits != 0u)) map_terms(P, bits, map_own, map_oth, set_w, inner_cell(P, p), inner_cell(P, q), g);
  }
}

// As inner_sample for any points: bounds tests for the images, clamped cells
// for the maps.
template <int ST>
__device__ __forceinline__ void outer_sample(const ProblemView& P, const void* img_own, const void* img_oth,
                                             const uint16_t* cells_own, const uint16_t* cells_oth,
                                             const float* map_own, const float* map_oth, const float* set_w,
                                             const float p[3], const float q[3], float& h, float& g) {
#pragma clang fp contract(off)
  bool fa, fb;
  const float a = image_at<ST>(P, img_own, cells_own, p[0], p[1], p[2], fa);
  const float b = image_at<ST>(P, img_oth, cells_oth, q[0], q[1], q[2], fb);
  h += (fa && fb) ? (a - b) * (a - b) : (fa == fb ? 0.f : 1.f);
  if (P.n_sets == 0) return;
  const MapCell cp = map_cell(P, p[0], p[1], p[2]);
  unsigned bits = cells_own[cp.i0] >> 8;
  if (bits == 0u) return;
  const MapCell cq = map_cell(P, q[0], q[1], q[2]);
  for (; bits; bits &= bits - 1u) {
    const int s = __builtin_ctz(bits);
    const float dn = map_at(P, map_own + static_cast<size_t>(s) * P.pvox, cp);
    if (dn < P.radius) {
      const float diff = dn - map_at(P, map_oth + static_cast<size_t>(s) * P.pvox, cq);
      g = fmaf(set_w[s] * (P.radius - dn) * P.inv_radius, diff * diff, g);
    }
  }
}

// The problem's view, the kernel's first argument, read again from the kernel
// arguments (scalar loads): its words would otherwise stay live in scalar
// registers and be spilled into lanes of vector registers.
typedef const __attribute__((address_space(4))) ProblemView* ViewPtr;

__device__ __forceinline__ ProblemView view() {
  ViewPtr p = (ViewPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const ProblemView*)p;
}

// 6 x signed volume of snapped vertices (exact: coordinates below 2^19).
__device__ __forceinline__ int64_t det6(const int v[4][3]) {
  const int64_t a0 = v[1][0] - v[0][0], a1 = v[1][1] - v[0][1], a2 = v[1][2] - v[0][2];
  const int64_t b0 = v[2][0] - v[0][0], b1 = v[2][1] - v[0][1], b2 = v[2][2] - v[0][2];
  const int64_t c0 = v[3][0] - v[0][0], c1 = v[3][1] - v[0][1], c2 = v[3][2] - v[0][2];
  return a0 * (b1 * c2 - b2 * c1) - a1 * (b0 * c2 - b2 * c0) + a2 * (b0 * c1 - b1 * c0);
}

// Each XCD (blocks dealt round-robin) gets one contiguous range of blocks, so
// neighbouring tets share its L2.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
  const int q = nb / 8, rem = nb % 8;
  const int x = b % 8, pos = b / 8;
  return x < rem ? x * (q + 1) + pos : rem * (q + 1) + (x - rem) * q + pos;
}

// Samples of a tet: its volume times the rate, rounded.
__device__ __forceinline__ int sample_count(int64_t D, double count_scale) {
  if (D == 0) return 0;
  const double x = floor(static_cast<double>(D < 0 ? -D : D) * count_scale + 0.5);
  return x > 0.0 ? (x >= kMaxSamples ? kMaxSamples : static_cast<int>(x)) : 0;
}

struct NoLds {};

// kStaged: a block takes one tet of `per` candidates, a wave each, `groups`
// blocks a tet.  Otherwise `per` = 4 waves take an item each.
template <int ST, bool kStaged>
__global__ __launch_bounds__(64 * (kStaged ? kBlockWaves : 4), 6) void k_eval_sobol(
    ProblemView P, const float* pts, int pop, int per, int groups, double inv_pop, double count_scale, uint64_t seed,
    const uint16_t* cells0, const uint16_t* cells1, Record* rec) {
  __shared__ std::conditional_t<kStaged, BoxLds, NoLds> L;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int block = xcd_remap(blockIdx.x, gridDim.x);
  int tet, cand;
  bool spare = false;
  if constexpr (kStaged) {
    tet = block / groups;
    const int first = (block - tet * groups) * per, last = min(pop, first + per) - 1;
    spare = first + wave > last;
    cand = min(first + wave, last);   // a wave to spare repeats the last
    if (threadIdx.x < 6) {
      (&L.lo[0][0])[threadIdx.x] = INT32_MAX;
      (&L.hi[0][0])[threadIdx.x] = INT32_MIN;
    }
    if (threadIdx.x < 2) L.found[threadIdx.x] = 0;
    if (threadIdx.x == 0) L.points = 0;
    __syncthreads();
  } else {
    const int item = block * 4 + wave;
    tet = static_cast<int>(static_cast<double>(item) * inv_pop);
    cand = item - tet * pop;
    if (cand < 0) {
      tet -= 1;
      cand += pop;
    } else if (cand >= pop) {
      tet += 1;
      cand -= pop;
    }
    if (tet >= P.n_tets) return;
    tet = __builtin_amdgcn_readfirstlane(tet);
    cand = __builtin_amdgcn_readfirstlane(cand);
  }
  const int lane = lane_id();
  Record* out = rec + (static_cast<size_t>(cand) * P.n_tets + tet) * 2;

  // snap (lane l < 24: mesh l / 12, vertex (l % 12) / 3, axis l % 3)
  const int4 tv = P.tets[tet];
  float coord = 0.f;
  if (lane < 24) {
    const int i = (lane % 12) / 3, k = lane % 3;
    const int v = i == 0 ? tv.x : (i == 1 ? tv.y : (i == 2 ? tv.z : tv.w));
    coord = pts[((static_cast<size_t>(cand) * 2 + lane / 12) * 3 + k) * P.n_points + v];
  }
  const bool ok = __ballot(lane >= 24 || fabsf(coord) < kCoordLimit) == ~0ull;
  if (!ok && !spare && lane < 2) out[lane] = Record{0.f, 0.f, 0u, 0.f, 0.f, 4u};
  if constexpr (!kStaged)
    if (!ok) return;
  if (!ok) coord = 0.f;   // no samples; the block's barriers are passed all the same
  // snapped coordinate of lane l < 24: mesh l / 12, vertex (l % 12) / 3, axis l % 3
  const int fix = lane < 24 ? static_cast<int>(rintf(coord * kFixOne)) : 0;

  // whether each tet stays a 2^-4 voxel inside [-1, n): then so do its points,
  // whose rounding is below 2^-10 (lambdas sum to 1 within 2^-21)
  const int axis = lane % 3, extent = axis == 0 ? P.nx : (axis == 1 ? P.ny : P.nz);
  const bool in = lane >= 24 || (fix >= -960 && fix <= 1024 * extent - 64);
  const bool inner = ok && __ballot(in) == ~0ull;
  int count[2];
  int64_t det[2];
#pragma unroll
  for (int d = 0; d < 2; d++) {
    int v[4][3];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int k = 0; k < 3; k++) v[i][k] = __builtin_amdgcn_readlane(fix, 12 * d + 3 * i + k);
    det[d] = det6(v);
    count[d] = ok ? sample_count(det[d], count_scale) : 0;
  }
  if constexpr (kStaged) {
    if (inner && lane < 24) {
      atomicMin(&L.lo[lane / 12][axis], (fix - 1) >> 10);
      atomicMax(&L.hi[lane / 12][axis], (fix + 1) >> 10);
    }
    if (inner && lane == 0) atomicAdd(&L.points, count[0] + count[1]);
  }

  // magnitude (Sec. 4.1.1): lane e < 10 takes edge e (6 edges, then the 4
  // spokes from the centroid), squared lengths exact in FP64
  double term = 0.0;
  {
    const int e = lane < 10 ? lane : 0;
    const int va = e < 3 ? 0 : (e < 5 ? 1 : (e < 6 ? 2 : e - 6));
    const int vb = e < 3 ? e + 1 : (e < 5 ? e - 1 : 3);
    double ls = 0.0, lt = 0.0;
#pragma unroll
    for (int k = 0; k < 3; k++) {
      const int sa = __shfl(fix, 3 * va + k, 64), sb = __shfl(fix, 3 * vb + k, 64);
      const int ta = __shfl(fix, 12 + 3 * va + k, 64), tb = __shfl(fix, 12 + 3 * vb + k, 64);
      double ds, dt;
      if (e < 6) {
        ds = static_cast<double>(sa - sb);
        dt = static_cast<double>(ta - tb);
      } else {   // 4 v_a - (v_0 + v_1 + v_2 + v_3), exact
        const int ss = __builtin_amdgcn_readlane(fix, k) + __builtin_amdgcn_readlane(fix, 3 + k) +
                       __builtin_amdgcn_readlane(fix, 6 + k) + __builtin_amdgcn_readlane(fix, 9 + k);
        const int st = __builtin_amdgcn_readlane(fix, 12 + k) + __builtin_amdgcn_readlane(fix, 15 + k) +
                       __builtin_amdgcn_readlane(fix, 18 + k) + __builtin_amdgcn_readlane(fix, 21 + k);
        ds = 4.0 * sa - ss;
        dt = 4.0 * ta - st;
      }
      ls = fma(ds, ds, ls);
      lt = fma(dt, dt, lt);
    }
    if (lane < 10) {
      const double den = sqrt(ls) + sqrt(lt);
      const double d = den > 0.0 ? (ls - lt) / den * (e < 6 ? 1.0 / 1024.0 : 1.0 / 4096.0) : 0.0;
      term = d * d;
    }
  }
  const float mag = __int_as_float(__builtin_amdgcn_readfirstlane(
      __float_as_int(static_cast<float>(static_cast<double>(P.elasticity[tet]) * wave_sum_d(term)))));

  // stage the boxes, if they fit
  Box box[2];
  bool staged = false;
  int found0 = 0, found1 = 0;
  if constexpr (kStaged) {
    __syncthreads();
    if (L.points > 0) {
      long long all = 0;
#pragma unroll
      for (int m = 0; m < 2; m++) {
        const int sy = __builtin_amdgcn_readfirstlane(L.hi[m][0] - L.lo[m][0] + 2);
        const int ly = __builtin_amdgcn_readfirstlane(L.hi[m][1] - L.lo[m][1] + 2);
        const int lz = __builtin_amdgcn_readfirstlane(L.hi[m][2] - L.lo[m][2] + 2);
        const int x0 = __builtin_amdgcn_readfirstlane(L.lo[m][0]), y0 = __builtin_amdgcn_readfirstlane(L.lo[m][1]);
        const int z0 = __builtin_amdgcn_readfirstlane(L.lo[m][2]);
        box[m] = Box{static_cast<int>(all) - (z0 * ly + y0) * sy - x0, sy, sy * ly};
        all += static_cast<long long>(sy) * ly * lz;
      }
      staged = all <= kBoxVoxels;
    }
    if (staged) {
      // half the threads a box, a thread a column of it
      const int half = blockDim.x >> 1, m = threadIdx.x >= half ? 1 : 0;
      const int x0 = L.lo[m][0], y0 = L.lo[m][1], z0 = L.lo[m][2];
      const int sy = m ? box[1].sy : box[0].sy, sz = m ? box[1].sz : box[0].sz;
      const int nz = L.hi[m][2] - z0 + 2, origin = (m ? box[1].first : box[0].first) + (z0 * sz + y0 * sy + x0);
      const void* img = m ? P.img[1] : P.img[0];
      const uint16_t* cells = m ? cells1 : cells0;
      const float inv = 1.f / static_cast<float>(sy);
      float top = 0.f;
      unsigned bits = 0;
      for (int c = threadIdx.x - (m ? half : 0); c < sz; c += half) {
        // exact: the quotient's error, 2^-22 of it, is below half a divisor's share
        const int y = static_cast<int>((static_cast<float>(c) + 0.5f) * inv), x = c - y * sy;
        int i = (z0 + 1) * P.pxy + (y0 + 1 + y) * P.px + x0 + 1 + x, e = origin + c;
#pragma unroll 4
        for (int z = 0; z < nz; z++, i += P.pxy, e += sz) {
          const float v = ld<ST>(img, i);
          const unsigned b = cells[i] >> 8;
          L.v[e] = v;
          L.band[e] = static_cast<uint8_t>(b);
          top = fmaxf(top, v);
          bits |= b;
        }
      }
      const int seen = (top > 0.f ? 1 : 0) | (bits ? 256 : 0);
      if (seen) atomicOr(&L.found[m], seen);
    }
    __syncthreads();
    if (!ok || spare) return;
    found0 = __builtin_amdgcn_readfirstlane(L.found[0]);
    found1 = __builtin_amdgcn_readfirstlane(L.found[1]);
  }
  const bool any_fg = ((found0 | found1) & 1) != 0;

  // this lane's Sobol integers (the 6 low bits of the index)
  uint32_t xlane[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int b = 0; b < 6; b++)
#pragma unroll
    for (int j = 0; j < 4; j++) xlane[j] ^= kDirections.v[j][b] & (0u - ((static_cast<uint32_t>(lane) >> b) & 1u));
  const int ref = P.ref_sign[tet];

#pragma unroll 1
  for (int d = 0; d < 2; d++) {
    // the sampled tet and the other one (wave-uniform)
    int own[4][3], oth[4][3];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int k = 0; k < 3; k++) {
        own[i][k] = __builtin_amdgcn_readlane(fix, 12 * d + 3 * i + k);
        oth[i][k] = __builtin_amdgcn_readlane(fix, 12 * (1 - d) + 3 * i + k);
      }
    const int64_t D = d == 0 ? det[0] : det[1];
    const int N = d == 0 ? count[0] : count[1];
    const int sg = (D > 0) - (D < 0);
    const bool viol = sg == 0 || sg != ref;
    const int64_t absD = D < 0 ? -D : D;
    const float vol = viol ? static_cast<float>(static_cast<double>(absD) * (1.0 / 6442450944.0)) : 0.f;
    float h = 0.f, g = 0.f;
    if (N > 0) {
      // the four shift words from a hash of the seed, the direction and the
      // tet (wave-uniform: scalar), applied to the lane's integers; r_j =
      // v_j 2^-24 with v_j = 2 floor(u_j / 2^9) + 1 of the integer u_j
      uint64_t hsh = splitmix(seed + kGolden * static_cast<uint64_t>(d + 1));
#pragma unroll
      for (int i = 0; i < 12; i++)
        hsh = splitmix(hsh + kGolden + static_cast<uint64_t>(static_cast<uint32_t>(own[i / 3][i % 3])));
      const uint64_t w0 = splitmix(hsh + kGolden), w1 = splitmix(hsh + 2 * kGolden);
      const uint32_t shift[4] = {static_cast<uint32_t>(w0), static_cast<uint32_t>(w0 >> 32),
                                 static_cast<uint32_t>(w1), static_cast<uint32_t>(w1 >> 32)};
      uint32_t xl[4];
#pragma unroll
      for (int j = 0; j < 4; j++) xl[j] = ((xlane[j] ^ shift[j]) >> 8) | 1u;
      // FP32 base vertex and edge vectors of both tets, in voxels (exact)
      float bo[3], eo[3][3], bt[3], et[3][3];
#pragma unroll
      for (int a = 0; a < 3; a++) {
        bo[a] = static_cast<float>(own[0][a]) * 0x1p-10f;
        bt[a] = static_cast<float>(oth[0][a]) * 0x1p-10f;
#pragma unroll
        for (int i = 0; i < 3; i++) {
          eo[i][a] = static_cast<float>(own[i + 1][a] - own[0][a]) * 0x1p-10f;
          et[i][a] = static_cast<float>(oth[i + 1][a] - oth[0][a]) * 0x1p-10f;
        }
      }
      uint32_t xk[4] = {0u, 0u, 0u, 0u};   // Sobol integers of 64 k (wave-uniform)
      for (int base = 0; base < N; base += kWave) {
        uint32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) v[j] = xl[j] ^ xk[j];
        const int c = __builtin_ctz((static_cast<uint32_t>(base) >> 6) + 1u);
#pragma unroll
        for (int j = 0; j < 4; j++) xk[j] ^= kSteps.v[c][j];
        if (base + lane >= N) break;
        float l[3], p[3], q[3];
        lambdas(v, l, [](float x) { return __builtin_amdgcn_rcpf(x); });
#pragma unroll
        for (int a = 0; a < 3; a++) {
          p[a] = __builtin_fmaf(l[2], eo[2][a], __builtin_fmaf(l[1], eo[1][a], __builtin_fmaf(l[0], eo[0][a], bo[a])));
          q[a] = __builtin_fmaf(l[2], et[2][a], __builtin_fmaf(l[1], et[1][a], __builtin_fmaf(l[0], et[0][a], bt[a])));
        }
        const ProblemView V = view();
        const void* img_own = d == 0 ? V.img[0] : V.img[1];
        const void* img_oth = d == 0 ? V.img[1] : V.img[0];
        const uint16_t* cells_own = d == 0 ? cells0 : cells1;
        const uint16_t* cells_oth = d == 0 ? cells1 : cells0;
        const float* map_own = d == 0 ? V.dmap[0] : V.dmap[1];
        const float* map_oth = d == 0 ? V.dmap[1] : V.dmap[0];
        const float* set_w = V.set_w + d * kMaxSets;
        if constexpr (kStaged)
          if (inner && staged) {
            staged_sample(V, L, d == 0 ? box[0] : box[1], d == 0 ? box[1] : box[0], any_fg,
                          ((d == 0 ? found0 : found1) >> 8) != 0, map_own, map_oth, set_w, p, q, h, g);
            continue;
          }
        if (inner)
          inner_sample<ST>(V, img_own, img_oth, cells_own, cells_oth, map_own, map_oth, set_w, p, q, h, g);
        else
          outer_sample<ST>(V, img_own, img_oth, cells_own, cells_oth, map_own, map_oth, set_w, p, q, h, g);
      }
      h = wave_sum_63(h);
      g = wave_sum_63(g);
    }
    if (lane_id() == 63)
      out[d] = Record{h, g, static_cast<uint32_t>(N), d == 0 ? mag : 0.f, vol, viol ? 1u : 0u};
  }
}

morea_status fail(morea_status s, const char* msg) {
  set_error(msg);
  return s;
}

morea_status device_fail(hipError_t e, const char* what) {
  char buf[256];
  snprintf(buf, sizeof(buf), "%s: %s", what, hipGetErrorString(e));
  set_error(buf);
  return MOREA_EDEVICE;
}

// Code per cell of the padded volume (lower corner at padded element i): bit
// 0 when a corner of the image holds a value > 0, bit 1 when all eight do,
// bits 8..15 the OR of the corners' band bytes.
template <int ST>
__global__ void k_cells(ProblemView P, const void* img, const uint8_t* band, uint16_t* cells) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= static_cast<int>(P.pvox)) return;
  const int x = i % P.px, y = (i / P.px) % (P.ny + 2), z = i / P.pxy;
  unsigned v = 0;
  if (x + 1 < P.px && y + 1 < P.ny + 2 && z + 1 < P.nz + 2) {
    const int j = i + P.pxy;
    const int idx[8] = {i, i + 1, i + P.px, i + P.px + 1, j, j + 1, j + P.px, j + P.px + 1};
    bool any = false, all = true;
    unsigned bits = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const bool pos = ld<ST>(img, idx[k]) > 0.f;
      any = any || pos;
      all = all && pos;
      bits |= band[idx[k]];
    }
    v = (any ? 1u : 0u) | (all ? 2u : 0u) | bits << 8;
  }
  cells[i] = static_cast<uint16_t>(v);
}

template <int ST>
hipError_t launch(const morea_problem* p, const float* pts, int pop, float rate, uint64_t seed, hipStream_t s) {
  const ProblemView& P = p->view;
  const double count_scale = static_cast<double>(rate) / 6442450944.0;   // rate / (6 * 2^30)
  const double inv_pop = 1.0 / pop;
  // candidates spread evenly over the blocks of a tet
  const int groups = (pop + kBlockWaves - 1) / kBlockWaves, per = (pop + groups - 1) / groups;
  const int turns = (per + 3) / 4 * 4;   // waves that would fill the same turns of four SIMDs
  const size_t blocks = static_cast<size_t>(P.n_tets) * groups;
  // spare waves must not take the launch to 2^32 threads
  const bool staged = per >= kStageWaves && p->tet_volume * rate * per * per / turns >= kStageSamples &&
                      2.0 * p->tet_box <= kBoxVoxels && blocks * 64 * per <= UINT32_MAX;
  if (staged) {
    const dim3 grid(static_cast<unsigned>(blocks));
    hipLaunchKernelGGL((k_eval_sobol<ST, true>), grid, dim3(64 * per), 0, s, P, pts, pop, per, groups, inv_pop,
                       count_scale, seed, p->cells[0], p->cells[1], p->work_records);
  } else {
    const dim3 grid(static_cast<unsigned>((static_cast<size_t>(P.n_tets) * pop + 3) / 4));
    hipLaunchKernelGGL((k_eval_sobol<ST, false>), grid, dim3(256), 0, s, P, pts, pop, 4, 0, inv_pop, count_scale, seed,
                       p->cells[0], p->cells[1], p->work_records);
  }
  return hipGetLastError();
}

}  // namespace sobol

hipError_t launch_cells(const ProblemView& P, int storage, const void* img, const uint8_t* band, uint16_t* cells,
                        hipStream_t s) {
  const dim3 grid((P.pvox + 255) / 256);
  switch (storage) {
    case kF32: hipLaunchKernelGGL(sobol::k_cells<kF32>, grid, dim3(256), 0, s, P, img, band, cells); break;
    case kBF16: hipLaunchKernelGGL(sobol::k_cells<kBF16>, grid, dim3(256), 0, s, P, img, band, cells); break;
    default: hipLaunchKernelGGL(sobol::k_cells<kF16>, grid, dim3(256), 0, s, P, img, band, cells); break;
  }
  return hipGetLastError();
}

}  // namespace morea

using namespace morea;

extern "C" morea_status morea_eval_sobol(morea_problem* p, const float* pts, int32_t pop, float rate,
                                         uint64_t seed, float* obj, uint8_t* flags, float* severity,
                                         uint32_t* counts, void* stream) {
  if (!p) return sobol::fail(MOREA_EINVAL, "problem is NULL");
  if (pop < 0) return sobol::fail(MOREA_EINVAL, "pop < 0");
  if (pop > p->max_population) return sobol::fail(MOREA_ERANGE, "pop above max_population");
  if (!(rate > 0.f) || !(rate < INFINITY)) return sobol::fail(MOREA_EINVAL, "rate must be finite and > 0");
  if (pop == 0) return MOREA_OK;
  if (!pts || !obj || !flags || !severity || !counts) return sobol::fail(MOREA_EINVAL, "NULL argument");
  {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return sobol::device_fail(e, "earlier device work failed");
  }
  const ProblemView& P = p->view;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t n_items = static_cast<size_t>(pop) * P.n_tets;
  if (n_items > 0) {
    hipError_t e;
    switch (p->storage) {
      case kF32: e = sobol::launch<kF32>(p, pts, pop, rate, seed, s); break;
      case kBF16: e = sobol::launch<kBF16>(p, pts, pop, rate, seed, s); break;
      default: e = sobol::launch<kF16>(p, pts, pop, rate, seed, s); break;
    }
    if (e != hipSuccess) return sobol::device_fail(e, "Sobol evaluation");
  }
  hipError_t e = launch_finalize(P, pts, pop, p->work_records, obj, flags, severity, counts, nullptr, s);
  if (e != hipSuccess) return sobol::device_fail(e, "Sobol evaluation");
  return MOREA_OK;
}
