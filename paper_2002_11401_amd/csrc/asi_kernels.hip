// HIP kernels (gfx950) of the spin-ice relaxation path.
//
// Model: flatspin dipole model (Jensen et al.), Sec. II.  All field and
// margin arithmetic is FP64 and this file is compiled without FMA
// contraction, so every kernel that evaluates the same expression on the
// same inputs produces the same bits -- plain, batched and served runs agree
// bitwise by construction.
//
//   k_nb_count / k_nb_fill  neighbour tables of Sec. II.C and the projected
//                           couplings of Eq. 3 (once per instance)
//   k_field                 full-field pass: Eq. 3 gathered in ascending
//                           neighbour order, plus applied field (Sec. II.D)
//                           and thermal field (Sec. II.E), Eq. 2, projected;
//                           switching key of Eq. 5 / Eq. 6; per-64-row maxima
//   k_relax                 one workgroup per instance: argmax over the
//                           flippable keys (ties: lowest index), flip, update
//                           the neighbours' fields incrementally, repeat
//                           until none can flip (Sec. II.H); several
//                           paths with the same flips: one at a time on a
//                           max tree or on approximated keys in LDS, and
//                           exact-order batches from a sorted window or from
//                           tile maxima
//   k_fused                 one workgroup per instance runs whole steps
//                           (field phase + relax) through its own protocol
#include <algorithm>
#include <climits>
#include <mutex>
#include <type_traits>
#include <utility>

#define ASI_KERNELS_UNIT 1
#include "asi_internal.h"

namespace asi {
namespace {

// ------------------------------------------------------------ Philox4x32-10
// Counter-based generator of Salmon et al. (SC'11): ten rounds; each round
// multiplies counter words 0 and 2 by the two round multipliers and xors the
// high halves into words 1 and 3 with the key; the key advances by the two
// Weyl increments between rounds.
struct U4 {
  uint32_t x, y, z, w;
};

__device__ inline U4 philox4x32_10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint32_t lo0 = 0xD2511F53u * c.x;
    const uint32_t hi0 = __umulhi(0xD2511F53u, c.x);
    const uint32_t lo1 = 0xCD9E8D57u * c.z;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c.z);
    c = U4{hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0};
  }
  return c;
}

// Thermal field of Sec. II.E: two independent N(0,1) draws for magnet i at
// step t (counter (i, t, 0, 0)), by Box-Muller on 53-bit uniforms
// u1 in (0, 1] and u2 in [0, 1).
__device__ inline void thermal_normals(uint64_t seed, uint32_t i, uint32_t t, double& z0,
                                       double& z1) {
  const U4 o = philox4x32_10(U4{i, t, 0u, 0u}, (uint32_t)seed, (uint32_t)(seed >> 32));
  const uint64_t a = ((((uint64_t)o.x) << 32) | o.y) >> 11;
  const uint64_t b = ((((uint64_t)o.z) << 32) | o.w) >> 11;
  const double u1 = (double)(a + 1) * 0x1p-53;
  const double u2 = (double)b * 0x1p-53;
  const double rad = sqrt(-2.0 * log(u1));
  const double ang = 6.283185307179586 * u2;
  double sn, cs;
  sincos(ang, &sn, &cs);
  z0 = rad * cs;
  z1 = rad * sn;
}

// Upper bound of x^e (x >= 0, e > 0, x within 2^-22) from the
// single-precision hardware log2 and exp2: log2 x is raised by 2^-20, past its
// error (x's own, its 24 bits and a few units of the hardware's: below 6e-7 for
// |log2 x| < 4), the exponent by log2(1.001), far past that of a larger
// |log2 x| (where x^e matters, e |log2 x| < 20, it is below 3e-6), of the product
// and of exp2; x below 2^-100 is raised to 2^-100, which only raises x^e.
__device__ inline float pow_bound(double x, double e) {
  const float xf = (float)fmax(x, 0x1p-100), ef = (float)e;
  return __builtin_amdgcn_exp2f(
      __builtin_fmaf(ef, __builtin_amdgcn_logf(xf) + 0x1p-20f, 0.00144197f));
}

// Switching key: the left-hand side of Eq. 5 when magnet i may flip, i.e.
// the field opposes the moment (Eq. 6, s_i h_par < 0) and Eq. 5 exceeds 1;
// otherwise 0.  Exponents ep = 2/gamma, eq = 2/beta.  When the bound puts
// the left-hand side below 1 the FP64 powers (which could only give a
// value <= 1: the bound exceeds their sum) are skipped: the key is the
// same, bit for bit.
// In two stages: key_needs_powers settles the key at 0, or gives the
// normalised field components a and q whose powers decide it.
__device__ inline bool key_needs_powers(int s, double hp, double hq, double hk, double b,
                                        double c, double ep, double eq, double& a, double& q) {
  // h_k > 0 always (checked at creation); testing it with the direction
  // makes h_k needed on every path, so its load is issued with the field's
  // and the spin's instead of after them
  const bool against = (hk > 0.0) && ((s > 0) ? (hp < 0.0) : (hp > 0.0));
  if (!against) return false;
  a = fabs(hp) / (b * hk);
  q = fabs(hq) / (c * hk);
  return !(pow_bound(a, ep) + pow_bound(q, eq) < 1.0f);
}
__device__ inline double key_from_powers(double a, double q, double ep, double eq) {
  const double L = pow(a, ep) + pow(q, eq);
  return (L > 1.0) ? L : 0.0;
}
__device__ inline double switching_key(int s, double hp, double hq, double hk, double b,
                                       double c, double ep, double eq) {
  double a = 0.0, q = 0.0;
  if (!key_needs_powers(s, hp, hq, hk, b, c, ep, eq, a, q)) return 0.0;
  return key_from_powers(a, q, ep, eq);
}

// The exact key for the rare lanes of a relax that need it: out of line, so
// that the FP64 powers' registers and constants stay out of the relax loop.
__device__ __attribute__((noinline)) double switching_key_far(const InstDev* __restrict__ I,
                                                              bool neg, double hp, double hq,
                                                              double hk) {
  return switching_key(neg ? -1 : 1, hp, hq, hk, I->b, I->c, I->e_par, I->e_perp);
}

// 32-bit code of a key for the relax that holds its keys in LDS: an
// approximation k of Eq. 5's left-hand side in the upper 24 bits (the float's
// bits above those of just below 1, less the lowest three: ordered like k, up
// to kCodeTop), two flags, and in the lowest 6 bits the magnet's place in its
// thread's tile; 0 when the magnet certainly cannot flip.
// The relative distance of k from the FP64 key (from the left-hand side, where
// that is at most 1) is bounded so:
//   - the normalised components are formed in FP64 and rounded once, 2^-24;
//   - v_log_f32 and v_exp_f32 are within an ulp.  With exponents e in
//     [1/4, 4], x the normalised component, the exponent e log2 x of the term
//     that matters is in error by at most |e log2 x| 2^-22 + 4 * 2.45 * 2^-24;
//     the term, and the sum, by that times ln 2, and 2^-23: 1.3e-6 (below
//     kCodeRel) for k < 16, where |e log2 x| < 4, 3.2e-6 for k < 2^16 (a small
//     term errs less against the sum);
//   - a component that underflows loses a term below (2^-126)^(1/4).
// Measured over 3e9 random fields and parameters: 7.0e-7 for k < 16, 2.1e-6
// for k < 2^16.  Instances with parameters outside these ranges are relaxed on
// other paths; a lane's k or h_k outside them (k_inverse_hk marks the latter by
// NaN) gives kCodeUnknown, which the relax replaces by the exact key's code.
constexpr float kCodeRel = 0x1p-19f;
constexpr uint32_t kCodeBase = 0x3f800000u - 256u;
constexpr float kCodeTop = 65000.0f;  // keys from here on share a code
constexpr uint32_t kCodePlace = 63u;
constexpr uint32_t kCodeDown = 64u;    // flag: the spin is -1
constexpr uint32_t kCodeExact = 128u;  // flag: the key array holds the FP64 key
__host__ __device__ constexpr uint32_t code_bits(uint32_t float_bits) {
  return ((float_bits - kCodeBase) >> 3) << 8;
}
// Codes below code_floor(v) belong to keys certainly below v's: v less eleven
// units (of 8 units in the last place of a float), and up to eight more with
// v.  Two approximations in the order of their keys, or a ratio of 1 - 2 * the
// bound above apart at most: 2 * 1.3e-6 * 2^24 = 44 units in the last place
// for k < 16 (and two code roundings, 16), 108 for k < 2^16.
__device__ inline uint32_t code_floor(uint32_t v) { return (v & ~255u) - (11u << 8) - (v >> 21); }
// From here the key is certainly above 1 (kCodeRel is 16 units in the last
// place above 1).
constexpr uint32_t kCodeSure = code_bits(0x3f800000u + 40u);
constexpr uint32_t kCodeUnknown = code_bits(0x477de800u) + 256u;  // above kCodeTop's

struct KeyPar {
  double bc;     // b / c (0 for c = infinity: no hard-axis term)
  float ep, eq;
};

__device__ inline KeyPar key_par(const InstDev* __restrict__ I) {
  return KeyPar{I->b / I->c, (float)I->e_par, (float)I->e_perp};
}

// Code of an FP64 key, without its place.
__device__ inline uint32_t code_of_key(double key, bool neg) {
  if (!(key > 0.0)) return 0u;
  const float k = (float)fmin(key, (double)kCodeTop);
  return code_bits(__float_as_uint(k)) | (neg ? kCodeDown : 0u);
}

// Code of the key from the field, without its place; g = 1 / (b h_k).
__device__ __forceinline__ uint32_t key_code(bool neg, double hp, double hq, double g,
                                             const KeyPar& P) {
  const float a = (float)(fabs(hp) * g);
  const float q = (float)(fabs(hq) * g * P.bc);
  const float k = __builtin_amdgcn_exp2f(P.ep * __builtin_amdgcn_logf(a)) +
                  __builtin_amdgcn_exp2f(P.eq * __builtin_amdgcn_logf(q));
  uint32_t v = k < kCodeTop ? code_bits(__float_as_uint(k)) : kCodeUnknown;  // NaN: unknown
  v |= neg ? kCodeDown : 0u;
  const bool can = ((neg ? hp : -hp) > 0.0) & !(k <= 1.0f - kCodeRel);
  return can ? v : 0u;
}

// Eq. 3 for a unit source moment mhat_s at (sx, sy) seen at (fx, fy),
// projected on the observer's easy axis (A) and hard axis (B);
// mhatperp = (-my, mx).  A is symmetric in (f, s) bit for bit: swapping
// the two negates r, which negates both dot products of the 3(.)(.) term.
__device__ inline void coupling(double fx, double fy, double fmx, double fmy, double sx,
                                double sy, double smx, double smy, double alpha, double& A,
                                double& B) {
  const double rx = fx - sx;
  const double ry = fy - sy;
  const double r2 = rx * rx + ry * ry;
  const double r = sqrt(r2);
  const double inv3 = 1.0 / (r2 * r);
  const double inv5 = inv3 / r2;
  const double af = fmx * rx + fmy * ry;
  const double as = smx * rx + smy * ry;
  const double pf = fmx * ry - fmy * rx;
  const double mm = fmx * smx + fmy * smy;
  const double pm = fmx * smy - fmy * smx;
  A = alpha * (3.0 * (af * as) * inv5 - mm * inv3);
  B = alpha * (3.0 * (pf * as) * inv5 - pm * inv3);
}

// Cross-lane moves of a double within rows of 16 lanes by DPP.
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(x >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double((long long)(unsigned)lo | ((long long)hi << 32));
}

__device__ inline double readlane_f64(double v, int lane) {
  const long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)x, lane);
  const int hi = __builtin_amdgcn_readlane((int)(x >> 32), lane);
  return __longlong_as_double((long long)(unsigned)lo | ((long long)hi << 32));
}

// Maximum over the 64 lanes, returned to every lane: butterfly within each
// row of 16 (quad swaps, half-row and row mirrors), then the four row
// results through scalar reads.
__device__ inline double wave_max_f64(double v) {
  v = fmax(v, dpp_f64<0xB1>(v));   // quad_perm [1,0,3,2]
  v = fmax(v, dpp_f64<0x4E>(v));   // quad_perm [2,3,0,1]
  v = fmax(v, dpp_f64<0x141>(v));  // row_half_mirror
  v = fmax(v, dpp_f64<0x140>(v));  // row_mirror
  const double r0 = readlane_f64(v, 0), r1 = readlane_f64(v, 16);
  const double r2 = readlane_f64(v, 32), r3 = readlane_f64(v, 48);
  return fmax(fmax(r0, r1), fmax(r2, r3));
}

// max(v, v moved by DPP): lanes without a source take 0.
template <int CTRL, int ROWS = 0xF>
__device__ inline uint32_t max_dpp_u32(uint32_t v) {
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false));
}

// Maximum of an unsigned value over each row of 16 lanes, in every lane.
__device__ inline uint32_t row_max_u32(uint32_t v) {
  v = max_dpp_u32<0xB1>(v);     // quad_perm [1,0,3,2]
  v = max_dpp_u32<0x4E>(v);     // quad_perm [2,3,0,1]
  v = max_dpp_u32<0x141>(v);    // row_half_mirror
  return max_dpp_u32<0x140>(v); // row_mirror
}

// Maximum over the 64 lanes, uniform.
__device__ inline uint32_t wave_max_u32(uint32_t v) {
  v = row_max_u32(v);
  v = max_dpp_u32<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v = max_dpp_u32<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Wave-wide argmax of (key, payload) where lane order is index order:
// largest key, and among equal keys the lowest lane.  All 64 lanes call;
// the result is uniform.
__device__ inline void wave_argmax(double& key, uint32_t& payload) {
  const double m = wave_max_f64(key);
  const unsigned long long bal = __ballot(key == m);
  const int src = __ffsll((unsigned long long)bal) - 1;
  payload = (uint32_t)__builtin_amdgcn_readlane((int)payload, src);
  key = m;
}

__device__ inline int64_t slot_of(int64_t i, int32_t D, int32_t k) {
  return ((i >> 6) * (int64_t)D + k) * kSlice + (i & (kSlice - 1));
}

// ------------------------------------------------------------ neighbours
// Coercive fields of Sec. II.G drawn on the device (hk == NULL): the first
// Box-Muller normal of Philox4x32-10 at counter (i, 0, 1, 0), uniforms
// formed as for the thermal field.
__global__ void k_draw_hk(double* __restrict__ hk, int64_t n, double mean, double k,
                          uint64_t seed) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const U4 o = philox4x32_10(U4{(uint32_t)i, 0u, 1u, 0u}, (uint32_t)seed, (uint32_t)(seed >> 32));
  const uint64_t a = ((((uint64_t)o.x) << 32) | o.y) >> 11;
  const uint64_t b = ((((uint64_t)o.z) << 32) | o.w) >> 11;
  const double u1 = (double)(a + 1) * 0x1p-53;
  const double u2 = (double)b * 0x1p-53;
  const double z0 = sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
  const double sd = k * mean;
  const double h = mean + sd * z0;
  const double lo = 1e-12 * mean;
  hk[i] = h < lo ? lo : h;
}

// 1 / (b h_k) for key_code; NaN where h_k or the result is outside the range
// in which its approximation holds.
__global__ void k_inverse_hk(const double* __restrict__ hk, int64_t n, double b,
                             double* __restrict__ g) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double v = hk[i];
  g[i] = v > 0x1p-60 && v < 0x1p60 ? 1.0 / (b * v) : __longlong_as_double(0x7ff8000000000000ll);
}

// Cells of side >= the cutoff, magnets sorted by cell (ascending index
// within a cell); a magnet's neighbours lie in its 3 x 3 cell block.
__global__ void k_nb_count(const double* __restrict__ x, const double* __restrict__ y,
                           const int32_t* __restrict__ cellx, const int32_t* __restrict__ celly,
                           const int32_t* __restrict__ cstart, const int32_t* __restrict__ cmem,
                           int64_t n, int64_t gx, int64_t gy, double cut2,
                           int32_t* __restrict__ len, int32_t* __restrict__ dup) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double xi = x[i], yi = y[i];
  const int64_t cx = cellx[i], cy = celly[i];
  int32_t cnt = 0;
  for (int64_t yy = cy - 1; yy <= cy + 1; ++yy) {
    if (yy < 0 || yy >= gy) continue;
    for (int64_t xx = cx - 1; xx <= cx + 1; ++xx) {
      if (xx < 0 || xx >= gx) continue;
      const int64_t c = yy * gx + xx;
      for (int32_t p = cstart[c]; p < cstart[c + 1]; ++p) {
        const int32_t j = cmem[p];
        if (j == i) continue;
        const double dx = xi - x[j];
        const double dy = yi - y[j];
        const double r2 = dx * dx + dy * dy;
        if (r2 <= cut2) {
          ++cnt;
          if (r2 == 0.0) *dup = 1;
        }
      }
    }
  }
  len[i] = cnt;
}

// Fills row i in ascending neighbour order by a 9-way merge of the
// (ascending) member lists of its 3 x 3 cell block, and computes the
// projected couplings of each pair; writes the sliced and the row-major
// tables.
__global__ void k_nb_fill(const double* __restrict__ x, const double* __restrict__ y,
                          const double* __restrict__ mx, const double* __restrict__ my,
                          const int32_t* __restrict__ cellx, const int32_t* __restrict__ celly,
                          const int32_t* __restrict__ cstart, const int32_t* __restrict__ cmem,
                          int64_t n, int64_t gx, int64_t gy, double cut2, double alpha,
                          int32_t D, int32_t* __restrict__ col, double* __restrict__ A,
                          double* __restrict__ B, int32_t* __restrict__ rcol,
                          double2* __restrict__ rAB) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double xi = x[i], yi = y[i], mxi = mx[i], myi = my[i];
  const int64_t cx = cellx[i], cy = celly[i];
  int32_t pos[9], end[9], head[9];
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    const int64_t xx = cx + (r % 3) - 1;
    const int64_t yy = cy + (r / 3) - 1;
    const bool ok = xx >= 0 && xx < gx && yy >= 0 && yy < gy;
    const int64_t c = yy * gx + xx;
    pos[r] = ok ? cstart[c] : 0;
    end[r] = ok ? cstart[c + 1] : 0;
    head[r] = pos[r] < end[r] ? cmem[pos[r]] : INT_MAX;
  }
  int32_t k = 0;
  while (true) {
    int32_t best = INT_MAX;
    int br = -1;
#pragma unroll
    for (int r = 0; r < 9; ++r)
      if (head[r] < best) {
        best = head[r];
        br = r;
      }
    if (br < 0) break;
#pragma unroll
    for (int r = 0; r < 9; ++r)
      if (r == br) {
        ++pos[r];
        head[r] = pos[r] < end[r] ? cmem[pos[r]] : INT_MAX;
      }
    const int32_t j = best;
    if (j == i) continue;
    const double xj = x[j], yj = y[j];
    const double dx = xi - xj;
    const double dy = yi - yj;
    if (dx * dx + dy * dy > cut2) continue;
    if (k >= D) break;  // cannot happen: D is the maximum count
    double a, b, ar, bt;
    const double mxj = mx[j], myj = my[j];
    coupling(xi, yi, mxi, myi, xj, yj, mxj, myj, alpha, a, b);
    coupling(xj, yj, mxj, myj, xi, yi, mxi, myi, alpha, ar, bt);
    const int64_t sl = slot_of(i, D, k);
    col[sl] = j;
    A[sl] = a;
    B[sl] = b;
    const int64_t rs = i * D + k;
    rcol[rs] = j;
    rAB[rs] = make_double2(a, bt);
    ++k;
  }
  for (; k < D; ++k) {
    const int64_t sl = slot_of(i, D, k);
    col[sl] = -1;
    A[sl] = 0.0;
    B[sl] = 0.0;
    const int64_t rs = i * D + k;
    rcol[rs] = -1;
    rAB[rs] = make_double2(0.0, 0.0);
  }
}

// ------------------------------------------------------------ field phase
// Field of row i at step t (Eq. 2): the dipolar sum of Eq. 3 -- gathered over
// the neighbours in ascending order with one accumulator per axis, left to
// right, or carried from earlier steps -- plus H[t], any local external
// field and the thermal draw, projected on the easy and hard axis; then the
// switching key.  Writes the row's total field and key and returns (key,
// index | sign bit).  Every field pass (grid-wide or inside a fused
// workgroup) calls this one function, so they agree bit for bit.
__device__ __forceinline__ double field_finish(const InstDev* __restrict__ I, int64_t i, int64_t t,
                                               double p, double pq, uint32_t& payload);

// Slots per chunk of the canonical dipolar sum (and of the high-degree
// pass), and entries per thread per chunk in the high-degree pass.
constexpr int kHdChunk = 64;
constexpr int kHdPer = 8;

__device__ __forceinline__ double field_row(const InstDev* __restrict__ I, int64_t i, int64_t t,
                                   uint32_t& payload) {
  const int8_t* __restrict__ s = I->s;
  const int32_t mode = I->field_mode;
  double p, pq;
  if (mode == kFieldFull || I->dirty[i]) {
    const int32_t L = I->len[i];
    const int64_t base = slot_of(i, I->D, 0);
    const int32_t* __restrict__ col = I->col + base;
    const double* __restrict__ A = I->A + base;
    const double* __restrict__ B = I->B + base;
    // Groups of 8 neighbours; the columns of the next group are fetched
    // with the couplings and spins of the current one, so each group costs
    // one round trip.  The canonical order of the sum: each chunk of 64
    // slots is added in ascending order from zero, and the chunk sums in
    // ascending order (up to 64 neighbours, the plain left-to-right sum);
    // every pass uses it, so all agree bit for bit.  The tables are streamed
    // once per pass (non-temporal loads), which leaves the L2 to the
    // gathered spins.
    // (A chunk sum that ends on a 64-slot boundary is added there, the last
    // one after the loop; a zero added after a full last chunk is exact.)
    p = 0.0;
    pq = 0.0;
    double cp = 0.0, cq = 0.0;
    int32_t jc[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) jc[u] = (u < L) ? __builtin_nontemporal_load(&col[u * kSlice]) : 0;
    for (int32_t k = 0; k < L; k += 8) {
      double a[8], b[8];
      int sg[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool ok = k + u < L;
        a[u] = ok ? __builtin_nontemporal_load(&A[(k + u) * kSlice]) : 0.0;
        b[u] = ok ? __builtin_nontemporal_load(&B[(k + u) * kSlice]) : 0.0;
        sg[u] = ok ? s[jc[u]] : 0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) jc[u] = (k + 8 + u < L) ? __builtin_nontemporal_load(&col[(k + 8 + u) * kSlice]) : 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (k + u < L) {
          cp += (sg[u] > 0) ? a[u] : -a[u];
          cq += (sg[u] > 0) ? b[u] : -b[u];
        }
      }
      if (((k + 8) & (kHdChunk - 1)) == 0) {
        p += cp;
        pq += cq;
        cp = 0.0;
        cq = 0.0;
      }
    }
    p += cp;
    pq += cq;
    if (mode != kFieldFull) {
      I->hd[i] = make_double2(p, pq);
      I->dirty[i] = 0;
    }
  } else {
    // carried, or no neighbour flipped since the last gather
    const double2 c = I->hd[i];
    p = c.x;
    pq = c.y;
  }
  return field_finish(I, i, t, p, pq, payload);
}

// Eq. 2 for row i from its dipolar sums (p, pq): plus H[t], the magnet's
// local external field (if any) and the thermal draw, projected; writes the total field and the key, returns the key.
__device__ __forceinline__ double field_finish(const InstDev* __restrict__ I, int64_t i, int64_t t,
                                               double p, double pq, uint32_t& payload) {
  const int8_t* __restrict__ s = I->s;
  const double mxi = I->mx[i], myi = I->my[i];
  double hp = p, hq = pq;
  if (t >= 0) {
    const double Hx = I->H[2 * t], Hy = I->H[2 * t + 1];
    hp = hp + (Hx * mxi + Hy * myi);
    hq = hq + (Hy * mxi - Hx * myi);
    if (I->hloc) {
      // the magnet's own external field (Sec. II.D), static or of step t
      const double2 l = I->hloc[(I->hloc_k > 1 ? t * I->n : 0) + i];
      hp = hp + (l.x * mxi + l.y * myi);
      hq = hq + (l.y * mxi - l.x * myi);
    }
    if (I->wave_ph) {
      // a travelling wave (Sec. II.D), evaluated here instead of stored per step
      const double a = I->wave_amp * sin(I->wave_ph[i] - I->wave_w * (double)t);
      const double lx = a * I->wave_ex, ly = a * I->wave_ey;
      hp = hp + (lx * mxi + ly * myi);
      hq = hq + (ly * mxi - lx * myi);
    }
    const double sg = I->sigma_t ? I->sigma_t[t] : I->sigma;
    if (sg > 0.0) {
      double z0, z1;
      thermal_normals(I->seed, (uint32_t)i, (uint32_t)t, z0, z1);
      const double tx = sg * z0, ty = sg * z1;
      hp = hp + (tx * mxi + ty * myi);
      hq = hq + (ty * mxi - tx * myi);
    }
  }
  I->h[i] = make_double2(hp, hq);
  const int si = s[i];
  const double key = switching_key(si, hp, hq, I->hk[i], I->b, I->c, I->e_par, I->e_perp);
  I->key[i] = key;
  payload = (uint32_t)i | (si < 0 ? 0x80000000u : 0u);
  return key;
}

// Key of row i for an instance whose relax paused mid-step: the relax keeps
// every field exact, so the key is that of the stored field (bit for bit the
// key an uninterrupted relax would hold).
__device__ __forceinline__ double stored_key(const InstDev* __restrict__ I, int64_t i,
                                             uint32_t& payload) {
  const int si = I->s[i];
  const double2 h = I->h[i];
  const double key = switching_key(si, h.x, h.y, I->hk[i], I->b, I->c, I->e_par, I->e_perp);
  I->key[i] = key;
  payload = (uint32_t)i | (si < 0 ? 0x80000000u : 0u);
  return key;
}

// Field phase for the 64 rows starting at row0 (a multiple of 64), by one
// wavefront: rows (or, resuming a paused relax, the keys of their stored fields), then
// their maximum key into the per-64-row table.  Returns the lane's (key,
// payload) for the candidate pool.
__device__ __forceinline__ double field_rows64(const InstDev* __restrict__ I, int64_t row0,
                                               int64_t t, uint32_t& payload,
                                               bool resume = false) {
  const int lane = threadIdx.x & 63;
  const int64_t i = row0 + lane;
  double key = 0.0;
  payload = 0;
  if (i < I->n) key = resume ? stored_key(I, i, payload) : field_row(I, i, t, payload);
  double mk = key;
  uint32_t mp = payload;
  wave_argmax(mk, mp);
  if (lane == 0) {
    I->t1key[row0 >> 6] = mk;
    I->t1idx[row0 >> 6] = mp;
  }
  return key;
}

// Append a flippable lane's entry at pool position base + its rank among
// the flippable lanes of the wavefront.
__device__ __forceinline__ void pool_put(const InstDev* __restrict__ I, double key,
                                         uint32_t payload, unsigned long long bal, int64_t base) {
  const int lane = threadIdx.x & 63;
  if (key > 0.0) {
    const int64_t q = base + __popcll(bal & ((1ull << lane) - 1ull));
    // A pass appends each row at most once to a pool emptied before it, so
    // q < n < ccap; past the end the entry is dropped and the relax, which
    // finds the count above ccap, fails the step (kPoolOverflow).
    if (q >= I->ccap) return;
    const uint32_t i = payload & 0x7fffffffu;
    I->cpay[0][q] = payload;
    I->ckey[0][q] = key;
    I->cver[0][q] = I->ver[i];
  }
}

// Field phase by one wavefront, appending its flippable rows to the pool
// with one atomic per wavefront.
__device__ __forceinline__ void field_rows64_pool(const InstDev* __restrict__ I, int64_t row0,
                                                  int64_t t, bool resume = false) {
  uint32_t payload;
  const double key = field_rows64(I, row0, t, payload, resume);
  const unsigned long long bal = __ballot(key > 0.0);
  if (bal) {
    int base = 0;
    if ((threadIdx.x & 63) == 0) base = atomicAdd(I->ccount, __popcll(bal));
    base = __builtin_amdgcn_readfirstlane(base);
    pool_put(I, key, payload, bal, base);
  }
}

// Grid-wide field pass: one lane per magnet, any number of instances; the
// block's flippable rows reach the pool with one atomic per block.  A paused
// instance (see RunDev) gets its relax structures rebuilt instead.
__global__ __launch_bounds__(kFieldBlock) void k_field(const InstDev* __restrict__ insts,
                                                      RunDev* __restrict__ runs,
                                                      const int32_t* __restrict__ blk_inst,
                                                      const int32_t* __restrict__ blk_row0) {
  __shared__ int wcount[kFieldBlock / 64];
  __shared__ int bbase;
  const int q = blk_inst[blockIdx.x];
  const RunDev* R = runs + q;
  const bool resume = R->paused != 0;
  if (!R->active && !resume) return;
  const InstDev* I = insts + q;
  const int wave = threadIdx.x >> 6;
  const int64_t wave_row0 = (int64_t)blk_row0[blockIdx.x] + wave * 64;
  uint32_t payload = 0;
  double key = 0.0;
  if (wave_row0 < I->n) key = field_rows64(I, wave_row0, R->t, payload, resume);
  const unsigned long long bal = __ballot(key > 0.0);
  if ((threadIdx.x & 63) == 0) wcount[wave] = __popcll(bal);
  __syncthreads();
  if (threadIdx.x == 0) {
    int tot = 0;
    for (int w = 0; w < kFieldBlock / 64; ++w) {
      const int c = wcount[w];
      wcount[w] = tot;
      tot += c;
    }
    bbase = tot ? atomicAdd(I->ccount, tot) : 0;
  }
  __syncthreads();
  if (bal) pool_put(I, key, payload, bal, (int64_t)bbase + wcount[wave]);
}

// Full-field pass for an instance of high degree (every row gathered): a
// workgroup of 8 R threads takes R consecutive rows of a 64-row slice (R =
// 64, 32, 16 or 8, fewer rows per workgroup for smaller instances, so that
// the device holds enough workgroups).  Each thread keeps one row, so it
// loads only that row's real slots (slot < len): no padding is read.  The
// slots are read in chunks of kHdChunk, eight entries per thread, the next
// chunk's couplings and spins in flight while the current one is added and
// the columns two chunks ahead; each entry's signed couplings are staged in
// LDS, and the lane of each row adds its chunk in ascending slot order: the
// same sums, in the same order, as field_row.  The workgroups of one slice
// are launched on the same XCD (block ids that differ by multiples of 8),
// so lines shared by two of them are fetched into one L2.

template <int R>
__global__ __launch_bounds__(8 * R) void k_field_hd(const InstDev* __restrict__ insts,
                                                    RunDev* __restrict__ runs) {
  constexpr int S = 64 / R;  // workgroups per slice
  __shared__ double sa[kHdChunk * R];
  __shared__ double sb[kHdChunk * R];
  __shared__ int lmax;
  const RunDev* Rn = runs;
  if (!Rn->active) return;
  const InstDev* I = insts;
  const int q = blockIdx.x;
  const int64_t slice = (int64_t)(q / (8 * S)) * 8 + (q % 8);
  const int sub = (q / 8) % S;
  const int64_t row0 = slice * 64;
  if (row0 >= I->n) return;
  const int tid = threadIdx.x;
  const int r = tid % R;    // the thread's row in the workgroup's R rows
  const int s0 = tid / R;   // its first slot in a chunk; then every 8th
  const int64_t i = row0 + sub * R + r;
  const int32_t L = (i < I->n) ? I->len[i] : 0;
  const int32_t D = I->D;
  const int64_t base = slot_of(row0, D, 0) + sub * R + r;  // slot 0 of the thread's row
  const int8_t* __restrict__ s = I->s;
  if (tid == 0) lmax = 0;
  __syncthreads();
  if (tid < R && L > 0) atomicMax(&lmax, L);
  __syncthreads();
  const int32_t Lw = lmax;  // slots of the longest of the workgroup's rows
  double p = 0.0, pq = 0.0;
  int32_t jc[kHdPer];
  double a[kHdPer], b[kHdPer];
  int sg[kHdPer];
  // chunk 0: columns, then couplings and spins; columns of chunk 1
#pragma unroll
  for (int u = 0; u < kHdPer; ++u) {
    const int k = s0 + 8 * u;
    jc[u] = (k < L) ? __builtin_nontemporal_load(&I->col[base + (int64_t)k * 64]) : 0;
  }
#pragma unroll
  for (int u = 0; u < kHdPer; ++u) {
    const int k = s0 + 8 * u;
    const bool ok = k < L;
    a[u] = ok ? __builtin_nontemporal_load(&I->A[base + (int64_t)k * 64]) : 0.0;
    b[u] = ok ? __builtin_nontemporal_load(&I->B[base + (int64_t)k * 64]) : 0.0;
    sg[u] = ok ? s[jc[u]] : 0;
  }
#pragma unroll
  for (int u = 0; u < kHdPer; ++u) {
    const int k = kHdChunk + s0 + 8 * u;
    jc[u] = (k < L) ? __builtin_nontemporal_load(&I->col[base + (int64_t)k * 64]) : 0;
  }
  for (int32_t k0 = 0; k0 < Lw; k0 += kHdChunk) {
#pragma unroll
    for (int u = 0; u < kHdPer; ++u) {
      const int e = (s0 + 8 * u) * R + r;
      sa[e] = (sg[u] > 0) ? a[u] : -a[u];
      sb[e] = (sg[u] > 0) ? b[u] : -b[u];
    }
    __syncthreads();
    // the next chunk's couplings and spins, and the columns after it, are
    // loaded while the current chunk is added
    const int32_t k1 = k0 + kHdChunk;
#pragma unroll
    for (int u = 0; u < kHdPer; ++u) {
      const int k = k1 + s0 + 8 * u;
      const bool ok = k < L;
      a[u] = ok ? __builtin_nontemporal_load(&I->A[base + (int64_t)k * 64]) : 0.0;
      b[u] = ok ? __builtin_nontemporal_load(&I->B[base + (int64_t)k * 64]) : 0.0;
      sg[u] = ok ? s[jc[u]] : 0;
    }
#pragma unroll
    for (int u = 0; u < kHdPer; ++u) {
      const int k = k1 + kHdChunk + s0 + 8 * u;
      jc[u] = (k < L) ? __builtin_nontemporal_load(&I->col[base + (int64_t)k * 64]) : 0;
    }
    if (tid < R && k0 < L) {
      // the chunk's sum from zero, then added to the row's (canonical order)
      const int kn = L - k0 < kHdChunk ? L - k0 : kHdChunk;
      double cp = 0.0, cq = 0.0;
      for (int kk = 0; kk < kn; ++kk) {
        cp += sa[kk * R + tid];
        cq += sb[kk * R + tid];
      }
      p += cp;
      pq += cq;
    }
    __syncthreads();
  }
  if (tid >= 64) return;
  uint32_t payload = 0;
  double key = 0.0;
  if (tid < R && i < I->n) key = field_finish(I, i, Rn->t, p, pq, payload);
  if (S == 1) {
    double mk = key;
    uint32_t mp = payload;
    wave_argmax(mk, mp);
    if (tid == 0) {
      I->t1key[row0 >> 6] = mk;
      I->t1idx[row0 >> 6] = mp;
    }
  }
  const unsigned long long bal = __ballot(key > 0.0);
  if (bal) {
    int pbase = 0;
    if (tid == 0) pbase = atomicAdd(I->ccount, __popcll(bal));
    pbase = __builtin_amdgcn_readfirstlane(pbase);
    pool_put(I, key, payload, bal, pbase);
  }
}

// The high-degree pass split over the 64-slot chunks, for instances too
// small to fill the device with k_field_hd (each of whose workgroups walks
// its rows' chunks one round trip after another).  k_field_hd_part: a
// 512-thread workgroup per (64-row slice, chunk) loads the chunk's slots of
// its rows (eight per thread, couplings and columns together, then the
// spins), stages the signed couplings in LDS, and the lane of each row adds
// its chunk in ascending slot order from zero; the sums go to I->part.
// k_field_hd_comb: a lane per row adds its chunk sums in ascending order --
// the canonical order of every pass -- then finishes the row (Eq. 2, the
// key), and each wavefront writes its 64 rows' maximum for the relax tree.
__global__ __launch_bounds__(512) void k_field_hd_part(const InstDev* __restrict__ insts,
                                                       RunDev* __restrict__ runs) {
  __shared__ double sa[kHdChunk * 64];
  __shared__ double sb[kHdChunk * 64];
  if (!runs->active) return;
  const InstDev* I = insts;
  const int nch = I->nch;
  const int64_t slice = blockIdx.x / nch;
  const int g = (int)(blockIdx.x % nch);
  const int64_t row0 = slice * 64;
  if (row0 >= I->n) return;
  const int tid = threadIdx.x;
  const int r = tid & 63;   // the thread's row in the slice
  const int s0 = tid >> 6;  // its first slot in the chunk; then every 8th
  const int64_t i = row0 + r;
  const int32_t L = (i < I->n) ? I->len[i] : 0;
  const int64_t base = slot_of(row0, I->D, 0) + r;  // slot 0 of the thread's row
  const int k0 = g * kHdChunk;
  const int8_t* __restrict__ s = I->s;
  int32_t jc[kHdPer];
  double a[kHdPer], b[kHdPer];
  int sg[kHdPer];
#pragma unroll
  for (int u = 0; u < kHdPer; ++u) {
    const int k = k0 + s0 + 8 * u;
    const bool ok = k < L;
    jc[u] = ok ? __builtin_nontemporal_load(&I->col[base + (int64_t)k * 64]) : 0;
    a[u] = ok ? __builtin_nontemporal_load(&I->A[base + (int64_t)k * 64]) : 0.0;
    b[u] = ok ? __builtin_nontemporal_load(&I->B[base + (int64_t)k * 64]) : 0.0;
  }
#pragma unroll
  for (int u = 0; u < kHdPer; ++u) sg[u] = (k0 + s0 + 8 * u < L) ? s[jc[u]] : 0;
#pragma unroll
  for (int u = 0; u < kHdPer; ++u) {
    const int e = (s0 + 8 * u) * 64 + r;
    sa[e] = (sg[u] > 0) ? a[u] : -a[u];
    sb[e] = (sg[u] > 0) ? b[u] : -b[u];
  }
  __syncthreads();
  if (tid < 64 && k0 < L) {
    const int kn = L - k0 < kHdChunk ? L - k0 : kHdChunk;
    double cp = 0.0, cq = 0.0;
    for (int kk = 0; kk < kn; ++kk) {
      cp += sa[kk * 64 + tid];
      cq += sb[kk * 64 + tid];
    }
    I->part[(int64_t)g * I->n + i] = make_double2(cp, cq);
  }
}

__global__ __launch_bounds__(256) void k_field_hd_comb(const InstDev* __restrict__ insts,
                                                       RunDev* __restrict__ runs) {
  const RunDev* Rn = runs;
  if (!Rn->active) return;
  const InstDev* I = insts;
  const int lane = threadIdx.x & 63;
  const int64_t g64 = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t row0 = g64 << 6;
  if (row0 >= I->n) return;
  const int64_t i = row0 + lane;
  uint32_t payload = 0;
  double key = 0.0;
  if (i < I->n) {
    const int32_t L = I->len[i];
    double p = 0.0, pq = 0.0;
    for (int c = 0; c * kHdChunk < L; ++c) {
      const double2 v = I->part[(int64_t)c * I->n + i];
      p += v.x;
      pq += v.y;
    }
    key = field_finish(I, i, Rn->t, p, pq, payload);
  }
  double mk = key;
  uint32_t mp = payload;
  wave_argmax(mk, mp);
  if (lane == 0) {
    I->t1key[g64] = mk;
    I->t1idx[g64] = mp;
  }
  const unsigned long long bal = __ballot(key > 0.0);
  if (bal) {
    int pbase = 0;
    if (lane == 0) pbase = atomicAdd(I->ccount, __popcll(bal));
    pbase = __builtin_amdgcn_readfirstlane(pbase);
    pool_put(I, key, payload, bal, pbase);
  }
}

// Per-64-row maxima of the keys a split high-degree pass wrote (one
// wavefront per 64 rows), for the relax tree.
__global__ __launch_bounds__(256) void k_slice_max(const InstDev* __restrict__ insts,
                                                   RunDev* __restrict__ runs) {
  if (!runs->active) return;
  const InstDev* I = insts;
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t i = (g << 6) + lane;
  if ((g << 6) >= I->n) return;
  double k = 0.0;
  uint32_t pay = 0u;
  if (i < I->n) {
    k = I->key[i];
    pay = (uint32_t)i | (I->s[i] < 0 ? 0x80000000u : 0u);
  }
  wave_argmax(k, pay);
  if (lane == 0) {
    I->t1key[g] = k;
    I->t1idx[g] = pay;
  }
}

// The relax workgroup's dynamic LDS.
extern __shared__ __align__(16) unsigned char lds_dyn[];

// A part of a relax called out of line.  Each starts on a 256-byte boundary: where
// the batches by tiles happened to start elsewhere, after changes to other
// functions, they were 1-2 % slower.
#define ASI_CALLED __attribute__((noinline, aligned(256)))

// Values that the whole workgroup shares but the compiler cannot know to be
// the same in every lane (arguments of a function called out of line, values
// read from LDS); a descriptor, which no kernel writes, also lies in constant
// memory (scalar loads).
#define ASI_LDS __attribute__((address_space(3)))
#define ASI_CONST __attribute__((address_space(4)))

__device__ __forceinline__ const InstDev* uniform(const InstDev* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return (const InstDev*)(const ASI_CONST InstDev*)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ int64_t uniform(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)((uint64_t)hi << 32 | lo);
}

// ------------------------------------------------------------ relax
struct RelaxLds {
  double* l1k;                // first level: maximum key of each tile
  uint32_t* l1i;              //   its index | sign bit
  int32_t* l1flag;            //   tile touched by the current flip
  unsigned long long* l1nk;   //   largest new key of the flip's updates (bits), 0: none
  unsigned long long* l1ni;   //   lowest (index << 1 | spin<0) among updates with that key
  int32_t* l1resc;            //   the tile's maximum was updated: rescan it
  int32_t* l1rlist;           //   tiles to rescan
  double* l2k;                // second level: maximum over 64 tiles
  uint32_t* l2i;
  int32_t* l2flag;            //   group touched by the current flip
};

__host__ __device__ inline size_t align16(size_t v) { return (v + 15) & ~(size_t)15; }

__host__ __device__ inline size_t relax_tree_lds_bytes(int64_t n, int32_t l1_shift) {
  const int64_t nt1 = (n + (1LL << l1_shift) - 1) >> l1_shift;
  const int64_t nt2 = (nt1 + kL2Group - 1) / kL2Group;
  size_t off = 0;
  off = align16(off + sizeof(unsigned long long) * nt1);
  off = align16(off + sizeof(unsigned long long) * nt1);
  off = align16(off + sizeof(double) * nt1);
  off = align16(off + sizeof(uint32_t) * nt1);
  for (int a = 0; a < 3; ++a) off = align16(off + sizeof(int32_t) * nt1);
  off = align16(off + sizeof(double) * nt2);
  off = align16(off + sizeof(uint32_t) * nt2);
  off = align16(off + sizeof(int32_t) * nt2);
  return off;
}

__device__ inline RelaxLds carve(unsigned char* base, int nt1, int nt2) {
  RelaxLds L;
  size_t off = 0;
  L.l1nk = (unsigned long long*)(base + off);
  off = align16(off + sizeof(unsigned long long) * nt1);
  L.l1ni = (unsigned long long*)(base + off);
  off = align16(off + sizeof(unsigned long long) * nt1);
  L.l1k = (double*)(base + off);
  off = align16(off + sizeof(double) * nt1);
  L.l1i = (uint32_t*)(base + off);
  off = align16(off + sizeof(uint32_t) * nt1);
  L.l1flag = (int32_t*)(base + off);
  off = align16(off + sizeof(int32_t) * nt1);
  L.l1resc = (int32_t*)(base + off);
  off = align16(off + sizeof(int32_t) * nt1);
  L.l1rlist = (int32_t*)(base + off);
  off = align16(off + sizeof(int32_t) * nt1);
  L.l2k = (double*)(base + off);
  off = align16(off + sizeof(double) * nt2);
  L.l2i = (uint32_t*)(base + off);
  off = align16(off + sizeof(uint32_t) * nt2);
  L.l2flag = (int32_t*)(base + off);
  return L;
}

struct RelaxShared {
  int nr;  // tiles to rescan
  int pause;  // the relax stops here and resumes in a later launch
  double key;
  uint32_t pay;
  // predicted next flip: high 32 bits of the best updated key, then its index
  unsigned long long pfk;
  // runner-up of the tree before the flip (j's own tile left out), packed the
  // same way; 0 when none is known
  unsigned long long ruk;
};

// True once the deadline (device constant-rate clock; 0: none) has passed.
__device__ inline bool past(uint64_t deadline) {
  return deadline != 0 && (uint64_t)wall_clock64() > deadline;
}

// ------------------------------------------------------------ speculative relax
// Exact-order batched relax for steps that start with many flippable
// magnets.  Candidates live in a pool in memory (filled by the field phase)
// and a hot window in LDS that is sorted best first (largest key, then lowest
// index).  Entries are (key, index | sign bit, version); an entry is valid
// while its version equals the magnet's version counter, which every change
// of the magnet's key bumps.  Every valid pool entry is no better than
// cold_max, so window entries better than cold_max can be taken in order.
//
// Entries that a batch's updates add above cold_max wait in a small sorted
// side list and join the window when that is full, so that a batch does not
// move the window.
//
// A batch takes the first B entries c_1 .. c_B of the window's safe part and
// the side list, and flips the longest prefix c_1 .. c_p (stale entries left
// out) that the one-at-a-time relax would flip in the same order: the members
// and their neighbour sets are pairwise disjoint (so no member's field or key
// depends on an earlier member of the prefix, and every touched magnet gets
// exactly one update), and no touched magnet's new key beats a later member of
// the prefix.  Then c_m is the argmax after c_1 .. c_{m-1} for every m <= p,
// and applying the prefix together gives the same flips, log, fields and keys,
// bit for bit.
constexpr int kWin = 2048;        // hot window entries
constexpr int kHash = 4096;       // conflict table slots
constexpr int kMaxPairs = 1024;   // member + neighbour slots per batch: one per thread
constexpr int kMaxMembers = 64;   // one per lane of the wavefront that chooses them
constexpr int kSide = 32;         // side-list entries
// A step whose batches so far, kSwitchBatches or more, commit fewer than
// kSwitchFlips (unless spec_switch is given) flips each on average -- an
// avalanche: every flip makes a neighbour the next candidate -- continues on the
// max tree, which costs about half a batch per flip on such steps.
constexpr int kSwitchBatches = 16;
// Where the one-at-a-time relax holds its keys in LDS, a batch costs about
// eight of its flips up to 10,000 magnets and five at 36,000, whose tiles are
// longer; but a step's batches shrink and grow again, so it goes over when all
// of its batches so far, four or more, commit fewer flips on average than 7, or
// 4 above 10,000 magnets at up to 64 neighbours.  (Four batches in a row below
// nine, as it was: 36,300-magnet kagome at 14 neighbours 2.04 us a flip, 1.11
// so; 24,300 at 8 neighbours 0.42, 0.25; 36,100-magnet Ising row at 4 2.82,
// 1.80.  With 4 throughout, 4,800-magnet kagome at 14 and 70 neighbours 1.52
// and 1.57, with 7 1.30 and 1.43; with 7 throughout the former 1.55 and 2.53.)
constexpr int kSwitchBatchesLds = 4;
constexpr double kSwitchFlips = 2.5, kSwitchFlipsLds = 7.0, kSwitchFlipsLdsLarge = 4.0;
constexpr int64_t kSwitchLargeN = 10000;
// A batch by tiles (relax_many) costs about a flip on the max tree, so those
// steps stay (36,180-magnet pinwheel at 24 neighbours 2.2 -> 1.4 us a flip).
// With keys in LDS a flip costs a third of a batch, but a step that starts
// with small batches often grows them again: going over below 1.5 flips a batch
// over four batches takes 0.80 us a flip on a 30,000-magnet kagome at 32
// neighbours (below 3: 1.12, never: 0.77) and 50 ms on the 29,040-magnet
// reversal at 60 neighbours, which is one avalanche (never: 129 ms).
constexpr int kManySwitchBatches = 4;
constexpr double kManySwitchLds = 1.5;

// Relax order of two magnets: larger key first, then lower index.
__device__ inline bool better(double ka, uint32_t pa, double kb, uint32_t pb) {
  return ka > kb || (ka == kb && (pa & 0x7fffffffu) < (pb & 0x7fffffffu));
}

// Order of pool and window entries: the relax order, then the newer version
// of the same magnet first, so that no two distinct entries tie.
__device__ inline bool better_e(double ka, uint32_t pa, uint32_t va, double kb, uint32_t pb,
                                uint32_t vb) {
  if (ka != kb) return ka > kb;
  const uint32_t ia = pa & 0x7fffffffu, ib = pb & 0x7fffffffu;
  if (ia != ib) return ia < ib;
  return va > vb;
}

struct SpecLds {
  unsigned char* win;  // hot window, two buffers of kWin entries each:
                       //   buffer b: keys at win + b * kWinBytes, then payloads, versions
  double* sk;       // staging / sort scratch (aliases the list of keys to evaluate)
  uint32_t* sp;
  uint32_t* sv;
  uint32_t* hidx;   // conflict table: magnet + 1 (0: empty)
  int32_t* hown;    //   first member that owns or touches that magnet
  double* lk;       // side list, best first
  uint32_t* lp;
  uint32_t* lv;
  double* mk;       // members, best first: key, payload, version (two sets, by turns)
  uint32_t* mp;
  uint32_t* mv;
  int32_t* mval;    // member's entry is current
};
constexpr int32_t kNoOwner = 0x7fffffff;

constexpr size_t kWinBytes = (size_t)kWin * 16;
__device__ inline double* win_k(const SpecLds& S, int b) {
  return (double*)(S.win + (size_t)b * kWinBytes);
}
__device__ inline uint32_t* win_p(const SpecLds& S, int b) {
  return (uint32_t*)(S.win + (size_t)b * kWinBytes + sizeof(double) * kWin);
}
__device__ inline uint32_t* win_v(const SpecLds& S, int b) {
  return (uint32_t*)(S.win + (size_t)b * kWinBytes + (sizeof(double) + sizeof(uint32_t)) * kWin);
}

__host__ __device__ inline size_t spec_lds_bytes() {
  return 2 * (size_t)kWin * 16 + (size_t)kWin * 16 + (size_t)kHash * 8 + (size_t)kSide * 16 +
         (size_t)kMaxMembers * (2 * 16 + 4);
}

__device__ inline SpecLds carve_spec(unsigned char* base) {
  SpecLds S;
  S.win = base;
  base += 2 * kWinBytes;
  S.sk = (double*)base;
  S.sp = (uint32_t*)(base + sizeof(double) * kWin);
  S.sv = S.sp + kWin;
  base += (size_t)kWin * 16;
  S.hidx = (uint32_t*)base;
  S.hown = (int32_t*)(S.hidx + kHash);
  base += (size_t)kHash * 8;
  S.lk = (double*)base;
  S.lp = (uint32_t*)(S.lk + kSide);
  S.lv = S.lp + kSide;
  base += (size_t)kSide * 16;
  S.mk = (double*)base;
  S.mp = (uint32_t*)(S.mk + 2 * kMaxMembers);
  S.mv = S.mp + 2 * kMaxMembers;
  S.mval = (int32_t*)(S.mv + 2 * kMaxMembers);
  return S;
}

struct SpecShared {
  int a0, nx, xb;   // window: first entry not consumed, end, buffer
  int B, pe;        // batch size; end of its prefix
  int nl, nl_next;  // side-list entries at the last choice; at this one
  int nm;           // entries that join the window
  int ns, npow, cb, pause;
  int64_t ncold, ncold_out, napp;
  double cmk;       // cold_max (key, payload, version); key -1: pool empty
  uint32_t cmp, cmv;
  double rk;        // best entry a merge discarded into the pool
  uint32_t rp, rv;
  double tau;       // refill threshold (selective refill)
  int over;         // selective refill: more entries above tau than fit
  double wk[16];    // per-wavefront best entries (selective refill)
  uint32_t wp[16], wv[16];
  uint64_t hash;
};

// Block-wide bitonic sort, best first, of P (a power of two) entries.
__device__ __forceinline__ void bitonic_best_first(double* k, uint32_t* p, uint32_t* v, int P) {
  const int tid = threadIdx.x, NT = blockDim.x;
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int q = tid; q < P / 2; q += NT) {
        const int lo = 2 * stride * (q / stride) + (q % stride);
        const int hi = lo + stride;
        const bool up = (lo & size) == 0;  // this segment runs best first
        const bool sw = up ? better_e(k[hi], p[hi], v[hi], k[lo], p[lo], v[lo])
                           : better_e(k[lo], p[lo], v[lo], k[hi], p[hi], v[hi]);
        if (sw) {
          const double tk = k[lo];
          k[lo] = k[hi];
          k[hi] = tk;
          const uint32_t tp = p[lo];
          p[lo] = p[hi];
          p[hi] = tp;
          const uint32_t tv = v[lo];
          v[lo] = v[hi];
          v[hi] = tv;
        }
      }
      __syncthreads();
    }
  }
}

// Number of entries taken from A among the first d outputs of merge(A, B)
// (both best first; on equal entries A goes first).
__device__ __forceinline__ int co_rank(int d, const double* ak, const uint32_t* ap,
                                      const uint32_t* av, int na, const double* bk,
                                      const uint32_t* bp, const uint32_t* bv, int nb) {
  int lo = d > nb ? d - nb : 0;
  int hi = d < na ? d : na;
  while (lo < hi) {
    const int i = (lo + hi) >> 1;
    const int j = d - i;
    if (j > 0 && i < na && !better_e(bk[j - 1], bp[j - 1], bv[j - 1], ak[i], ap[i], av[i]))
      lo = i + 1;
    else
      hi = i;
  }
  return lo;
}

// Merge A = the window's entries not consumed with B = staging[0, nb) (both
// best first): the first `keep` outputs become the window (other buffer), the
// rest are appended to pool buffer pb at sh.ncold_out; sh.rk/rp keeps the best
// entry sent to the pool.
__device__ __forceinline__ void merge_keep(const InstDev* I, const SpecLds& S, SpecShared& sh, int nb,
                           int pb) {
  const int tid = threadIdx.x, NT = blockDim.x;
  const int xb = sh.xb, a0 = sh.a0, na = sh.nx - a0;
  const int keep = na + nb < kWin ? na + nb : kWin;
  const double* ak = win_k(S, xb) + a0;
  const uint32_t* ap = win_p(S, xb) + a0;
  const uint32_t* av = win_v(S, xb) + a0;
  double* ok = win_k(S, xb ^ 1);
  uint32_t* op = win_p(S, xb ^ 1);
  uint32_t* ov = win_v(S, xb ^ 1);
  uint32_t* pool_p = I->cpay[pb];
  double* pool_k = I->ckey[pb];
  uint32_t* pool_v = I->cver[pb];
  const int total = na + nb;
  const int per = (total + NT - 1) / NT;
  const int d0 = tid * per < total ? tid * per : total;
  const int d1 = d0 + per < total ? d0 + per : total;
  const int64_t base = sh.ncold_out;
  if (d0 < d1) {
    int i = co_rank(d0, ak, ap, av, na, S.sk, S.sp, S.sv, nb);
    int j = d0 - i;
    for (int d = d0; d < d1; ++d) {
      double ek;
      uint32_t epay, ever;
      if (j >= nb || (i < na && !better_e(S.sk[j], S.sp[j], S.sv[j], ak[i], ap[i], av[i]))) {
        ek = ak[i];
        epay = ap[i];
        ever = av[i];
        ++i;
      } else {
        ek = S.sk[j];
        epay = S.sp[j];
        ever = S.sv[j];
        ++j;
      }
      if (d < keep) {
        ok[d] = ek;
        op[d] = epay;
        ov[d] = ever;
      } else {
        const int64_t q = base + (d - keep);
        pool_k[q] = ek;
        pool_p[q] = epay;
        pool_v[q] = ever;
        if (d == keep && better_e(ek, epay, ever, sh.rk, sh.rp, sh.rv)) {
          sh.rk = ek;
          sh.rp = epay;
          sh.rv = ever;
        }
      }
    }
  }
  __syncthreads();
  if (tid == 0) {
    sh.ncold_out += total - keep;
    sh.xb ^= 1;
    sh.a0 = 0;
    sh.nx = keep;
  }
  __syncthreads();
}

// Sort staging entries [0, ns) best first.  Up to one entry per thread:
// each thread counts the entries that beat its own (every thread reads the
// same entry at a time, a broadcast) and moves it to that rank; no two
// entries tie under the pool order.  Larger sets: bitonic sort, padded to a
// power of two.
__device__ __forceinline__ void sort_staging(const SpecLds& S, int ns) {
  const int tid = threadIdx.x;
  if (ns <= (int)blockDim.x) {
    double k = 0.0;
    uint32_t p = 0, v = 0;
    int rank = 0;
    if (tid < ns) {
      k = S.sk[tid];
      p = S.sp[tid];
      v = S.sv[tid];
      for (int q = 0; q < ns; ++q) rank += better_e(S.sk[q], S.sp[q], S.sv[q], k, p, v) ? 1 : 0;
    }
    __syncthreads();
    if (tid < ns) {
      S.sk[rank] = k;
      S.sp[rank] = p;
      S.sv[rank] = v;
    }
    __syncthreads();
    return;
  }
  int P = 1;
  while (P < ns) P <<= 1;
  for (int q = ns + tid; q < P; q += blockDim.x) {
    S.sk[q] = -1.0;
    S.sp[q] = 0x7fffffffu;
    S.sv[q] = 0u;
  }
  __syncthreads();
  bitonic_best_first(S.sk, S.sp, S.sv, P);
}

// Window := best kWin entries of (window + valid pool entries); the other
// valid pool entries move to the other pool buffer; cold_max becomes exact.
__device__ __forceinline__ void refill(const InstDev* I, const SpecLds& S, SpecShared& sh) {
  const int tid = threadIdx.x, NT = blockDim.x;
  const int cb = sh.cb;
  const int64_t ncold = sh.ncold;
  if (tid == 0) {
    sh.ncold_out = 0;
    sh.rk = -1.0;
    sh.rp = 0x7fffffffu;
    sh.rv = 0u;
  }
  __syncthreads();
  for (int64_t c0 = 0; c0 < ncold; c0 += kWin) {
    const int m = (int)(ncold - c0 < kWin ? ncold - c0 : kWin);
    for (int q = tid; q < m; q += NT) {
      const uint32_t pay = I->cpay[cb][c0 + q];
      const uint32_t ver = I->cver[cb][c0 + q];
      const bool ok = I->ver[pay & 0x7fffffffu] == ver;
      S.sk[q] = ok ? I->ckey[cb][c0 + q] : -1.0;
      S.sp[q] = ok ? pay : 0x7fffffffu;
      S.sv[q] = ok ? ver : (uint32_t)q;  // invalid entries: distinct, sorted last
    }
    __syncthreads();
    sort_staging(S, m);
    if (tid == 0) {
      int lo = 0, hi = m;  // valid entries sort first
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (S.sk[mid] > 0.0) lo = mid + 1; else hi = mid;
      }
      sh.ns = lo;
    }
    __syncthreads();
    merge_keep(I, S, sh, sh.ns, cb ^ 1);
  }
  if (tid == 0) {
    sh.cb = cb ^ 1;
    sh.ncold = sh.ncold_out;
    sh.cmk = sh.rk;
    sh.cmp = sh.rp;
    sh.cmv = sh.rv;
  }
  __syncthreads();
}

// Refill for a large pool: a threshold tau from a sorted sample of the
// pool's keys puts about kWin / 2 entries above it; one pass drops stale
// entries, sends the current ones above tau to staging and those at or
// below tau to the other pool buffer, keeping the best of those (pool
// order) as the cold bound; staging is sorted and merged into the window,
// whose overflow joins the pool and the bound, which stays exact.  Only
// about kWin entries are sorted instead of the whole pool.  If more current
// entries than staging holds lie above tau, or none does, the pass is
// discarded and the full refill runs instead.
__device__ __forceinline__ void refill_select(const InstDev* I, const SpecLds& S, SpecShared& sh) {
  const int tid = threadIdx.x, NT = blockDim.x, lane = tid & 63, wave = tid >> 6;
  const int cb = sh.cb;
  const int64_t ncold = sh.ncold;
  for (int q = tid; q < kWin; q += NT) {
    S.sk[q] = I->ckey[cb][(int64_t)q * ncold / kWin];
    S.sp[q] = (uint32_t)q;
    S.sv[q] = 0u;
  }
  __syncthreads();
  bitonic_best_first(S.sk, S.sp, S.sv, kWin);
  if (tid == 0) {
    int r = (int)((int64_t)(kWin / 2) * kWin / ncold);
    if (r < 1) r = 1;
    sh.tau = S.sk[r];
    sh.ns = 0;
    sh.over = 0;
    sh.ncold_out = 0;
    sh.rk = -1.0;
    sh.rp = 0x7fffffffu;
    sh.rv = 0u;
  }
  __syncthreads();
  const double tau = sh.tau;
  const unsigned long long lt = (1ull << lane) - 1ull;
  double bk = -1.0;
  uint32_t bp = 0x7fffffffu, bv = 0u;
  for (int64_t q0 = 0; q0 < ncold; q0 += NT) {
    const int64_t q = q0 + tid;
    bool up = false, down = false;
    double k = 0.0;
    uint32_t pay = 0, ver = 0;
    if (q < ncold) {
      k = I->ckey[cb][q];
      pay = I->cpay[cb][q];
      ver = I->cver[cb][q];
      const bool cur = I->ver[pay & 0x7fffffffu] == ver;
      up = cur && k > tau;
      down = cur && !(k > tau);
    }
    const unsigned long long bu = __ballot(up), bd = __ballot(down);
    int ubase = 0, dbase = 0;
    if (lane == 0) {
      if (bu) ubase = atomicAdd(&sh.ns, __popcll(bu));
      if (bd) dbase = (int)atomicAdd((unsigned long long*)&sh.ncold_out, (unsigned long long)__popcll(bd));
    }
    ubase = __builtin_amdgcn_readfirstlane(ubase);
    dbase = __builtin_amdgcn_readfirstlane(dbase);
    if (up) {
      const int pos = ubase + __popcll(bu & lt);
      if (pos < kWin) {
        S.sk[pos] = k;
        S.sp[pos] = pay;
        S.sv[pos] = ver;
      } else {
        sh.over = 1;
      }
    }
    if (down) {
      const int64_t pos = dbase + __popcll(bd & lt);
      I->ckey[cb ^ 1][pos] = k;
      I->cpay[cb ^ 1][pos] = pay;
      I->cver[cb ^ 1][pos] = ver;
      if (better_e(k, pay, ver, bk, bp, bv)) {
        bk = k;
        bp = pay;
        bv = ver;
      }
    }
  }
  // best entry sent down: per wavefront, then over the wavefronts
  for (int off = 32; off > 0; off >>= 1) {
    const double ok = __shfl_down(bk, off);
    const uint32_t op = __shfl_down(bp, off), ov = __shfl_down(bv, off);
    if (lane + off < 64 && better_e(ok, op, ov, bk, bp, bv)) {
      bk = ok;
      bp = op;
      bv = ov;
    }
  }
  if (lane == 0) {
    sh.wk[wave] = bk;
    sh.wp[wave] = bp;
    sh.wv[wave] = bv;
  }
  __syncthreads();
  // Too many current entries above tau, or none (ties at the top of the
  // sample can put tau on the best key): the full refill, from the same pool.
  if (sh.over || sh.ns == 0) {
    refill(I, S, sh);
    return;
  }
  if (tid == 0) {
    for (int w = 0; w < (NT >> 6); ++w)
      if (better_e(sh.wk[w], sh.wp[w], sh.wv[w], sh.rk, sh.rp, sh.rv)) {
        sh.rk = sh.wk[w];
        sh.rp = sh.wp[w];
        sh.rv = sh.wv[w];
      }
  }
  __syncthreads();
  const int ns = sh.ns;
  sort_staging(S, ns);
  merge_keep(I, S, sh, ns, cb ^ 1);
  if (tid == 0) {
    sh.cb = cb ^ 1;
    sh.ncold = sh.ncold_out;
    sh.cmk = sh.rk;
    sh.cmp = sh.rp;
    sh.cmv = sh.rv;
  }
  __syncthreads();
}


// End of the window's safe part: its entries better than cold_max (all of
// them when the pool is empty), counted by one wavefront (every lane gets the
// end): they are a prefix, so 64 segment ends locate the boundary's segment,
// and one lane per entry of that segment finds it.
__device__ __forceinline__ int safe_end_wave(const SpecLds& S, const SpecShared& sh) {
  const int lane = threadIdx.x & 63;
  const int a0 = sh.a0, nx = sh.nx - a0;
  if (sh.ncold == 0 || nx == 0) return sh.nx;
  const double* k = win_k(S, sh.xb) + a0;
  const uint32_t* p = win_p(S, sh.xb) + a0;
  const uint32_t* v = win_v(S, sh.xb) + a0;
  const double cmk = sh.cmk;
  const uint32_t cmp = sh.cmp, cmv = sh.cmv;
  const int step = (nx + 63) >> 6;
  const int e = (lane + 1) * step - 1;
  const bool ok = e < nx && better_e(k[e], p[e], v[e], cmk, cmp, cmv);
  const int c = __popcll(__ballot(ok));
  const int e2 = c * step + lane;
  const bool ok2 = lane < step && e2 < nx && better_e(k[e2], p[e2], v[e2], cmk, cmp, cmv);
  return a0 + c * step + __popcll(__ballot(ok2));
}

__device__ inline uint32_t hash_slot(uint32_t i) { return (i * 2654435761u) >> (32 - 12); }

// Out of line, so that their registers stay out of the batch loop's.
__device__ ASI_CALLED void call_refill(const InstDev* I, ASI_LDS SpecShared* sh) {
  const SpecLds S = carve_spec(lds_dyn);
  SpecShared& h = *(SpecShared*)sh;
  if (h.ncold > 4 * kWin)
    refill_select(uniform(I), S, h);
  else
    refill(uniform(I), S, h);
}
// staging[0, nm) joins the window; what that pushes out joins the pool.
__device__ ASI_CALLED void call_join(const InstDev* I, ASI_LDS SpecShared* sh, int nm) {
  const SpecLds S = carve_spec(lds_dyn);
  SpecShared& h = *(SpecShared*)sh;
  nm = __builtin_amdgcn_readfirstlane(nm);
  if (threadIdx.x == 0) {
    h.ncold_out = h.ncold;
    h.rk = h.cmk;
    h.rp = h.cmp;
    h.rv = h.cmv;
  }
  __syncthreads();
  sort_staging(S, nm);
  merge_keep(uniform(I), S, h, nm, h.cb);
  if (threadIdx.x == 0) {
    h.ncold = h.ncold_out;
    h.cmk = h.rk;
    h.cmp = h.rp;
    h.cmv = h.rv;
  }
  __syncthreads();
}
__device__ ASI_CALLED double pow_far(double x, double e) { return pow(x, e); }

// Relax at step t in speculative batches (needs 1024 threads).  flips,
// logpos and hash are the running counters (hash significant in thread 0).
// Returns 0, -5 (flip cap reached with a flippable magnet left),
// 1 (deadline passed after at least one batch, flippable magnets left) or
// 2 (the mean batch is too small, see kSwitchBatches: the flippable magnets
// crowd each other's neighbourhoods, and the step goes on one flip at a time).
// What bounds it: a chain of phases per batch, six barriers apart -- the
// members' choice (one wavefront), their rows, their neighbours' fields (in
// flight while the conflicts are found; one wavefront folds the last batch into
// the hash meanwhile), the FP64 powers, one to a lane, and the commit: 21,000
// cycles for 16 members at 32 neighbours.  Against batches of up to 2,048 slots
// that merged the window each time (23,000 cycles): kagome of 120,000 magnets at
// 4 neighbours 0.215 -> 0.174 us a flip, of 24,300 0.27 -> 0.23, of 1.2M 0.28 ->
// 0.25, of 120,000 at 70 neighbours 1.47 -> 1.43.
__device__ __forceinline__ int relax_spec(const InstDev* __restrict__ I, int64_t t, unsigned char* lds,
                          SpecShared& sh, int64_t ncand, int64_t& flips, int64_t& logpos,
                          uint64_t& hash, uint64_t deadline) {
  const int tid = threadIdx.x, NT = blockDim.x, lane = tid & 63;
  const bool chooser = tid < 64, clerk = tid >= NT - 64;  // the first and the last wavefront
  SpecLds S = carve_spec(lds);
  const int32_t D = I->D;
  const int32_t mode = I->field_mode;
  const double pb = I->b, pc = I->c, ep = I->e_par, eq = I->e_perp;
  const int64_t max_flips = I->max_flips;
  const int PW = D + 1;  // pair slots per member: its neighbours and itself
  int Bmax = kMaxPairs / PW;
  if (Bmax > kMaxMembers) Bmax = kMaxMembers;
  // Members taken per batch: about twice the last committed prefix, since
  // the members past the prefix only cost loads and key evaluations;
  // doubled while whole batches commit.
  int bcap = Bmax;
  const int sm = tid / PW, sk = tid % PW;  // the thread's pair slot: member and place in its row
  for (int q = tid; q < kHash; q += NT) {
    S.hidx[q] = 0u;
    S.hown[q] = kNoOwner;
  }
  if (tid == 0) {
    sh.a0 = 0;
    sh.nx = 0;
    sh.xb = 0;
    sh.cb = 0;
    sh.ns = 0;
    sh.napp = 0;
    sh.nl = 0;
    sh.ncold = ncand;
    sh.cmk = 1e300;  // unknown until the first refill
    sh.cmp = 0;
    sh.cmv = 0;
  }
  __syncthreads();
  int status = 0;
  const int64_t flips0 = flips;
  const bool keys_in_lds = I->lds_keys != 0;
  const int nswitch = keys_in_lds ? kSwitchBatchesLds : kSwitchBatches;
  const double sw = I->spec_switch >= 0.0 ? I->spec_switch
                    : !keys_in_lds        ? kSwitchFlips
                    : I->n > kSwitchLargeN && D <= kManyMaxD ? kSwitchFlipsLdsLarge : kSwitchFlipsLds;
  int nbatch = 0;
  int set = 0;        // the members' set
  int consumed = 0;   // entries of the last batch that are done with
  unsigned long long committed = 0ull;  // members of the last batch that flipped
  // The clerk folds the last batch's flips into the hash while the next one's
  // rows are on their way.
  auto fold = [&]() {
    if (!clerk || committed == 0ull) return;
    const uint32_t jr = S.mp[(set ^ 1) * kMaxMembers + lane] & 0x7fffffffu;
    for (unsigned long long c = committed; c; c &= c - 1ull) {
      const uint32_t j = (uint32_t)__builtin_amdgcn_readlane((int)jr, __ffsll(c) - 1);
      hash = (hash ^ (((uint64_t)(uint32_t)t << 32) | j)) * 0x100000001b3ull;
    }
  };
  // the choosing wavefront's own: the window's safe part, its lanes' ranks in
  // the last batch, and the side list's remainder
  int a0 = 0, s_end = 0, nl = 0, rank_w = kMaxMembers, rank_l = kMaxMembers;
  while (true) {
    const int ns = sh.ns;
    // ---- the side list would overflow: it and the new entries join the window
    if (sh.nl + ns > kSide) {
      const int nl0 = sh.nl;
      if (chooser) {
        a0 += __popcll(__ballot(rank_w < consumed));
        const int cl = __popcll(__ballot(rank_l < consumed));
        rank_w = rank_l = kMaxMembers;
        const int rem = nl0 - cl;  // the side list's remainder goes behind the new entries
        if (lane < rem) {
          S.sk[ns + lane] = S.lk[cl + lane];
          S.sp[ns + lane] = S.lp[cl + lane];
          S.sv[ns + lane] = S.lv[cl + lane];
        }
        if (lane == 0) {
          sh.ncold += sh.napp;
          sh.napp = 0;
          sh.a0 = a0;
          sh.nm = ns + rem;
        }
      }
      __syncthreads();
      call_join(I, (ASI_LDS SpecShared*)&sh, sh.nm);
      if (tid == 0) {
        sh.ns = 0;
        sh.nl = 0;
      }
      __syncthreads();
      if (chooser) {
        a0 = 0;
        nl = 0;
        consumed = 0;
        s_end = safe_end_wave(S, sh);
      }
    }
    // ---- choice of the next members (first wavefront): its lanes hold the
    // window's next entries and the side list's, new entries among them; an
    // entry's rank is the number of entries that beat it.  The last wavefront
    // folds the batch just committed into the hash.
    bool refilled = false, none = false;
    while (true) {
      if (chooser) {
        a0 += __popcll(__ballot(rank_w < consumed));
        const int cl = __popcll(__ballot(rank_l < consumed));
        const int fresh = sh.ns, rem = nl - cl;
        nl = rem + fresh;
        const double* wk = win_k(S, sh.xb);
        const uint32_t* wp = win_p(S, sh.xb);
        const uint32_t* wv = win_v(S, sh.xb);
        const bool has_w = a0 + lane < s_end, has_l = lane < nl;
        double kw = 0.0, kl = 0.0;
        uint32_t pw = 0, vw = 0, pl = 0, vl = 0;
        if (has_w) {
          kw = wk[a0 + lane];
          pw = wp[a0 + lane];
          vw = wv[a0 + lane];
        }
        if (has_l) {
          const bool old = lane < rem;
          kl = old ? S.lk[cl + lane] : S.sk[lane - rem];
          pl = old ? S.lp[cl + lane] : S.sp[lane - rem];
          vl = old ? S.lv[cl + lane] : S.sv[lane - rem];
        }
        // the side list with the new entries sorted in (few: each is ranked in turn)
        if (fresh) {
          int in_l = lane < rem ? lane : 0;  // entries that beat the lane's
          for (int r = rem; r < nl; ++r) {
            const double rk = readlane_f64(kl, r);
            const uint32_t rp = (uint32_t)__builtin_amdgcn_readlane((int)pl, r);
            const uint32_t rv = (uint32_t)__builtin_amdgcn_readlane((int)vl, r);
            const bool by = has_l && better_e(rk, rp, rv, kl, pl, vl);
            const int above = __popcll(__ballot(lane < rem && !by));  // old ones that beat it
            in_l += by ? 1 : 0;
            if (lane == r) in_l += above;
          }
          if (has_l) {
            S.lk[in_l] = kl;
            S.lp[in_l] = pl;
            S.lv[in_l] = vl;
            kl = S.lk[lane];  // the lane's entry, best first
            pl = S.lp[lane];
            vl = S.lv[lane];
          }
        } else if (has_l && cl) {
          S.lk[lane] = kl;
          S.lp[lane] = pl;
          S.lv[lane] = vl;
        }
        // ranks: how many side-list entries beat the lane's window entry, and
        // the other way round
        const int nw = __popcll(__ballot(has_w));
        int lo_w = 0, up_w = has_w ? nl : 0, lo_l = 0, up_l = has_l ? (nw < bcap ? nw : bcap) : 0;
        while (__ballot(lo_w < up_w || lo_l < up_l)) {
          const int mw = (lo_w + up_w) >> 1, ml = (lo_l + up_l) >> 1;
          const int iw = mw < kSide ? mw : 0, il = a0 + (ml < nw ? ml : 0);
          const bool bl = better_e(S.lk[iw], S.lp[iw], S.lv[iw], kw, pw, vw);
          const bool bw = better_e(wk[il], wp[il], wv[il], kl, pl, vl);
          if (lo_w < up_w) {
            if (bl) lo_w = mw + 1; else up_w = mw;
          }
          if (lo_l < up_l) {
            if (bw) lo_l = ml + 1; else up_l = ml;
          }
        }
        rank_w = has_w ? lane + lo_w : kMaxMembers;
        rank_l = has_l ? lane + lo_l : kMaxMembers;
        const int avail = nw + nl;
        const int B = avail < bcap ? avail : bcap;
        const int m0 = set * kMaxMembers;
        if (rank_w < B) {
          S.mk[m0 + rank_w] = kw;
          S.mp[m0 + rank_w] = pw;
          S.mv[m0 + rank_w] = vw;
        }
        if (rank_l < B) {
          S.mk[m0 + rank_l] = kl;
          S.mp[m0 + rank_l] = pl;
          S.mv[m0 + rank_l] = vl;
        }
        consumed = 0;
        if (lane == 0) {
          sh.B = B;
          sh.pe = B;
          sh.nl_next = nl;
          sh.ncold += sh.napp;
          sh.napp = 0;
          sh.pause = (flips > flips0 && past(deadline)) ? 1 : 0;
        }
      }
      __syncthreads();
      // nothing to take, or the pool's room for a batch's entries runs out
      const bool dry = sh.B == 0;
      if (refilled || !(dry || sh.ncold + kMaxPairs + kWin > I->ccap)) {
        none = dry;
        break;
      }
      if (sh.ncold == 0 && dry) {
        none = true;
        break;
      }
      // the side list joins the window, then the pool's best refill it
      const int nl1 = sh.nl_next;
      if (nl1 > 0) {
        if (chooser) {
          if (lane < nl1) {
            S.sk[lane] = S.lk[lane];
            S.sp[lane] = S.lp[lane];
            S.sv[lane] = S.lv[lane];
          }
          if (lane == 0) sh.a0 = a0;
        }
        __syncthreads();
        call_join(I, (ASI_LDS SpecShared*)&sh, nl1);
      } else {
        if (tid == 0) sh.a0 = a0;
        __syncthreads();
      }
      call_refill(I, (ASI_LDS SpecShared*)&sh);
      if (chooser) {
        a0 = sh.a0;
        nl = 0;
        rank_w = rank_l = kMaxMembers;
        s_end = safe_end_wave(S, sh);
        if (lane == 0) sh.ns = 0;
      }
      refilled = true;
    }
    if (none) break;  // the pool held stale entries only, or nothing
    if (sh.pause) {  // flippable magnets remain
      status = 1;
      break;
    }
    const int B = sh.B;
    const double* const mk = S.mk + set * kMaxMembers;
    const uint32_t* const mp = S.mp + set * kMaxMembers;
    const uint32_t* const mv = S.mv + set * kMaxMembers;
    // ---- round trip 1: the members' versions and rows; round trip 2: the
    // neighbours' state, in flight while the conflicts are found
    bool on = sm < B;
    int pi = -1, si = 0;
    double2 ab = make_double2(0.0, 0.0), hi = ab, di = ab;
    double hki = 0.0;
    uint32_t vi = 0;
    if (on) {
      const uint32_t j = mp[sm] & 0x7fffffffu;
      if (sk == D) {
        pi = (int)j;
      } else {
        const int64_t sl = (int64_t)j * D + sk;
        pi = I->rcol[sl];
        ab = I->rAB[sl];
      }
    }
    if (tid < B) S.mval[tid] = (I->ver[mp[tid] & 0x7fffffffu] == mv[tid]) ? 1 : 0;
    if (tid == 0) {
      sh.npow = 0;
      sh.ns = 0;
      sh.nl = nl;
    }
    fold();
    on = on && pi >= 0;  // else a padding slot
    if (on && sk < D) {
      hi = I->h[pi];
      hki = I->hk[pi];
      si = I->s[pi];
      vi = I->ver[pi];
      if (mode == kFieldCarry) di = I->hd[pi];
    }
    __syncthreads();
    // members whose entries are current, by lane
    const unsigned long long valid = __ballot(lane < B && S.mval[lane < B ? lane : 0] != 0);
    // ---- pairwise disjoint neighbour sets: of the members that meet at a
    // magnet all but the first end the prefix
    int hs = -1;
    on = on && ((valid >> sm) & 1ull) != 0ull;
    if (on) {
      const uint32_t want = (uint32_t)pi + 1u;
      uint32_t q = hash_slot((uint32_t)pi);
      while (true) {
        const uint32_t old = atomicCAS(&S.hidx[q], 0u, want);
        if (old == 0u || old == want) break;
        q = (q + 1) & (kHash - 1);
      }
      hs = (int)q;
      const int first = atomicMin(&S.hown[q], sm);
      if (first != kNoOwner) atomicMin(&sh.pe, first > sm ? first : sm);
    }
    // ---- the neighbours' new fields.  Keys the switching bound cannot settle
    // go through a dense list in LDS, so that the FP64 powers run on full
    // wavefronts.
    double nh_p = 0.0, nh_q = 0.0, nd_p = 0.0, nd_q = 0.0, nkey = 0.0;
    int ppos = -1;
    double* pw_a = S.sk;            // kMaxPairs doubles
    double* pw_q = (double*)S.sp;   // kMaxPairs doubles (sp and sv)
    const bool nb = on && sk < D;  // the slot holds a neighbour
    {
      bool need = false;
      double pa = 0.0, pq = 0.0;
      if (nb) {
        const double two = (mp[sm] & 0x80000000u) ? 2.0 : -2.0;  // s_new = -s_old
        const double da = two * ab.x, db = two * ab.y;
        nh_p = hi.x + da;
        nh_q = hi.y + db;
        nd_p = di.x + da;
        nd_q = di.y + db;
        need = key_needs_powers(si, nh_p, nh_q, hki, pb, pc, ep, eq, pa, pq);
      }
      const unsigned long long bal = __ballot(need);
      if (bal) {
        int base = 0;
        if (lane == 0) base = atomicAdd(&sh.npow, __popcll(bal));
        base = __builtin_amdgcn_readfirstlane(base);
        if (need) {
          ppos = base + __popcll(bal & ((1ull << lane) - 1ull));
          pw_a[ppos] = pa;
          pw_q[ppos] = pq;
        }
      }
    }
    __syncthreads();
    const int p_ab = sh.pe;
    const int npow = sh.npow;
    // one power per lane: the even lane's term and the odd lane's, added
    for (int e = tid; e < 2 * npow; e += NT) {
      const bool odd = (e & 1) != 0;
      const double x = odd ? pw_q[e >> 1] : pw_a[e >> 1];
      const double r = pow_far(x, odd ? eq : ep);
      const double L = r + dpp_f64<0xB1>(r);  // quad_perm [1,0,3,2]
      if (!odd) pw_a[e >> 1] = (L > 1.0) ? L : 0.0;
    }
    __syncthreads();
    // ---- a new key that beats a later member of the prefix ends it there
    if (ppos >= 0 && sm < p_ab) {
      nkey = pw_a[ppos];
      if (nkey > 0.0) {
        const uint32_t npay = (uint32_t)pi | (si < 0 ? 0x80000000u : 0u);
        int lo = sm + 1, up = p_ab;
        while (lo < up) {
          const int mid = (lo + up) >> 1;
          if (better(nkey, npay, mk[mid], mp[mid])) up = mid; else lo = mid + 1;
        }
        if (lo < p_ab) atomicMin(&sh.pe, lo);
      }
    }
    __syncthreads();
    int pe = sh.pe;
    committed = pe < 64 ? valid & ((1ull << pe) - 1ull) : valid;
    int p = __popcll(committed);
    const int64_t left = max_flips - flips;
    if (p > left) {  // the flip cap: the prefix's first `left` members
      while (p > left) {
        pe = 63 - __clzll(committed);
        committed &= ~(1ull << pe);
        --p;
      }
    }
    if (p <= 0 && valid != 0ull) {
      status = -5;
      break;
    }
    // ---- commit the prefix's members and their neighbours
    if (tid < 64 && ((committed >> tid) & 1ull)) {
      const uint32_t mpay = mp[tid];
      const uint32_t j = mpay & 0x7fffffffu;
      I->s[j] = (mpay & 0x80000000u) ? (int8_t)1 : (int8_t)-1;
      I->key[j] = 0.0;
      I->ver[j] = mv[tid] + 1u;
    }
    if (clerk && ((committed >> lane) & 1ull)) {  // log the members in order
      const int64_t q = logpos + __popcll(committed & ((1ull << lane) - 1ull));
      if (q < I->log_cap) {
        I->log_t[q] = (int32_t)t;
        I->log_j[q] = (int32_t)(mp[lane] & 0x7fffffffu);
      }
    }
    const double cmk = sh.cmk;
    const uint32_t cmp = sh.cmp, cmv = sh.cmv;
    const int cb = sh.cb;
    const int64_t ncold = sh.ncold;
    // flippable touched magnets go to staging (if they beat the pool) or to
    // the pool, with one LDS atomic per wavefront for each
    const unsigned long long lt = (1ull << lane) - 1ull;
    bool st = false, co = false;
    uint32_t npay = 0, v1 = 0;
    if (hs >= 0) {  // the conflict table is left empty
      S.hidx[hs] = 0u;
      S.hown[hs] = kNoOwner;
    }
    if (nb && sm < pe) {
      I->h[pi] = make_double2(nh_p, nh_q);
      if (mode == kFieldCarry) {
        I->hd[pi] = make_double2(nd_p, nd_q);
      } else if (mode == kFieldDirty) {
        I->dirty[pi] = 1;
      }
      I->key[pi] = nkey;
      v1 = vi + 1u;
      I->ver[pi] = v1;
      if (nkey > 0.0) {
        npay = (uint32_t)pi | (si < 0 ? 0x80000000u : 0u);
        st = better_e(nkey, npay, v1, cmk, cmp, cmv);
        co = !st;
      }
    }
    const unsigned long long bs = __ballot(st), bc = __ballot(co);
    int sbase = 0, cbase = 0;
    if (lane == 0) {
      if (bs) sbase = atomicAdd(&sh.ns, __popcll(bs));
      if (bc) cbase = (int)atomicAdd((unsigned long long*)&sh.napp, (unsigned long long)__popcll(bc));
    }
    sbase = __builtin_amdgcn_readfirstlane(sbase);
    cbase = __builtin_amdgcn_readfirstlane(cbase);
    if (st) {
      const int q = sbase + __popcll(bs & lt);
      S.sk[q] = nkey;
      S.sp[q] = npay;
      S.sv[q] = v1;
    }
    if (co) {
      const int64_t q = ncold + cbase + __popcll(bc & lt);
      I->ckey[cb][q] = nkey;
      I->cpay[cb][q] = npay;
      I->cver[cb][q] = v1;
    }
    logpos += p;
    flips += p;
    ++nbatch;
    bcap = (p >= B) ? 2 * B : 2 * p + 2;
    if (bcap < 8) bcap = 8;
    if (bcap > Bmax) bcap = Bmax;
    // entries done with: the prefix's (stale ones among them), or the whole
    // batch when every valid member went
    consumed = (pe >= 64 || (valid >> pe) == 0ull) ? B : pe;
    set ^= 1;
    if (nbatch >= nswitch && (double)(flips - flips0) < sw * nbatch) status = 2;
    __syncthreads();
    if (status == 2) break;
  }
  if (status != -5) fold();  // (there nothing was committed since the last fold)
  if (tid == NT - 64) sh.hash = hash;
  __syncthreads();
  hash = sh.hash;
  return status;
}

// Relax one instance at step t with the whole workgroup (Sec. II.H).  The
// flippable keys are kept in a three-level max tree: the key array in
// memory, first-level tiles of 2^l1_shift magnets and second-level groups of
// 64 tiles in LDS, built from the per-64-row maxima of the field phase
// (with kFlatOk, up to kFlatTiles tiles the root reads the tiles directly).
// Per flip: the root gives j; thread 0 flips it and logs it; the threads
// update j's neighbours (dipolar and total field += 2 s_new * coupling, new
// key); the touched tiles are brought up to date from the updates, or
// rescanned when their maximum fell, and then the touched groups.  Returns
// 0, -5 (flip cap reached with a flippable magnet left) or 1 (deadline
// passed, checked every 16 flips, with flippable magnets left).
template <bool kFlatOk>
__device__ __forceinline__ int relax_tree(const InstDev* __restrict__ I, int64_t t, unsigned char* lds_raw,
                          RelaxShared& sh, int64_t& flips, int64_t& logpos, uint64_t& hash,
                          uint64_t deadline) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int NT = blockDim.x, NW = NT >> 6;
  const int64_t n = I->n;
  const int l1s = I->l1_shift;
  const int nt1 = (int)((n + (1LL << l1s) - 1) >> l1s);
  const int nt2 = (nt1 + kL2Group - 1) / kL2Group;
  const int64_t nt0 = (n + 63) >> 6;
  const int per0 = 1 << (l1s - 6);  // per-64-row maxima in one tile
  const int seg = 1 << (l1s - 6);   // magnets per lane in a tile rescan
  RelaxLds L = carve(lds_raw, nt1, nt2);

  const int32_t D = I->D;
  const int32_t* __restrict__ colp = I->rcol;
  typedef double f64x2 __attribute__((ext_vector_type(2)));
  const f64x2* __restrict__ ABp = (const f64x2*)(const double2*)I->rAB;
  const double* __restrict__ hkp = I->hk;
  int8_t* __restrict__ sp = I->s;
  double2* __restrict__ hp2 = I->h;
  double2* __restrict__ hd2 = I->hd;
  double* __restrict__ keyp = I->key;
  uint8_t* __restrict__ dirtyp = I->dirty;
  const int32_t mode = I->field_mode;
  const double pb = I->b, pc = I->c, ep = I->e_par, eq = I->e_perp;
  const int64_t max_flips = I->max_flips;

  // first level from the per-64-row maxima of the field phase (loads in
  // groups of 8, issued together)
  for (int e = tid; e < nt1; e += NT) {
    double bk = 0.0;
    uint32_t bi = 0;
    for (int u0 = 0; u0 < per0; u0 += 8) {
      double kk[8];
      uint32_t ki[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t f = (int64_t)e * per0 + u0 + u;
        const bool ok = u0 + u < per0 && f < nt0;
        kk[u] = ok ? I->t1key[f] : 0.0;
        ki[u] = ok ? I->t1idx[f] : 0u;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (kk[u] > bk) {
          bk = kk[u];
          bi = ki[u];
        }
      }
    }
    L.l1k[e] = bk;
    L.l1i[e] = bi;
    L.l1flag[e] = 0;
    L.l1nk[e] = 0ull;
    L.l1ni[e] = ~0ull;
    L.l1resc[e] = 0;
  }
  if (tid == 0) {
    sh.nr = 0;
    sh.pfk = 0ull;
    sh.ruk = 0ull;
  }
  __syncthreads();
  for (int g = wave; g < nt2; g += NW) {
    const int e = g * kL2Group + lane;
    double k = (e < nt1) ? L.l1k[e] : 0.0;
    uint32_t pay = (e < nt1) ? L.l1i[e] : 0u;
    wave_argmax(k, pay);
    if (lane == 0) {
      L.l2k[g] = k;
      L.l2i[g] = pay;
      L.l2flag[g] = 0;
    }
  }
  __syncthreads();

  int status = 0;
  const int per2 = (nt2 + 63) >> 6;
  const int64_t flips0 = flips;
  // Row of the predicted next flip (the best magnet the last update pushed
  // over the astroid, the usual next flip of an avalanche), loaded while the
  // tree is brought up to date; used when the prediction holds.  The pair of a
  // slot stays in the registers that it is loaded into: taken apart, it was
  // waited for at once (45,300-magnet pinwheel reversal at 632 neighbours 357 ms,
  // 337 so).
  int64_t pf_j = -1;
  constexpr int kAhead = kFlatOk ? 2 : 1;  // slots a thread (as many as the registers allow)
  int32_t pf_c[kAhead];
  f64x2 pf_ab[kAhead];
#pragma unroll
  for (int h = 0; h < kAhead; ++h) {
    pf_c[h] = -1;
    pf_ab[h] = f64x2{0.0, 0.0};
  }

  // Up to kFlatTiles tiles the root reads the first level directly (at most
  // eight ascending tiles per lane) and the second level is not kept; only
  // in the tree-only kernel, whose registers allow it.
  const bool flat = kFlatOk && nt1 <= kFlatTiles;
  const int per1 = (nt1 + 63) >> 6;
  // tid, where registers are short as a value of this flip: addresses formed
  // from it are formed again, which is cheaper than their way to memory and back
  auto own = [&]() {
    int v = tid;
    if (!kFlatOk) asm volatile("" : "+v"(v));
    return v;
  };

  while (true) {
    if (wave == 0) {
      double bk = 0.0;
      uint32_t bp = 0;
      if (flat) {
        // the lane's tiles four at a time, each group's reads issued together
        for (int u0 = 0; u0 < per1; u0 += 4) {
          double kk[4];
          uint32_t ii[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int e = lane * per1 + u0 + u;
            const int ec = (u0 + u < per1 && e < nt1) ? e : 0;
            kk[u] = L.l1k[ec];
            ii[u] = L.l1i[ec];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int e = lane * per1 + u0 + u;
            if (u0 + u < per1 && e < nt1 && kk[u] > bk) {
              bk = kk[u];
              bp = ii[u];
            }
          }
        }
      } else {
        // second level of the groups the last flip touched (their flags; at
        // most kMaxL1Tiles / kL2Group = 32 groups, one per lane), then the root
        const bool gf = lane < nt2 && L.l2flag[lane] != 0;
        unsigned long long gbal = __ballot(gf);
        if (gf) L.l2flag[lane] = 0;
        while (gbal) {
          const int g = __ffsll(gbal) - 1;
          gbal &= gbal - 1ull;
          const int e = g * kL2Group + lane;
          double k = (e < nt1) ? L.l1k[e] : 0.0;
          uint32_t p2 = (e < nt1) ? L.l1i[e] : 0u;
          wave_argmax(k, p2);
          if (lane == 0) {
            L.l2k[g] = k;
            L.l2i[g] = p2;
          }
        }
        for (int u = 0; u < per2; ++u) {
          const int g = lane * per2 + u;
          if (g < nt2) {
            const double k = L.l2k[g];
            if (k > bk) {
              bk = k;
              bp = L.l2i[g];
            }
          }
        }
      }
      wave_argmax(bk, bp);
      if (lane == 0) {
        sh.key = bk;
        sh.pay = bp;
        sh.pause = (flips > flips0 && ((flips - flips0) & 15) == 0 && past(deadline)) ? 1 : 0;
      }
    }
    __syncthreads();
    const double top = sh.key;
    const uint32_t pay = sh.pay;
    if (!(top > 0.0)) break;
    if (sh.pause) {
      status = 1;
      break;
    }
    if (flips >= max_flips) {
      status = -5;
      break;
    }
    const int64_t j = pay & 0x7fffffffu;
    const int s_new = (pay & 0x80000000u) ? 1 : -1;
    if (tid == 0) {
      const uint64_t w = ((uint64_t)(uint32_t)t << 32) | (uint64_t)(uint32_t)j;
      hash = (hash ^ w) * 0x100000001b3ull;
      const int e = (int)(j >> l1s);
      L.l1resc[e] = 1;  // j was its tile's maximum
      L.l1flag[e] = 1;
    }
    ++logpos;
    ++flips;
    const double two = (s_new > 0) ? 2.0 : -2.0;
    // Update the neighbours.  A touched tile whose maximum was not among the
    // updated magnets, or kept at least its key, keeps that maximum unless an
    // update beats it, so it needs no rescan: the largest new key of the tile is found with LDS
    // atomics (positive doubles order like their bit patterns), then the
    // lowest index among the updates holding it.
    const bool incr = D <= 2 * NT;
    const bool hit = j == pf_j;
    // The predicted row's loads were issued before the last tile rescans,
    // whose loads the wavefront has waited for, so they are complete; using
    // the registers here makes that known, and no wait below is widened to
    // them.
#pragma unroll
    for (int h = 0; h < kAhead; ++h) asm volatile("" ::"v"(pf_c[h]), "v"(pf_ab[h]));
    int u_i[2], u_e[2], u_s[2];
    double u_k[2];
    double tb_k = 0.0;  // this thread's best updated key, for the prediction
    uint32_t tb_i = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) u_i[h] = -1;
    for (int k = own(), h = 0; k < D; k += NT, ++h) {
      const int64_t sl = j * D + k;
      const bool pre = hit && h < kAhead;
      // the slot's column and couplings together (a padding slot holds -1
      // and zeros), then every load of the neighbour's state before any
      // store, so that each costs one round trip
      const int32_t i = pre ? pf_c[h & (kAhead - 1)] : colp[sl];
      const f64x2 cab = pre ? pf_ab[h & (kAhead - 1)] : ABp[sl];
      const double ca = cab.x, cb = cab.y;
      if (i >= 0) {
        const double2 hi = hp2[i];
        const double2 di = (mode == kFieldCarry) ? hd2[i] : make_double2(0.0, 0.0);
        const int si = sp[i];
        const double hki = hkp[i];
        const double da = two * ca;
        const double db = two * cb;
        const double hp = hi.x + da;
        const double hq = hi.y + db;
        const double kk = switching_key(si, hp, hq, hki, pb, pc, ep, eq);
        if (mode == kFieldCarry) {
          hd2[i] = make_double2(di.x + da, di.y + db);
        } else if (mode == kFieldDirty) {
          dirtyp[i] = 1;
        }
        hp2[i] = make_double2(hp, hq);
        keyp[i] = kk;
        const int e = (int)(i >> l1s);
        const double ek = L.l1k[e];
        const uint32_t ei = L.l1i[e];
        L.l1flag[e] = 1;
        if (!incr || (ek > 0.0 && (ei & 0x7fffffffu) == (uint32_t)i && kk < ek)) L.l1resc[e] = 1;
        if (kk > 0.0) atomicMax(&L.l1nk[e], (unsigned long long)__double_as_longlong(kk));
        if (kk > tb_k) {
          tb_k = kk;
          tb_i = (uint32_t)i;
        }
        if (h < 2) {
          u_i[h] = i;
          u_e[h] = e;
          u_s[h] = si;
          u_k[h] = kk;
        }
      }
    }
    // Runner-up hint, by the last wavefront when it updates no neighbour:
    // the best magnet of the tree outside j's tile (the other groups' maxima,
    // then the other tiles of j's group), the usual next flip when no update
    // beats it.  Read while the tree is unchanged since the root.
    if (wave == NW - 1 && D <= (NW - 1) * 64) {
      const int ej = (int)(j >> l1s), gj = ej / kL2Group;
      double rk = 0.0;
      uint32_t rp = 0;
      if (flat) {
        for (int u = 0; u < per1; ++u) {
          const int e = lane * per1 + u;
          if (e < nt1 && e != ej && L.l1k[e] > rk) {
            rk = L.l1k[e];
            rp = L.l1i[e];
          }
        }
      } else {
        for (int u = 0; u < per2; ++u) {
          const int g = lane * per2 + u;
          if (g < nt2 && g != gj && L.l2k[g] > rk) {
            rk = L.l2k[g];
            rp = L.l2i[g];
          }
        }
        const int e = gj * kL2Group + lane;
        if (e < nt1 && e != ej && L.l1k[e] > rk) {
          rk = L.l1k[e];
          rp = L.l1i[e];
        }
      }
      wave_argmax(rk, rp);
      if (lane == 0)
        sh.ruk = rk > 0.0 ? (((unsigned long long)__double_as_longlong(rk) & 0xffffffff00000000ull) |
                             (unsigned long long)(rp & 0x7fffffffu))
                          : 0ull;
    }
    // the flipped magnet's own stores, issued after the neighbour loads so
    // that waiting for those loads does not wait for these
    if (tid == 0) {
      sp[j] = (int8_t)s_new;
      keyp[j] = 0.0;
      if (logpos - 1 < I->log_cap) {
        I->log_t[logpos - 1] = (int32_t)t;
        I->log_j[logpos - 1] = (int32_t)j;
      }
    }
    wave_argmax(tb_k, tb_i);
    if (lane == 0 && tb_k > 0.0)
      atomicMax(&sh.pfk, ((unsigned long long)__double_as_longlong(tb_k) & 0xffffffff00000000ull) |
                             (unsigned long long)tb_i);
    __syncthreads();
    {
      // the next flip is probably the better of the best updated neighbour
      // and the runner-up (compared on the keys' high bits)
      const unsigned long long pk = sh.pfk > sh.ruk ? sh.pfk : sh.ruk;
      pf_j = pk ? (int64_t)(pk & 0xffffffffull) : -1;
      if (pf_j >= 0) {
#pragma unroll
        for (int h = 0; h < kAhead; ++h) {
          const int k = tid + h * NT;
          if (k < D) {
            const int64_t sl = pf_j * D + k;
            pf_c[h] = colp[sl];
            pf_ab[h] = ABp[sl];
          }
        }
      }
    }
    if (incr) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (u_i[h] >= 0 && u_k[h] > 0.0 &&
            (unsigned long long)__double_as_longlong(u_k[h]) == L.l1nk[u_e[h]])
          atomicMin(&L.l1ni[u_e[h]], ((unsigned long long)u_i[h] << 1) | (u_s[h] < 0 ? 1ull : 0ull));
      }
    }
    __syncthreads();
    if (tid == 0) sh.pfk = 0ull;  // every thread has read it
    // touched tiles: a scan of the flags (nt1 <= kMaxL1Tiles), each tile's
    // state read at once
    for (int e = own(); e < nt1; e += NT) {
      if (!L.l1flag[e]) continue;
      if (L.l1resc[e]) {
        L.l1rlist[atomicAdd(&sh.nr, 1)] = e;
      } else {
        const unsigned long long nkb = L.l1nk[e];
        if (nkb != 0ull) {
          const double nk = __longlong_as_double((long long)nkb);
          const unsigned long long ni = L.l1ni[e];
          const uint32_t np = (uint32_t)(ni >> 1) | ((ni & 1ull) ? 0x80000000u : 0u);
          if (!(L.l1k[e] > 0.0) || better(nk, np, L.l1k[e], L.l1i[e])) {
            L.l1k[e] = nk;
            L.l1i[e] = np;
          }
        }
        L.l1flag[e] = 0;
        L.l2flag[e / kL2Group] = 1;
      }
      L.l1nk[e] = 0ull;
      L.l1ni[e] = ~0ull;
    }
    __syncthreads();
    const int nr = sh.nr;
    for (int u = wave; u < nr; u += NW) {
      const int e = L.l1rlist[u];
      const int64_t r0 = ((int64_t)e << l1s) + (int64_t)lane * seg;
      double bk = 0.0;
      uint32_t bp = 0;
      // the lane's segment in groups of 8, each group's loads issued together
      // (whole groups inside the arrays: four 16-byte key loads and one
      // 8-byte spin load, the group starting on a 64-byte boundary)
      for (int m0 = 0; m0 < seg; m0 += 8) {
        double kk[8];
        int ss[8];
        if (seg >= 8 && r0 + m0 + 8 <= n) {
          const double2* k2 = reinterpret_cast<const double2*>(keyp + r0 + m0);
          const uint64_t s8 = *reinterpret_cast<const uint64_t*>(sp + r0 + m0);
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            const double2 v = k2[m];
            kk[2 * m] = v.x;
            kk[2 * m + 1] = v.y;
          }
#pragma unroll
          for (int m = 0; m < 8; ++m) ss[m] = (int)(int8_t)(uint8_t)(s8 >> (8 * m));
        } else {
          // short segment or the array's end: every load issued at once, an
          // index past the segment replaced by magnet 0 and its key dropped
#pragma unroll
          for (int m = 0; m < 8; ++m) {
            const int64_t ii = r0 + m0 + m;
            const int64_t ic = (m0 + m < seg && ii < n) ? ii : 0;
            kk[m] = keyp[ic];
            ss[m] = sp[ic];
          }
#pragma unroll
          for (int m = 0; m < 8; ++m) {
            if (!(m0 + m < seg && r0 + m0 + m < n)) {
              kk[m] = 0.0;
              ss[m] = 0;
            }
          }
        }
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          if (kk[m] > bk) {
            bk = kk[m];
            bp = (uint32_t)(r0 + m0 + m) | (ss[m] < 0 ? 0x80000000u : 0u);
          }
        }
      }
      wave_argmax(bk, bp);
      if (lane == 0) {
        L.l1k[e] = bk;
        L.l1i[e] = bp;
        L.l1flag[e] = 0;
        L.l1resc[e] = 0;
        L.l2flag[e / kL2Group] = 1;
      }
    }
    __syncthreads();
    if (tid == 0) sh.nr = 0;
  }
  return status;
}

// Per-64-row maxima of the stored keys -- the lowest level of the relax
// tree -- rebuilt by the whole workgroup, four 64-row groups per wavefront
// at a time (their loads issued together).
__device__ __forceinline__ void rebuild_t1(const InstDev* __restrict__ I) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, NW = blockDim.x >> 6;
  const int64_t n = I->n, ng = (n + 63) >> 6;
  for (int64_t g0 = (int64_t)wave * 4; g0 < ng; g0 += (int64_t)NW * 4) {
    double k[4];
    uint32_t p[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = ((g0 + u) << 6) + lane;
      k[u] = 0.0;
      p[u] = 0u;
      if (g0 + u < ng && i < n) {
        k[u] = I->key[i];
        p[u] = (uint32_t)i | (I->s[i] < 0 ? 0x80000000u : 0u);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      wave_argmax(k[u], p[u]);
      if (lane == 0 && g0 + u < ng) {
        I->t1key[g0 + u] = k[u];
        I->t1idx[g0 + u] = p[u];
      }
    }
  }
  __syncthreads();
}

// ------------------------------------------------------------ relax, keys in LDS
// One-at-a-time relax for instances whose keys fit in LDS (kLdsMaxN magnets):
// the code of every magnet, a spin bit per magnet, and per wavefront the best
// code of the magnets its threads own.
// A thread owns one tile of consecutive magnets: an odd multiple of 4 of them
// (so that the 16-byte reads of neighbouring threads' tiles meet different LDS
// banks), as few as cover the instance.
__host__ __device__ inline int flip_tile(int64_t n, int threads) {
  const int chunks = (int)((n + 4 * threads - 1) / (4 * threads));
  return 4 * (chunks | 1);
}

__host__ __device__ inline size_t flip_lds_bytes(int64_t n, int threads) {
  const int per = flip_tile(n, threads);
  const size_t tiles = (size_t)((n + per - 1) / per);
  return tiles * per * 4 + align16((size_t)((n + 31) / 32) * 4) + (size_t)threads * 4;
}

struct FlipShared {
  uint2 best[kMaxRelaxWaves];  // per wavefront: code, its tile << 8 | codes near it
  double rk[kMaxRelaxWaves];   // resolving a near-tie: per wavefront exact key and index
  uint32_t ri[kMaxRelaxWaves]; //   (index << 1 | sign bit; bit 31: an unknown key became known)
  int pause;
};

// A global load at a 32-bit byte offset from a uniform base.
template <class T>
__device__ __forceinline__ T load_at(const ASI_GLOBAL T* base, uint32_t bytes) {
  return *(const ASI_GLOBAL T*)((const ASI_GLOBAL char*)base + bytes);
}
template <class T>
__device__ __forceinline__ void store_at(ASI_GLOBAL T* base, uint32_t bytes, T v) {
  *(ASI_GLOBAL T*)((ASI_GLOBAL char*)base + bytes) = v;
}

// A launch's parts that are not its hot loop are called out of line, so that
// each part's registers are allocated for itself: inlined into one kernel, the
// relax with keys in LDS took 2.6 us a flip instead of 2.1.
// What a relax reads and advances, in LDS while it is called out of line.
struct RelaxCount {
  int64_t flips, logpos;
  uint64_t hash;
};

// ------------------------------------------------------------ speculative relax, tiles
// Speculative batches without a sorted window, for up to kManyMaxN magnets and
// kManyMinD to kManyMaxD neighbours: of each tile of 64 (128) consecutive magnets
// LDS holds the largest key, its place and a bound of the second, and of each of
// 256 (512) rows of tiles the two largest keys.  The rows' bests that beat every row's second are
// the first magnets of the relax order.
constexpr int kManyMembers = 32;
constexpr int kManyHash = 2048;  // conflict table slots (at most 1,056 in use)
constexpr int kManyList = 1088;  // tiles that a batch changes (at most 1,056)
// Up to 2^19 magnets tiles of 64 in 256 rows, above tiles of 128 in 512 rows:
// half the tiles, and twice the rows for the more candidates of such sizes (20
// steps of a 1M-magnet kagome 17.3 ms against 18.0 with 256 rows; a
// 200,000-magnet square 1.91 us a flip with 256 rows against 2.06).
constexpr int kManyRows = 256, kManyRowsBig = 512;

template <int kRows>
struct ManyShared {
  double best[kRows], sec[kRows];  // per row: largest key, (at most) the second,
  uint32_t idx[kRows];                 //   the largest's magnet
  using Stale = std::conditional_t<kRows == 256, uint32_t, unsigned long long>;
  Stale stale[64];                         // a byte per row: a tile of it changed
  double ck[kRows];                    // candidates: key, magnet
  uint32_t ci[kRows];
  double mk[kManyMembers];                 // members, best first: key,
  uint32_t mi[2][kManyMembers];            //   magnet (two sets, by turns),
  unsigned long long vm[kManyMembers];     //   its neighbours' largest new key (bits)
  alignas(16) int pe, nt, nc, npow, pause;  // end of the prefix; changed tiles; candidates; keys to evaluate
};

template <int kRows>
__host__ __device__ constexpr int many_tile_shift() {
  return kRows == kManyRows ? 6 : 7;
}
template <int kRows>
__host__ __device__ inline int many_tiles(int64_t n) {  // rounded up to whole rows
  const int sh = many_tile_shift<kRows>();
  return (int)((((n + (1 << sh) - 1) >> sh) + 4 * kRows - 1) & ~(int64_t)(4 * kRows - 1));
}
template <int kRows>
__host__ __device__ inline size_t many_lds(int64_t n) {
  const size_t tiles = (size_t)many_tiles<kRows>(n);
  return sizeof(ManyShared<kRows>) + tiles * 13 + (size_t)1024 * 25 + kManyHash * 4 + tiles / 8 +
         kManyList * 2;
}
inline size_t many_lds_bytes(int64_t n) {
  return n <= kManyMaxN64 ? many_lds<kManyRows>(n) : many_lds<kManyRowsBig>(n);
}

union RelaxParts {
  RelaxShared tree;
  SpecShared spec;
  FlipShared flip;
};
struct RelaxState {
  RelaxCount c;
  RelaxParts u;
};

// Relax at step t, one flip at a time.  Each thread owns a tile of
// consecutive magnets and keeps its largest code in a register.  Per flip:
//   - the wavefronts' best codes give the winner, whose row is loaded.  If no
//     other code reaches its floor (code_floor), and it is surely above 1, it is
//     the magnet the exact keys would pick; else the exact FP64 keys of the
//     codes that near decide (keys of 0 are struck out, equal keys go to the
//     lower index); an exact key is kept in the key array until the magnet's
//     field changes;
//   - the threads update the neighbours' fields and codes;  [barrier]
//   - the owners of changed tiles rescan them in LDS and their wavefronts
//     renew their best.  [barrier]
// The last wavefront, which updates no neighbour below 960 of them, does the
// flip's bookkeeping.
// What bounds it: one dependent chain per flip -- the flipped magnet's row,
// then its neighbours' fields (two round trips to memory, ~1,100 of ~3,500
// cycles), two barriers, three LDS round trips, and the instructions between
// them, which issue one by one (about eight cycles each).  Against the max
// tree it leaves out of that chain the FP64 powers (~200 dependent
// instructions each; exact keys are evaluated for 1-8 % of the flips), the
// rescans of tiles in memory and three of five barriers: per flip 6.2 -> 1.5
// us on a 5,100-magnet anneal at 632 neighbours, 5.6 -> 1.9 on a
// 20,200-magnet reversal at 632, 5.1 -> 1.7 on a 29,040-magnet reversal at
// 60; with every key tied (no disorder) 5.1 -> 1.3.  Tried and slower: the
// runner-up's row loaded ahead (right for 20-80 % of the flips; its loads
// return before the neighbours' can), tiles dealt to the wavefronts in turn
// (more wavefronts rescan), a changed tile rescanned by half a wavefront.
// Returns as relax_tree.
template <bool kTile1>
__device__ __forceinline__ int relax_lds(const InstDev* __restrict__ I, int64_t t, unsigned char* lds_raw,
                                         RelaxState& st, int64_t ncand, bool from_pool,
                                         uint64_t deadline) {
  FlipShared& sh = st.u.flip;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int NT = blockDim.x;
  const bool clerk = tid == NT - 64;
  const int32_t n = (int32_t)I->n;
  const int NW = NT >> 6;
  const int per = kTile1 ? 4 : flip_tile(n, NT), nc = per >> 2;
  // tile of magnet i: i / per, exact for i < 2^16 and per <= 64
  const uint32_t per_inv = 0xffffffffu / (uint32_t)per + 1u;
  auto tile_of = [&](uint32_t i) { return __umulhi(i, per_inv); };
  const int32_t npad = (int32_t)((n + per - 1) / per) * per;
  uint32_t* const code = (uint32_t*)lds_raw;
  uint32_t* const spin = code + npad;  // bit per magnet: spin -1
  // per tile: a code of it changed
  uint32_t* const touched = (uint32_t*)((unsigned char*)spin + align16((size_t)((n + 31) / 32) * 4));

  const int32_t D = I->D;
  const int32_t mode = I->field_mode;
  const bool carry = mode == kFieldCarry;
  const KeyPar P = key_par(I);
  const int64_t left0 = I->max_flips - uniform(st.c.flips);  // flips this call may make
  const int64_t logpos = uniform(st.c.logpos);
  uint64_t hash = st.c.hash;
  int64_t done = 0;
  const ASI_GLOBAL int32_t* const rcol = I->rcol;
  const ASI_GLOBAL double2* const rAB = I->rAB;
  ASI_GLOBAL double2* const hh = I->h;
  ASI_GLOBAL double2* const hd = I->hd;
  const ASI_GLOBAL double* const ghk = I->ghk;

  for (int q = tid; q < npad / 4; q += NT) ((uint4*)code)[q] = make_uint4(0u, 0u, 0u, 0u);
  // sign bits of 32 spins per word, from four 8-byte loads (the array's
  // allocation is a multiple of 256 bytes)
  for (int q = tid; q < (n + 31) / 32; q += NT) {
    const ASI_GLOBAL uint64_t* s8 = (const ASI_GLOBAL uint64_t*)I->s + 4 * (int64_t)q;
    uint64_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = (8 * (4 * q + u) < n) ? s8[u] : 0ull;
    uint32_t w = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      w |= (uint32_t)((((v[u] >> 7) & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56) << (8 * u);
    spin[q] = w;
  }
  touched[tid] = 0u;
  if (tid < kMaxRelaxWaves) sh.best[tid] = make_uint2(0u, 0u);
  if (tid == 0) sh.pause = 0;
  __syncthreads();
  auto put = [&](uint32_t i, double key, bool neg) {  // the key array holds this key
    const uint32_t tl = tile_of(i);
    code[i] = code_of_key(key, neg) | kCodeExact | (i - tl * (uint32_t)per);
    touched[tl] = 1u;
  };
  if (from_pool) {  // the field phase's list of flippable magnets
    for (int64_t q = tid; q < ncand; q += NT) {
      const uint32_t pay = I->cpay[0][q];
      put(pay & 0x7fffffffu, I->ckey[0][q], (pay >> 31) != 0u);
    }
  } else {  // the key array, which the speculative relax keeps exact
    for (int32_t i = tid; i < n; i += NT) {
      const double key = load_at(I->key, (uint32_t)i * 8u);
      if (key > 0.0) put((uint32_t)i, key, load_at(I->s, (uint32_t)i) < 0);
    }
  }
  __syncthreads();

  // The thread's slot of a flip: slot tid of the flipped magnet's row (a
  // padding slot holds column -1 and zeros) and the neighbour's state.
  struct Slot {
    int32_t i0;
    double2 ab, h, d;
    double g;
  };
  auto load_row = [&](int32_t j, int k, int32_t& i0, double2& ab) {
    const uint32_t e = (uint32_t)j * (uint32_t)D + (uint32_t)k;  // n * D * 16 < 2^32
    i0 = load_at(rcol, e * 4u);
    ab = load_at(rAB, e * 16u);
  };
  auto load_state = [&](Slot& q) {
    const uint32_t i = (uint32_t)max(q.i0, 0);
    q.h = load_at(hh, i * 16u);
    q.g = load_at(ghk, i * 8u);
    if (carry) q.d = load_at(hd, i * 16u);
  };
  // The neighbour's new field and code; the carried sum, which nothing waits
  // for, last.
  auto change = [&](const Slot& q, double two) {
    const uint32_t i = (uint32_t)max(q.i0, 0);
    const bool neg = (spin[i >> 5] >> (i & 31u)) & 1u;
    const double da = two * q.ab.x, db = two * q.ab.y;
    const double hp = q.h.x + da, hq = q.h.y + db;
    const uint32_t v = key_code(neg, hp, hq, q.g, P);
    if (q.i0 >= 0) {
      const uint32_t tl = tile_of(i);
      code[i] = v ? v | (i - tl * (uint32_t)per) : 0u;
      if (!kTile1) touched[tl] = 1u;
      store_at(hh, i * 16u, make_double2(hp, hq));
      if (carry)
        store_at(hd, i * 16u, make_double2(q.d.x + da, q.d.y + db));
      else if (mode == kFieldDirty)
        store_at(I->dirty, i, (uint8_t)1);
    }
  };

  // Flip j (down: its spin is -1), its row's slots of this thread loaded in q.
  int32_t j = -1;  // last flipped magnet (its spin bit toggled by the clerk later)
  auto flip = [&](Slot& q, bool down) {
    const double two = down ? 2.0 : -2.0;  // 2 s_new
    if (tid < D) change(q, two);
    for (int k = tid + NT; k < D; k += NT) {
      load_row(j, k, q.i0, q.ab);
      load_state(q);
      change(q, two);
    }
    if (clerk) {
      code[j] = 0u;
      if (!kTile1) touched[tile_of((uint32_t)j)] = 1u;
      store_at(I->s, (uint32_t)j, down ? (int8_t)1 : (int8_t)-1);
      if (logpos + done < I->log_cap) {
        I->log_t[logpos + done] = (int32_t)t;
        I->log_j[logpos + done] = j;
      }
      hash = (hash ^ (((uint64_t)(uint32_t)t << 32) | (uint64_t)(uint32_t)j)) * 0x100000001b3ull;
    }
    ++done;
    __syncthreads();
  };

  uint32_t* const tile = code + tid * per;
  uint32_t mx = 0;  // largest code of the thread's tile
  int status = 0;
  bool stop = false;
  while (true) {
    uint32_t Mv;  // the largest code
    while (true) {
      // owners of changed tiles (tiles of four codes: every owner, which is
      // cheaper than flags)
      const bool mine = kTile1 ? tid < npad / 4 : touched[tid] != 0u;
      if (__ballot(mine)) {
        uint32_t near_mx = 0;  // tiles of four: codes near the largest
        if (mine) {
          const uint4* const c4 = (const uint4*)tile;
          if (kTile1) {
            const uint4 c = c4[0];
            mx = max(max(c.x, c.y), max(c.z, c.w));
            const uint32_t T = code_floor(mx);
            near_mx = (c.x >= T) + (c.y >= T) + (c.z >= T) + (c.w >= T);
          } else {
            touched[tid] = 0u;
            mx = 0;
            for (int u0 = 0; u0 < nc; u0 += 5) {
              // five 16-byte reads at a time, the last one again past the end
              uint4 c[5];
#pragma unroll
              for (int u = 0; u < 5; ++u) c[u] = c4[min(u0 + u, nc - 1)];
#pragma unroll
              for (int u = 0; u < 5; ++u) mx = max(mx, max(max(c[u].x, c[u].y), max(c[u].z, c[u].w)));
            }
          }
        }
        // the wavefront's best; codes near it: one per lane, and the others of
        // the best lane's tile
        const uint32_t m = wave_max_u32(mx);
        const uint32_t T = code_floor(m);
        uint32_t cnt = (uint32_t)__popcll(__ballot(mx >= T)) - 1u;
        if (kTile1) {
          cnt += near_mx;
        } else {
          const int wl = __ffsll((unsigned long long)__ballot(mx == m)) - 1;
          const uint32_t v = lane < per ? code[(wave * 64 + wl) * per + lane] : 0u;
          cnt += (uint32_t)__popcll(__ballot(v >= T));
        }
        if (mx == m) sh.best[wave] = make_uint2(m, (uint32_t)tid << 8 | (cnt & 255u));
      }
      if (clerk) {
        if (j >= 0) atomicXor(&spin[j >> 5], 1u << (j & 31));
        if (deadline) sh.pause = (done > 0 && (done & 15) == 0 && past(deadline)) ? 1 : 0;
      }
      __syncthreads();
      const uint2 e = sh.best[lane & 15];
      Mv = row_max_u32(e.x);
      // the wavefronts whose best is near the largest: normally one
      const uint32_t near = (uint32_t)__ballot(e.x >= code_floor(Mv)) & 0xffffu;
      const int w = __ffs(near) - 1;
      const uint32_t M = (uint32_t)__builtin_amdgcn_readlane((int)e.x, w);
      const uint32_t meta = (uint32_t)__builtin_amdgcn_readlane((int)e.y, w);
      j = (int32_t)(meta >> 8) * per + (int32_t)(M & kCodePlace);
      // near ties, a key that may be below 1, and the end (no code: near == 0)
      if ((near & (near - 1u)) != 0u || near == 0u || (meta & 255u) != 1u || M < kCodeSure ||
          M >= kCodeUnknown)
        break;
      Slot q;
      if (tid < D) {
        load_row(j, tid, q.i0, q.ab);
        load_state(q);
      }
      stop = done >= left0 || (deadline && sh.pause);
      if (stop) break;
      flip(q, (M & kCodeDown) != 0u);
    }
    Mv = (uint32_t)__builtin_amdgcn_readfirstlane((int)Mv);
    if (stop || Mv == 0u) break;
    // exact keys of the codes near the largest
    const uint32_t T = code_floor(Mv);
    double bk = 0.0;
    uint32_t bp = 0x7fffffffu;  // index | sign bit
    bool unknown = false;
    if (mx >= T) {
      uint64_t at = 0;  // their places in the tile
      for (int u = 0; u < nc; ++u) {
        const uint4 c = ((const uint4*)tile)[u];
        at |= (uint64_t)((c.x >= T ? 1u : 0u) | (c.y >= T ? 2u : 0u) | (c.z >= T ? 4u : 0u) |
                         (c.w >= T ? 8u : 0u)) << (4 * u);
      }
      while (at) {
        const int u = __ffsll((unsigned long long)at) - 1;
        at &= at - 1ull;
        const uint32_t c = tile[u];
        const uint32_t i = (uint32_t)(tid * per + u);
        const bool neg = (c & kCodeDown) != 0u;
        double K;
        if (c & kCodeExact) {
          K = load_at(I->key, i * 8u);
        } else {
          const double2 h = load_at(hh, i * 16u);
          K = switching_key_far(I, neg, h.x, h.y, load_at(I->hk, i * 8u));
          store_at(I->key, i * 8u, K);
          tile[u] = K > 0.0 ? code_of_key(K, neg) | kCodeExact | (uint32_t)u : 0u;
          if (!kTile1) touched[tid] = 1u;
          unknown |= c >= kCodeUnknown;
        }
        const uint32_t pay = i | (neg ? 0x80000000u : 0u);
        if (better(K, pay, bk, bp)) {
          bk = K;
          bp = pay;
        }
      }
    }
    // largest key, lowest index, over the wavefront and then the workgroup (the
    // index above the sign: ~(index << 1 | sign) is largest for the lowest index)
    const double wk = wave_max_f64(bk);
    const uint32_t wi = ~wave_max_u32(bk == wk ? ~(bp << 1 | bp >> 31) : 0u) & 0x7fffffffu;
    const bool wu = __ballot(unknown) != 0ull;
    if (lane == 0) {
      sh.rk[wave] = wk;
      sh.ri[wave] = wi | (wu ? 0x80000000u : 0u);
    }
    __syncthreads();
    const int ql = lane & 15;
    const double ek = ql < NW ? sh.rk[ql] : 0.0;
    const uint32_t ei = ql < NW ? sh.ri[ql] : 0u;
    const double rk = wave_max_f64(ek);
    // none of them can flip, or one's place in the order was unknown until now:
    // choose again by the new codes
    j = -1;
    if (!(rk > 0.0) || __ballot((ei >> 31) != 0u) != 0ull) continue;
    stop = done >= left0 || (deadline && sh.pause);
    if (stop) break;
    const uint32_t jx = ~wave_max_u32(ek == rk ? ~ei : 0u);
    j = (int32_t)(jx >> 1);
    Slot q;
    if (tid < D) {
      load_row(j, tid, q.i0, q.ab);
      load_state(q);
    }
    flip(q, (jx & 1u) != 0u);
  }
  if (stop) status = deadline && sh.pause ? 1 : -5;
  if (clerk) {
    st.c.flips += done;
    st.c.logpos = logpos + done;
    st.c.hash = hash;
  }
  __syncthreads();
  return status;
}

// The two largest values of a group of lanes from each lane's two.
template <int CTRL>
__device__ __forceinline__ void top2_step(double& m, double& s) {
  const double om = dpp_f64<CTRL>(m), os = dpp_f64<CTRL>(s);
  s = fmax(fmax(s, os), fmin(m, om));
  m = fmax(m, om);
}
// Relax at step t in speculative batches by tiles (needs 1024 threads).  A
// batch takes the rows' bests that beat every row's second, in their order, as
// many as the workgroup has a lane for each neighbour (if there is none, the
// largest key alone).  A wavefront, or half of one, loads its member's row and
// its neighbours' state and looks whether they meet another member's in the
// conflict table; the FP64 powers of the new keys go to dense lanes; the prefix
// that the one-at-a-time relax would flip in this order (see above) is
// committed.  16 lanes then scan each changed tile again, and each row that owns
// one.
// What bounds it: a chain of eight phases a barrier apart, 13,000-15,000 cycles
// a batch: the tiles (one trip to memory, 2,000), their rows (2,000), the
// candidates and their ranks (2,600), the members' rows and neighbours (two
// trips, 4,400; the rows of coming members are loaded ahead into the cache),
// the powers (2,500: one dense pass instead of one per wavefront, which took
// 4,400) and the commit.  Magnets whose key stays 0 leave their tile alone: 15
// tiles a batch instead of 39.  Against the window's batches it has no sorts,
// no merges and no refills (21,000 cycles a batch of about the same members):
// 120,000-magnet kagome at 32 neighbours 1.04 -> 0.71 us a flip, 40,000
// 1.45 -> 0.78, 500,000 0.94 -> 0.75, 60,000-magnet square at 60 neighbours
// 3.08 -> 1.93 (its members crowd: 1.9 a batch, the cost of a max-tree flip
// either way).  Below 17 neighbours the window's batches win, which take up to
// 64 members where this takes 32 (30,000-magnet kagome at 4 neighbours 0.20
// against 0.46).  Above 2^19 magnets: square at 60 neighbours, 641,000, 2.7 ->
// 2.2, 1M-magnet kagome reversal 0.94 -> 0.72.
// Returns as relax_spec.
template <int kRows>
__device__ __forceinline__ int relax_many(const InstDev* __restrict__ I, int64_t t, RelaxState& st,
                                          int64_t ncand, uint64_t deadline) {
  using Shared = ManyShared<kRows>;
  Shared& sh = *(Shared*)lds_dyn;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = tid >> 4, l16 = tid & 15;  // the lane's place among those that scan a tile or a row
  const int NT = 1024;
  const int32_t n = (int32_t)I->n;
  const int32_t D = I->D;
  constexpr int tsh = many_tile_shift<kRows>();  // tiles of 64 or 128
  const int ntp = many_tiles<kRows>(n), span = ntp / kRows;
  const uint32_t span_inv = 0xffffffffu / (uint32_t)span + 1u;  // row of a tile: exact below 2^16
  const int wsh = D > 32 ? 6 : 5;             // lanes per member
  const int m = tid >> wsh, slot = lane & ((1 << wsh) - 1);  // the lane's member, its place there
  const int Bmax = NT >> wsh;
  double* const T1 = (double*)(lds_dyn + sizeof(Shared));       // per tile: largest key
  double* const pw = T1 + ntp;                // keys to evaluate: field components,
  double* const ph = pw + 2 * NT;             //   h_k,
  uint32_t* const T2 = (uint32_t*)(ph + NT);  // per tile: a bound of the second (upper word),
  uint32_t* const hown = T2 + ntp;
  uint32_t* const bits = hown + kManyHash;     // tile listed
  uint16_t* const list = (uint16_t*)(bits + ntp / 32);
  uint8_t* const pm = (uint8_t*)(list + kManyList);  //   member (keys to evaluate)
  uint8_t* const tp = pm + NT;                       //   the largest's place (tiles)

  const int32_t mode = I->field_mode;
  const bool carry = mode == kFieldCarry;
  const double pb = I->b, pc = I->c, ep = I->e_par, eq = I->e_perp, pbc = pb / pc;
  const int64_t left0 = I->max_flips - uniform(st.c.flips);  // flips this call may make
  const int64_t logpos = uniform(st.c.logpos);
  uint64_t hash = st.c.hash;  // the last wavefront's
  int64_t done = 0;
  ASI_GLOBAL double* const key = I->key;
  ASI_GLOBAL double2* const hh = I->h;
  ASI_GLOBAL double2* const hd = I->hd;
  const double sw = I->spec_switch >= 0.0 ? I->spec_switch : I->lds_keys != 0 ? kManySwitchLds : 0.0;
  int64_t done1 = 0;
  int nbatch = 0;

  for (int q = tid; q < ntp; q += NT) {
    T1[q] = 0.0;
    T2[q] = 0u;
  }
  for (int q = tid; q < ntp / 32; q += NT) bits[q] = 0u;
  for (int q = tid; q < kManyHash; q += NT) hown[q] = 0u;
  if (tid < kRows) {
    sh.best[tid] = 0.0;
    sh.sec[tid] = 0.0;
    sh.idx[tid] = 0u;
    ((uint8_t*)sh.stale)[tid] = 0;
  }
  if (tid == 0) {
    sh.nt = 0;
    sh.pause = 0;
  }
  __syncthreads();
  for (int64_t q = tid; q < ncand; q += NT) {
    const uint32_t tl = (I->cpay[0][q] & 0x7fffffffu) >> tsh;
    atomicOr(&bits[tl >> 5], 1u << (tl & 31u));
  }
  __syncthreads();
  // a tile's two largest keys, by 16 lanes, each with four or eight consecutive keys
  auto rescan_tile = [&](uint32_t tl) {
    const uint32_t i0 = (tl << tsh) + ((uint32_t)l16 << (tsh - 4));
    const uint32_t last = (uint32_t)(n - 1) & ~1u;  // (n odd: its second lies in the allocation's padding)
    const ASI_GLOBAL double2* const k2 = (const ASI_GLOBAL double2*)key;
    auto pair = [&](uint32_t u) { return load_at(k2, min(i0 + u, last) * 8u); };
    double2 v0 = pair(0), v1 = pair(2), v2, v3;
    if (tsh > 6) {
      v2 = pair(4);
      v3 = pair(6);
    }
    double m = 0.0, s2 = 0.0;
    uint32_t at = 0;
    auto take = [&](double x, uint32_t place) {
      x = i0 + place < (uint32_t)n ? x : 0.0;
      s2 = fmax(s2, fmin(m, x));
      at = x > m ? place : at;
      m = fmax(m, x);
    };
    take(v0.x, 0);
    take(v0.y, 1);
    take(v1.x, 2);
    take(v1.y, 3);
    if (tsh > 6) {
      take(v2.x, 4);
      take(v2.y, 5);
      take(v3.x, 6);
      take(v3.y, 7);
    }
    const double mine = m;
    top2_step<0xB1>(m, s2);
    top2_step<0x4E>(m, s2);
    top2_step<0x141>(m, s2);
    top2_step<0x140>(m, s2);
    // the first lane that has it: the lowest magnet among equal keys
    const uint32_t has = (uint32_t)(__ballot(mine == m) >> (lane & 48)) & 0xffffu;
    if (l16 == __ffs(has) - 1) {
      T1[tl] = m;
      // (at most infinity's: one more would be not a number, which fmax passes over)
      T2[tl] = s2 > 0.0 ? min((uint32_t)(__double_as_longlong(s2) >> 32) + 1u, 0x7ff00000u) : 0u;
      tp[tl] = (uint8_t)(((uint32_t)l16 << (tsh - 4)) + at);
      const uint32_t r = __umulhi(tl, span_inv);
      ((uint8_t*)sh.stale)[(r & 63u) * (kRows / 64) + (r >> 6)] = 1;
    }
  };
  for (int w0 = r16; w0 < ntp / 32; w0 += 64) {
    uint32_t b = bits[w0];
    while (b) {
      const int q = __ffs(b) - 1;
      b &= b - 1u;
      rescan_tile((uint32_t)(w0 * 32 + q));
    }
    if (l16 == 0) bits[w0] = 0u;
  }
  // list a tile whose keys changed, once
  auto touch = [&](uint32_t i) {
    const uint32_t tl = i >> tsh, b = 1u << (tl & 31u);
    if (!(atomicOr(&bits[tl >> 5], b) & b)) list[atomicAdd(&sh.nt, 1)] = (uint16_t)tl;
  };
  // the largest of a lane's share of the rows' values
  auto max_of_lane = [&](const double* v) {
    double x = 0.0;
#pragma unroll
    for (int u = 0; u < kRows / 128; ++u) {
      const double2 e = ((const double2*)v)[u * 64 + lane];
      x = fmax(x, fmax(e.x, e.y));
    }
    return x;
  };
  // conflict table: magnet + 1 and the first member there.  Of the members
  // that meet at a magnet all but the first end the prefix.
  auto meet = [&](uint32_t i) {
    const uint32_t want = (i + 1u) << 5 | (uint32_t)m;
    uint32_t q = (i * 2654435761u) >> (32 - 11);
    while (true) {
      uint32_t old = atomicCAS(&hown[q], 0u, want);
      if (old == 0u) break;
      if ((old ^ want) >> 5 == 0u) {
        old = atomicMin(&hown[q], want);
        const int first = (int)(old & 31u);
        if (first != m) atomicMin(&sh.pe, first > m ? first : m);
        break;
      }
      q = (q + 1) & (kManyHash - 1);
    }
    return (int)q;
  };

  int status = 0;
  int set = 0;
  int fold_n = 0;  // members of the last batch, to be folded into the hash
  auto fold = [&]() {
    if (wave != kMaxRelaxWaves - 1) return;
    const uint32_t jr = sh.mi[set ^ 1][lane & (kManyMembers - 1)];
    // times 2^40 + 435, in two words of the scalar unit
    uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)hash);
    uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(hash >> 32));
    for (int r = 0; r < fold_n; ++r) {
      lo ^= (uint32_t)__builtin_amdgcn_readlane((int)jr, r);
      hi ^= (uint32_t)t;
      hi = hi * 435u + __umulhi(lo, 435u) + (lo << 8);
      lo *= 435u;
    }
    hash = (uint64_t)hi << 32 | lo;
  };
  uint32_t ahead[3] = {0u, 0u, 0u}, seen = 0u;  // loaded ahead into the cache; used by nobody
  while (true) {
    // ---- changed tiles
    __syncthreads();
    const int nt = sh.nt;
    for (int r = r16; r < nt; r += 64) {
      const uint32_t tl = list[r];
      rescan_tile(tl);
      if (l16 == 0) atomicAnd(&bits[tl >> 5], ~(1u << (tl & 31u)));
    }
    __syncthreads();
    // ---- their rows
    // of the 16 lanes' rows, every 64th
    typename Shared::Stale stale = sh.stale[r16];
    if (__ballot(stale != 0)) {
      if (l16 == 0 && stale != 0) sh.stale[r16] = 0;
      uint32_t at = 0xffffffffu;
      while (stale) {
        const int r = r16 + ((__ffsll((unsigned long long)stale) - 1) >> 3) * 64;
        stale &= stale - 1;
        double x = 0.0, s2 = 0.0;
        at = 0xffffffffu;
        for (int u = l16; u < span; u += 16) {
          const int tl = r * span + u;
          const double a = T1[tl], b = __longlong_as_double((long long)((uint64_t)T2[tl] << 32));
          const uint32_t place = (uint32_t)tl << tsh | tp[tl];
          s2 = fmax(fmax(s2, b), fmin(x, a));
          at = a > x ? place : at;
          x = fmax(x, a);
        }
        const double mine = x;
        top2_step<0xB1>(x, s2);
        top2_step<0x4E>(x, s2);
        top2_step<0x141>(x, s2);
        top2_step<0x140>(x, s2);
        at = ~row_max_u32(mine == x ? ~at : 0u);
        if (l16 == 0) {
          sh.best[r] = x;
          sh.sec[r] = s2;
          sh.idx[r] = at;
        }
      }
      if (at < (uint32_t)n) {  // a future member: its row on its way to the cache
        seen ^= ahead[0] ^ ahead[1];
        const int64_t e = (int64_t)at * D;
        ahead[0] = __float_as_uint(*(const ASI_GLOBAL float*)&I->rAB[e + min(l16 * 8, D - 1)]);
        ahead[1] = (uint32_t)I->rcol[e + min(l16 * 32, D - 1)];
      }
    }
    if (tid < kManyMembers) sh.vm[tid] = 0ull;
    if (tid == 0) {
      sh.pe = kManyMembers;
      sh.nt = 0;
      sh.nc = 0;
      sh.npow = 0;
      if (deadline) sh.pause = (done > 0 && past(deadline)) ? 1 : 0;
    }
    __syncthreads();
    // ---- the candidates: the rows' bests above every second
    {
      constexpr int kOwn = kRows / kMaxRelaxWaves;  // rows of a wavefront
      const int r = wave * kOwn + (lane & (kOwn - 1));
      const double rk = sh.best[r];
      const uint32_t ri = sh.idx[r];
      const double T = wave_max_f64(max_of_lane(sh.sec));
      const bool is = lane < kOwn && rk > T;
      const unsigned long long bal = __ballot(is);
      if (bal) {
        int base = 0;
        if (lane == 0) base = atomicAdd(&sh.nc, __popcll(bal));
        base = __builtin_amdgcn_readfirstlane(base);
        if (is) {
          const int q = base + __popcll(bal & ((1ull << lane) - 1ull));
          sh.ck[q] = rk;
          sh.ci[q] = ri;
        }
      }
    }
    __syncthreads();
    // ---- the members: the candidates by rank
    uint32_t* const mi = sh.mi[set];
    const int nc = sh.nc;
    int B = min(nc, Bmax);
    if (nc == 0) {  // the largest key, the lowest magnet among equal ones
      const double x = wave_max_f64(max_of_lane(sh.best));
      if (!(x > 0.0)) break;
      uint32_t i = 0u;
#pragma unroll
      for (int u = 0; u < kRows / 64; ++u)
        i = max(i, sh.best[u * 64 + lane] == x ? ~sh.idx[u * 64 + lane] : 0u);
      i = ~wave_max_u32(i);
      if (tid == 0) {
        sh.mk[0] = x;
        mi[0] = i;
      }
      B = 1;
    } else {
      for (int q = wave; q < nc; q += kMaxRelaxWaves) {
        const double c = sh.ck[q];
        const uint32_t ci = sh.ci[q];
        int rank = 0;
        for (int u = lane; u - lane < nc; u += 64) {
          const double k = u < nc ? sh.ck[u] : 0.0;
          const uint32_t ki = u < nc ? sh.ci[u] : 0u;
          rank += __popcll(__ballot(k > c || (k == c && ki < ci)));
        }
        if (rank < Bmax && lane == 0) {
          sh.mk[rank] = c;
          mi[rank] = ci;
        }
      }
    }
    __syncthreads();
    if (deadline && sh.pause) {  // flippable magnets remain
      status = 1;
      break;
    }
    if (done >= left0) {
      status = -5;
      break;
    }
    // ---- the members' rows, their neighbours' state, conflicts and fields
    const bool on = m < B;
    uint32_t j = 0, i = 0;
    int32_t i0 = -1;
    int hs = -1, hj = -1, sj = 0, si = 0;
    double2 ab = make_double2(0.0, 0.0), nh = ab, nd = ab;
    double hki = 0.0, old = 0.0;
    if (on) {
      j = mi[m];
      if (slot < D) {
        const int64_t sl = (int64_t)j * D + slot;
        i0 = I->rcol[sl];
        ab = I->rAB[sl];
      }
      sj = load_at(I->s, j);
      // its tile, scanned next, on its way to the cache
      seen ^= ahead[2];
      ahead[2] = __float_as_uint(*(const ASI_GLOBAL float*)&key[min((j >> tsh << tsh) + (uint32_t)(slot & 7) * 16u, (uint32_t)n - 1u)]);
      if (slot == 0) hj = meet(j);
    }
    if (fold_n) fold();
    i = (uint32_t)max(i0, 0);
    if (i0 >= 0) {
      nh = load_at(hh, i * 16u);
      hki = load_at(I->hk, i * 8u);
      si = load_at(I->s, i);
      old = load_at(key, i * 8u);
      if (carry) nd = load_at(hd, i * 16u);
      hs = meet(i);
    }
    const bool down = sj < 0;
    int pos = -1;
    if (wave << (6 - wsh) < B) {
      const double two = down ? 2.0 : -2.0;  // 2 s_new
      const double da = two * ab.x, db = two * ab.y;
      nh = make_double2(nh.x + da, nh.y + db);
      nd = make_double2(nd.x + da, nd.y + db);
      bool need = i0 >= 0 && (si > 0 ? nh.x < 0.0 : nh.x > 0.0);
      if (need) {
        // the bound of key_needs_powers, its quotients from a reciprocal within
        // 2^-22, which the bound allows for; not a number is evaluated
        const double g = __builtin_amdgcn_rcp(pb * hki);
        const float e = pow_bound(fabs(nh.x) * g, ep) + pow_bound(fabs(nh.y) * g * pbc, eq);
        need = !(e < 1.0f);
      }
      const unsigned long long bal = __ballot(need);
      if (bal) {
        int base = 0;
        if (lane == 0) base = atomicAdd(&sh.npow, __popcll(bal));
        base = __builtin_amdgcn_readfirstlane(base);
        if (need) {
          pos = base + __popcll(bal & ((1ull << lane) - 1ull));
          pw[2 * pos] = fabs(nh.x);
          pw[2 * pos + 1] = fabs(nh.y);
          ph[pos] = hki;
          pm[pos] = (uint8_t)m;
        }
      }
    }
    __syncthreads();
    // ---- the powers, one per lane: the even lane's term and the odd lane's
    const int npow = sh.npow;
    int pe = min(sh.pe, B);
    if (npow) {
      for (int e = tid; e < 2 * npow; e += NT) {
        const double r = pow_far(pw[e] / (((e & 1) ? pc : pb) * ph[e >> 1]), (e & 1) ? eq : ep);
        const double L = r + dpp_f64<0xB1>(r);  // quad_perm [1,0,3,2]
        if (!(e & 1)) {
          pw[e] = (L > 1.0) ? L : 0.0;
          if (L > 1.0) atomicMax(&sh.vm[pm[e >> 1]], (unsigned long long)__double_as_longlong(L));
        }
      }
      __syncthreads();
      // a new key that beats a later member ends the prefix there
      const double km = sh.mk[lane & (kManyMembers - 1)];
      const double vm = __longlong_as_double((long long)sh.vm[lane & (kManyMembers - 1)]);
      unsigned long long b = __ballot(lane < pe && vm >= readlane_f64(km, pe - 1));
      while (b) {
        const int q = __ffsll(b) - 1;
        b &= b - 1ull;
        const unsigned long long over = __ballot(lane > q && lane < pe && km <= readlane_f64(vm, q));
        if (over) pe = __ffsll(over) - 1;
        if (q >= pe) break;
      }
    }
    // ---- commit the prefix
    int p = pe;
    if (p > left0 - done) p = (int)(left0 - done);
    if (hs >= 0) hown[hs] = 0u;  // the conflict table is left empty
    if (hj >= 0) hown[hj] = 0u;
    if (m < p) {
      if (i0 >= 0) {
        const double nkey = pos >= 0 ? pw[2 * pos] : 0.0;
        if (nkey != old) {
          store_at(key, i * 8u, nkey);
          touch(i);
        }
        store_at(hh, i * 16u, nh);
        if (carry)
          store_at(hd, i * 16u, nd);
        else if (mode == kFieldDirty)
          store_at(I->dirty, i, (uint8_t)1);
      }
      if (slot == 0) {
        store_at(key, j * 8u, 0.0);
        touch(j);
        store_at(I->s, j, down ? (int8_t)1 : (int8_t)-1);
        const int64_t q = logpos + done + m;
        if (q < I->log_cap) {
          I->log_t[q] = (int32_t)t;
          I->log_j[q] = (int32_t)j;
        }
      }
    }
    fold_n = p;
    set ^= 1;
    done += p;
    if (++nbatch == kManySwitchBatches) {
      if ((double)(done - done1) < sw * kManySwitchBatches) {
        status = 2;
        break;
      }
      nbatch = 0;
      done1 = done;
    }
  }
  fold();  // the last batch's flips
  __syncthreads();
  if (tid < kRows) sh.ci[tid] = seen ^ ahead[0] ^ ahead[1] ^ ahead[2];  // (their use)
  if (tid == NT - 1) {
    st.c.flips += done;
    st.c.logpos = logpos + done;
    st.c.hash = hash;
  }
  __syncthreads();
  return status;
}

template <int kRows>
__device__ ASI_CALLED int call_many(const InstDev* I, int64_t t, ASI_LDS RelaxState* st,
                                    int64_t ncand, uint64_t deadline) {
  return relax_many<kRows>(uniform(I), uniform(t), *(RelaxState*)st, uniform(ncand),
                           (uint64_t)uniform((int64_t)deadline));
}

__device__ __forceinline__ int run_spec(const InstDev* I, int64_t t, RelaxState* st, int64_t ncand,
                                       uint64_t deadline) {
  int64_t flips = uniform(st->c.flips), logpos = uniform(st->c.logpos);
  uint64_t hash = (uint64_t)uniform((int64_t)st->c.hash);
  const int status = relax_spec(I, t, lds_dyn, st->u.spec, ncand, flips, logpos, hash, deadline);
  __syncthreads();
  if (threadIdx.x == 0) st->c = RelaxCount{flips, logpos, hash};
  __syncthreads();
  return status;
}

__device__ ASI_CALLED int call_spec(const InstDev* I, int64_t t, ASI_LDS RelaxState* st,
                                    int64_t ncand, uint64_t deadline) {
  return run_spec(uniform(I), uniform(t), (RelaxState*)st, uniform(ncand),
                  (uint64_t)uniform((int64_t)deadline));
}

template <bool kFlatOk>
__device__ __forceinline__ int run_tree(const InstDev* I, int64_t t, RelaxState* st, bool rebuild,
                                       uint64_t deadline) {
  if (rebuild) rebuild_t1(I);
  int64_t flips = uniform(st->c.flips), logpos = uniform(st->c.logpos);
  uint64_t hash = (uint64_t)uniform((int64_t)st->c.hash);
  const int status = relax_tree<kFlatOk>(I, t, lds_dyn, st->u.tree, flips, logpos, hash, deadline);
  __syncthreads();
  if (threadIdx.x == 0) st->c = RelaxCount{flips, logpos, hash};
  __syncthreads();
  return status;
}

template <bool kTile1>
__device__ ASI_CALLED int call_lds(const InstDev* I, int64_t t, ASI_LDS RelaxState* st,
                                   int64_t ncand, bool from_pool, uint64_t deadline) {
  return relax_lds<kTile1>(uniform(I), uniform(t), lds_dyn, *(RelaxState*)st, uniform(ncand),
                           from_pool, (uint64_t)uniform((int64_t)deadline));
}

// The field phase of a whole instance by one workgroup.
__device__ ASI_CALLED void call_field(const InstDev* I0, int64_t t, bool resume) {
  const InstDev* I = uniform(I0);
  const int wave = threadIdx.x >> 6, NW = blockDim.x >> 6;
  for (int64_t row0 = (int64_t)wave * 64; row0 < I->n; row0 += (int64_t)NW * 64)
    field_rows64_pool(I, row0, uniform(t), resume);
  __syncthreads();
}

// Relax one instance at step t (Sec. II.H) and advance its run cursor.
// Steps that start with enough flippable magnets (spec_min, and a degree that
// leaves room for batches) take the speculative path; the others, and a
// speculative step whose batches stay small, go one flip at a time: with every
// key in LDS where they fit (kPathLds, kPathLdsSpec), else on the max tree
// (kPathTree, kPathSpec).  A paused step resumes on the path it was on.  All
// flip exactly the magnets, in exactly the order, of the one-at-a-time relax.
// kPathMixed holds the parts of kPathSpec and kPathLdsSpec, for launches with
// instances of both kinds.
// The one-at-a-time relax is inline (the mixed kernel's max tree): called, it
// stored and loaded some 60 registers a lane at each step, 2-3 us (a step of
// 40,000 magnets without flips took 12 us instead of 9.5; 6.0 now), and had
// registers of its loop spilled.
template <int kPath>
__device__ __forceinline__ int relax_step(const InstDev* __restrict__ I, RunDev* __restrict__ R, int64_t t,
                          RelaxState& st, uint64_t deadline) {
  constexpr bool kMixed = kPath == kPathMixed, kLds = kPath == kPathLds || kPath == kPathLdsSpec;
  const bool lds = kMixed ? I->lds_keys != 0 : kLds;
  const int64_t ncand = __hip_atomic_load(I->ccount, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int64_t acc0 = R->step_acc;  // flips of step t before a pause
  if (threadIdx.x == 0) st.c = RelaxCount{acc0, R->flips, R->hash};
  __syncthreads();
  bool spec = false;
  int status = 2;
  if ((int64_t)(uint32_t)ncand > I->ccap) {
    status = kPoolOverflow;  // cannot happen while every pass starts from an empty pool
  } else if (ncand == 0) {
    status = 0;  // nothing can flip (the field phase lists every magnet that can)
  } else {
    if constexpr (kPath != kPathTree && kPath != kPathLds) {
      spec = blockDim.x == 1024 && (R->paused ? R->spec != 0
                                              : I->D <= kSpecMaxD && ncand >= I->spec_min);
      if (spec)
        status = !many_fits(I->n, I->D)
                     ? (kPath == kPathSpec ? run_spec(I, t, &st, ncand, deadline)
                                           : call_spec(I, t, (ASI_LDS RelaxState*)&st, ncand, deadline))
                 : lds || I->n <= kManyMaxN64
                     ? call_many<kManyRows>(I, t, (ASI_LDS RelaxState*)&st, ncand, deadline)
                     : call_many<kManyRowsBig>(I, t, (ASI_LDS RelaxState*)&st, ncand, deadline);
    }
    if (status == 2) {
      const bool tile1 = flip_tile(I->n, (int)blockDim.x) == 4;
      if constexpr (kLds)
        status = tile1 ? relax_lds<true>(I, t, lds_dyn, st, ncand, !spec, deadline)
                       : relax_lds<false>(I, t, lds_dyn, st, ncand, !spec, deadline);
      else if (!kMixed || !lds)
        status = run_tree<kPath == kPathTree>(I, t, &st, spec, deadline);
      else
        status = tile1 ? call_lds<true>(I, t, (ASI_LDS RelaxState*)&st, ncand, !spec, deadline)
                       : call_lds<false>(I, t, (ASI_LDS RelaxState*)&st, ncand, !spec, deadline);
      spec = false;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_store(I->ccount, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t flips = st.c.flips;
    R->flips += flips - acc0;
    R->flips_call += flips - acc0;
    R->hash = st.c.hash;
    if (status == 1) {
      R->step_acc = flips;
      R->paused = 1;
      R->spec = spec ? 1 : 0;
      R->active = 0;
    } else {
      if (t >= 0 && t < I->K && I->step_flips) I->step_flips[t] = (int32_t)flips;
      R->step_acc = 0;
      R->paused = 0;
      R->cur_step = t;
      R->t = t + 1;
      if (status != 0) R->status = status;
      R->active = (status == 0 && R->t < R->t_end) ? 1 : 0;
    }
  }
  __syncthreads();
  return status;
}

template <int kPath>
__global__ __launch_bounds__(64 * kMaxRelaxWaves) void k_relax(const InstDev* __restrict__ insts,
                                                              RunDev* __restrict__ runs) {
  RunDev* R = runs + blockIdx.x;
  // a relax paused at a burst deadline finishes its step here, its
  // structures rebuilt by the preceding field launch
  if (!R->active && !R->paused) return;
  const InstDev* I = insts + blockIdx.x;
  __shared__ RelaxState st;
  relax_step<kPath>(I, R, R->t, st, 0);
}

// One workgroup per instance runs whole field steps -- its own field phase,
// wavefront by wavefront, then the relax -- through its own protocol, so
// instances never wait for each other between steps.  Stops after max_steps
// steps, at the end of the protocol, on ELOOP, or once budget_ticks of the
// constant-rate device clock have passed: checked between steps and inside
// the relax, which then pauses mid-step.  A paused instance finishes the
// step it stopped in first, its relax structures rebuilt (by the preceding
// field launch when first_ready); the flips it makes, and their order, are
// those of an uninterrupted relax.
template <int kPath>
__global__ __launch_bounds__(64 * kMaxRelaxWaves) void k_fused(const InstDev* __restrict__ insts,
                                                              RunDev* __restrict__ runs,
                                                              int64_t max_steps,
                                                              int64_t budget_ticks,
                                                              int32_t first_ready) {
  RunDev* R = runs + blockIdx.x;
  const bool paused = R->paused != 0;
  if (!R->active && !paused) return;
  const InstDev* I = uniform(insts + blockIdx.x);
  __shared__ RelaxState st;
  __shared__ int go;
  const uint64_t t_start = wall_clock64();
  const uint64_t deadline = budget_ticks > 0 ? t_start + (uint64_t)budget_ticks : 0;
  bool ready = first_ready != 0;
  if (paused && !ready) {
    call_field(I, R->t, true);
    ready = true;
  }
  for (int64_t k = 0; k < max_steps; ++k) {
    const int64_t t = R->t;
    if (!ready) call_field(I, t, false);
    ready = false;
    if (relax_step<kPath>(I, R, t, st, deadline) != 0) break;
    if (threadIdx.x == 0) go = (R->active && !past(deadline)) ? 1 : 0;
    __syncthreads();
    if (!go) break;
  }
}

// Run-cursor update, launched on the stream so it orders with the kernels
// (and can sit inside a captured graph).
__global__ void k_set_run(RunDev* R, int32_t* ccount, int64_t t, int64_t t_end, int32_t active,
                          int32_t reset_log, int64_t cur_step) {
  if (threadIdx.x != 0) return;
  if (ccount) *ccount = 0;  // the next field pass starts an empty candidate pool
  R->t = t;
  R->t_end = t_end;
  R->active = active;
  R->status = 0;
  R->flips_call = 0;
  R->paused = 0;
  R->step_acc = 0;
  if (reset_log) {
    R->flips = 0;
    R->hash = 0xcbf29ce484222325ull;
    R->cur_step = cur_step;
  }
}

// ------------------------------------------------------------ analysis
// Net magnetisation M = sum_i s_i mhat_i, the quantity a hysteresis loop
// plots (as M / M_S, M_S = n for unit moments).  Reduced in a fixed order,
// so the same spins give the same bits on every call: thread k of block b
// adds rows b*T + k, then every G*T rows, in ascending order; the block
// halves its sums in LDS; one block then halves the G block sums.
constexpr int kMagThreads = 256;
constexpr int kMagBlocks = 256;   // == kMagThreads: the final block takes one sum per thread

__device__ __forceinline__ void mag_halve(double* sx, double* sy) {
  for (int w = kMagThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      sx[threadIdx.x] = sx[threadIdx.x] + sx[threadIdx.x + w];
      sy[threadIdx.x] = sy[threadIdx.x] + sy[threadIdx.x + w];
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kMagThreads)
k_mag_partial(const int8_t* __restrict__ s, const double* __restrict__ mx,
              const double* __restrict__ my, int64_t n, double* __restrict__ part) {
  __shared__ double sx[kMagThreads], sy[kMagThreads];
  const int64_t stride = (int64_t)kMagBlocks * kMagThreads;
  double ax = 0.0, ay = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kMagThreads + threadIdx.x; i < n; i += stride) {
    const bool up = s[i] > 0;
    ax = ax + (up ? mx[i] : -mx[i]);
    ay = ay + (up ? my[i] : -my[i]);
  }
  sx[threadIdx.x] = ax;
  sy[threadIdx.x] = ay;
  __syncthreads();
  mag_halve(sx, sy);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = sx[0];
    part[2 * blockIdx.x + 1] = sy[0];
  }
}

__global__ void __launch_bounds__(kMagThreads)
k_mag_final(const double* __restrict__ part, double* __restrict__ out) {
  __shared__ double sx[kMagThreads], sy[kMagThreads];
  sx[threadIdx.x] = part[2 * threadIdx.x];
  sy[threadIdx.x] = part[2 * threadIdx.x + 1];
  __syncthreads();
  mag_halve(sx, sy);
  if (threadIdx.x == 0) {
    out[0] = sx[0];
    out[1] = sy[0];
  }
}

static_assert(2 * kMagBlocks == kMagPartials, "block sums buffer");

// Net magnetisation of groups of magnets, e.g. the islands meeting at each
// vertex (the vertex maps of Sec. IV.B): group g sums s_i mhat_i over
// idx[ptr[g] .. ptr[g+1]) in that order, one thread per group.
__global__ void __launch_bounds__(256)
k_group_mag(const int8_t* __restrict__ s, const double* __restrict__ mx,
            const double* __restrict__ my, const int64_t* __restrict__ ptr,
            const int32_t* __restrict__ idx, int64_t ngroups, double* __restrict__ out) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= ngroups) return;
  double ax = 0.0, ay = 0.0;
  for (int64_t e = ptr[g]; e < ptr[g + 1]; ++e) {
    const int32_t i = idx[e];
    const bool up = s[i] > 0;
    ax = ax + (up ? mx[i] : -mx[i]);
    ay = ay + (up ? my[i] : -my[i]);
  }
  out[2 * g] = ax;
  out[2 * g + 1] = ay;
}

// Spin-spin correlation by separation (Sec. IV.B): a pair (i, j) of
// neighbours correlates +1 when its dipolar energy -s_i s_j A_ij is at its
// minimum (s_i s_j A_ij > 0), -1 at its maximum, and 0 when the coupling
// vanishes (|A_ij| <= 1e-9 |alpha| / r^3, i.e. zero up to rounding).  Each
// pair counts once (j > i) in bin floor(r / w) of its distance r; pairs past
// the last bin are skipped.  The distance is formed with correctly rounded
// operations only, so the bin is the same as any IEEE evaluation of the
// same expression.  Sums and counts are integers, added per workgroup in
// LDS and then once per bin into the global totals.
__global__ void __launch_bounds__(256)
k_corr(const InstDev* __restrict__ I, const double* __restrict__ xy, double w, int32_t nbins,
       double abs_alpha, unsigned long long* __restrict__ sum, unsigned long long* __restrict__ cnt) {
  extern __shared__ int32_t lds_bins[];   // [2][nbins]
  int32_t* bs = lds_bins;
  int32_t* bc = lds_bins + nbins;
  for (int b = threadIdx.x; b < 2 * nbins; b += blockDim.x) lds_bins[b] = 0;
  __syncthreads();
  const int64_t n = I->n, D = I->D;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double xi = xy[2 * i], yi = xy[2 * i + 1];
    const int si = I->s[i];
    const int32_t L = I->len[i];
    // the sliced tables: slot k of 64 consecutive rows is contiguous, so
    // the lanes of a wavefront (consecutive rows) load it together
    for (int32_t k = 0; k < L; ++k) {
      const int64_t sl = slot_of(i, (int32_t)D, k);
      const int32_t j = I->col[sl];
      if (j <= i) continue;
      const double dx = __dsub_rn(xi, xy[2 * (int64_t)j]);
      const double dy = __dsub_rn(yi, xy[2 * (int64_t)j + 1]);
      const double r = __dsqrt_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)));
      const double q = floor(__ddiv_rn(r, w));
      if (!(q < (double)nbins)) continue;
      const int b = (int)q;
      const double a = I->A[sl];
      int c = 0;
      if (fabs(a) > 1e-9 * abs_alpha / (r * r * r)) c = ((si * I->s[j]) * (a > 0.0 ? 1 : -1) > 0) ? 1 : -1;
      atomicAdd(&bs[b], c);
      atomicAdd(&bc[b], 1);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < nbins; b += blockDim.x) {
    if (bc[b] != 0) {
      atomicAdd(&sum[b], (unsigned long long)(long long)bs[b]);
      atomicAdd(&cnt[b], (unsigned long long)bc[b]);
    }
  }
}

// Switching order of a flip log (Sec. IV.D): the log position of each
// magnet's first switch, and the twice-average rank of each magnet in that
// order.  Switched magnets have distinct first positions; a magnet that
// never switched is placed after all of them, so those magnets share the
// ranks S+1 .. n (S = switched magnets) and each gets their mean.  All of it
// is integer arithmetic: the results do not depend on the order of atomics.
constexpr int kRankBlock = 1024;  // log entries per block of the rank scan

__global__ void __launch_bounds__(256)
k_fill_u64(unsigned long long* __restrict__ p, int64_t n, unsigned long long v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// pos[j] = smallest log position k with log_j[k] == j (pos preset to L).
__global__ void __launch_bounds__(256)
k_first_switch(const int32_t* __restrict__ log_j, int64_t L, unsigned long long* __restrict__ pos) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < L;
       k += (int64_t)gridDim.x * blockDim.x)
    atomicMin(&pos[log_j[k]], (unsigned long long)k);
}

// Log entry k is a first switch when pos[log_j[k]] == k.  Returns its
// exclusive rank among the first switches of this block's entries (uniform
// over the block after the call: wave totals in wtot[16]).
__device__ __forceinline__ int first_rank_in_block(const int32_t* __restrict__ log_j, int64_t L,
                                                   const unsigned long long* __restrict__ pos,
                                                   int* wtot, bool& first, int32_t& j,
                                                   int& block_total) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t k = (int64_t)blockIdx.x * kRankBlock + tid;
  first = false;
  j = 0;
  if (k < L) {
    j = log_j[k];
    first = pos[j] == (unsigned long long)k;
  }
  const unsigned long long bal = __ballot(first);
  if (lane == 0) wtot[wave] = __popcll(bal);
  __syncthreads();
  int before = 0, tot = 0;
  for (int w = 0; w < kRankBlock / 64; ++w) {
    if (w < wave) before += wtot[w];
    tot += wtot[w];
  }
  block_total = tot;
  return before + __popcll(bal & ((1ull << lane) - 1ull));
}

__global__ void __launch_bounds__(kRankBlock)
k_first_count(const int32_t* __restrict__ log_j, int64_t L,
              const unsigned long long* __restrict__ pos, int64_t* __restrict__ cnt) {
  __shared__ int wtot[kRankBlock / 64];
  bool first;
  int32_t j;
  int tot;
  (void)first_rank_in_block(log_j, L, pos, wtot, first, j, tot);
  if (threadIdx.x == 0) cnt[blockIdx.x] = tot;
}

// Exclusive scan of the nb block counts by one workgroup (chunks of 1024
// with a running carry); total[0] = number of switched magnets.
__global__ void __launch_bounds__(kRankBlock)
k_scan_counts(const int64_t* __restrict__ cnt, int64_t nb, int64_t* __restrict__ off,
              int64_t* __restrict__ total) {
  __shared__ int64_t buf[kRankBlock];
  __shared__ int64_t carry;
  const int tid = threadIdx.x;
  if (tid == 0) carry = 0;
  __syncthreads();
  for (int64_t c0 = 0; c0 < nb; c0 += kRankBlock) {
    const int64_t v = (c0 + tid < nb) ? cnt[c0 + tid] : 0;
    buf[tid] = v;
    __syncthreads();
    for (int d = 1; d < kRankBlock; d <<= 1) {  // inclusive Hillis-Steele scan
      const int64_t add = tid >= d ? buf[tid - d] : 0;
      __syncthreads();
      buf[tid] += add;
      __syncthreads();
    }
    if (c0 + tid < nb) off[c0 + tid] = carry + buf[tid] - v;
    __syncthreads();
    if (tid == 0) carry += buf[kRankBlock - 1];
    __syncthreads();
  }
  if (tid == 0) total[0] = carry;
}

// Every magnet first gets the mean rank of the never-switched group,
// 2r = S + 1 + n; then each first switch overwrites its magnet's value.
__global__ void __launch_bounds__(256)
k_rank_rest(int64_t* __restrict__ r2, int64_t n, const int64_t* __restrict__ total) {
  const int64_t v = total[0] + 1 + n;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    r2[i] = v;
}

__global__ void __launch_bounds__(kRankBlock)
k_rank_switched(const int32_t* __restrict__ log_j, int64_t L,
                const unsigned long long* __restrict__ pos, const int64_t* __restrict__ off,
                int64_t* __restrict__ r2) {
  __shared__ int wtot[kRankBlock / 64];
  bool first;
  int32_t j;
  int tot;
  const int r = first_rank_in_block(log_j, L, pos, wtot, first, j, tot);
  if (first) r2[j] = 2 * (off[blockIdx.x] + r + 1);
}

// Pearson correlation of two rank vectors from exact sums: with u = 2r -
// (n + 1) per magnet, one block adds u_a u_b, u_a^2 and u_b^2 of its 256
// magnets into part[3 b .. 3 b + 2] (each |u| < n <= 2^27, so a block sum
// stays below 2^62).
constexpr int kCorrRankThreads = 256;

__global__ void __launch_bounds__(kCorrRankThreads)
k_rank_corr(const int64_t* __restrict__ r2a, const int64_t* __restrict__ r2b, int64_t n,
            long long* __restrict__ part) {
  __shared__ long long sab[kCorrRankThreads], saa[kCorrRankThreads], sbb[kCorrRankThreads];
  const int tid = threadIdx.x;
  const int64_t i = (int64_t)blockIdx.x * kCorrRankThreads + tid;
  long long ua = 0, ub = 0;
  if (i < n) {
    ua = (long long)(r2a[i] - (n + 1));
    ub = (long long)(r2b[i] - (n + 1));
  }
  sab[tid] = ua * ub;
  saa[tid] = ua * ua;
  sbb[tid] = ub * ub;
  __syncthreads();
  for (int w = kCorrRankThreads / 2; w > 0; w >>= 1) {
    if (tid < w) {
      sab[tid] += sab[tid + w];
      saa[tid] += saa[tid + w];
      sbb[tid] += sbb[tid + w];
    }
    __syncthreads();
  }
  if (tid == 0) {
    part[3 * blockIdx.x] = sab[0];
    part[3 * blockIdx.x + 1] = saa[0];
    part[3 * blockIdx.x + 2] = sbb[0];
  }
}

// Exact totals of the nb block sums of k_rank_corr, one workgroup: each
// thread adds a strided subset of the blocks into 128-bit (low, high)
// accumulators, then the threads' accumulators are added pairwise in LDS.
// Integer sums, so the totals do not depend on the order (|total| < 2^81).
struct I128 {
  unsigned long long lo;
  long long hi;
};

__device__ inline I128 add128(I128 a, I128 b) {
  I128 r;
  r.lo = a.lo + b.lo;
  r.hi = a.hi + b.hi + (r.lo < a.lo ? 1 : 0);
  return r;
}

__device__ inline I128 widen(long long v) {
  I128 r;
  r.lo = (unsigned long long)v;
  r.hi = v < 0 ? -1 : 0;
  return r;
}

__global__ void __launch_bounds__(kCorrRankThreads)
k_rank_corr_total(const long long* __restrict__ part, int64_t nb, long long* __restrict__ tot) {
  __shared__ I128 acc[3][kCorrRankThreads];
  const int tid = threadIdx.x;
  I128 a[3] = {{0ull, 0}, {0ull, 0}, {0ull, 0}};
  for (int64_t b = tid; b < nb; b += kCorrRankThreads)
    for (int c = 0; c < 3; ++c) a[c] = add128(a[c], widen(part[3 * b + c]));
  for (int c = 0; c < 3; ++c) acc[c][tid] = a[c];
  __syncthreads();
  for (int w = kCorrRankThreads / 2; w > 0; w >>= 1) {
    if (tid < w)
      for (int c = 0; c < 3; ++c) acc[c][tid] = add128(acc[c][tid], acc[c][tid + w]);
    __syncthreads();
  }
  if (tid < 3) {
    tot[2 * tid] = (long long)acc[tid][0].lo;
    tot[2 * tid + 1] = acc[tid][0].hi;
  }
}

// ------------------------------------------------------------ measurement
// Dependent-load latency: each of the first `lanes` lanes of one wavefront
// follows a chain of indices from its own start (each load's address comes
// from the previous load), `hops` times; lane 0 records the elapsed ticks of
// the device's constant-rate clock.  With 64 lanes a hop is one scattered
// 64-address gather, the unit of work of the relax's neighbour updates.  The
// chain is built and checked on the host to be one cycle over the buffer,
// so every load is in bounds however many hops are taken.
__global__ void k_chase(const int32_t* __restrict__ chain, const int32_t* __restrict__ starts,
                        int32_t lanes, int64_t hops, unsigned long long* __restrict__ out) {
  const int lane = threadIdx.x;
  if (blockIdx.x != 0 || lane >= lanes) return;
  int32_t p = starts[lane];
  const uint64_t t0 = wall_clock64();
  for (int64_t h = 0; h < hops; ++h) p = chain[p];
  const uint64_t t1 = wall_clock64();
  if (lane == 0) out[0] = t1 - t0;
  out[1 + lane] = (unsigned long long)p;  // keeps every chain live
}

}  // namespace

// ------------------------------------------------------------ launchers
void launch_chase(const int32_t* chain, const int32_t* starts, int32_t lanes, int64_t hops,
                  unsigned long long* out, hipStream_t st) {
  hipLaunchKernelGGL(k_chase, dim3(1), dim3(64), 0, st, chain, starts, lanes, hops, out);
}

int64_t switching_scratch_count(int64_t L) {
  const int64_t nb = std::max<int64_t>(1, (L + kRankBlock - 1) / kRankBlock);
  return 2 * nb + 1;
}

void launch_switching_ranks(const int32_t* log_j, int64_t L, int64_t n, unsigned long long* pos,
                            int64_t* r2, int64_t* scratch, hipStream_t st) {
  const int64_t nb = std::max<int64_t>(1, (L + kRankBlock - 1) / kRankBlock);
  const unsigned gn = (unsigned)std::min<int64_t>(4096, std::max<int64_t>(1, (n + 255) / 256));
  const unsigned gl = (unsigned)std::min<int64_t>(4096, std::max<int64_t>(1, (L + 255) / 256));
  int64_t* cnt = scratch;
  int64_t* off = scratch + nb;
  int64_t* total = scratch + 2 * nb;
  hipLaunchKernelGGL(k_fill_u64, dim3(gn), dim3(256), 0, st, pos, n, (unsigned long long)L);
  if (L > 0)
    hipLaunchKernelGGL(k_first_switch, dim3(gl), dim3(256), 0, st, log_j, L, pos);
  hipLaunchKernelGGL(k_first_count, dim3((unsigned)nb), dim3(kRankBlock), 0, st, log_j, L, pos,
                     cnt);
  hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(kRankBlock), 0, st, cnt, nb, off, total);
  hipLaunchKernelGGL(k_rank_rest, dim3(gn), dim3(256), 0, st, r2, n, total);
  hipLaunchKernelGGL(k_rank_switched, dim3((unsigned)nb), dim3(kRankBlock), 0, st, log_j, L, pos,
                     off, r2);
}

int64_t rank_corr_blocks(int64_t n) { return (n + kCorrRankThreads - 1) / kCorrRankThreads; }

void launch_rank_corr_total(const long long* part, int64_t nb, long long* tot, hipStream_t st) {
  hipLaunchKernelGGL(k_rank_corr_total, dim3(1), dim3(kCorrRankThreads), 0, st, part, nb, tot);
}

// ------------------------------------------------------------ static scratch
// Scratch of the allocation-free switching-order comparison: one array per
// GPU for the life of the process.  In host code `scratch` only names the
// symbol; its device address comes from hipGetSymbolAddress, per device.
namespace {

constexpr size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
constexpr size_t kRhoRankBytes = align256(8 * (size_t)kStaticRhoMaxN);
constexpr size_t kRhoTmpBytes =
    align256(8 * (size_t)(2 * ((kStaticRhoMaxLog + kRankBlock - 1) / kRankBlock) + 1));
constexpr size_t kRhoPartBytes =
    align256(8 * 3 * (size_t)((kStaticRhoMaxN + kCorrRankThreads - 1) / kCorrRankThreads));
constexpr size_t kRhoTotBytes = align256(8 * 6);
constexpr size_t kScratchBytes = 4 * kRhoRankBytes + 2 * kRhoTmpBytes + kRhoPartBytes + kRhoTotBytes;

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
unsigned char* g_scratch_ptr[kMaxScratchDevices] = {};

}  // namespace

size_t static_scratch_bytes() { return kScratchBytes; }

StaticRhoScratch carve_static_rho(unsigned char* base) {
  StaticRhoScratch S;
  size_t off = 0;
  for (int k = 0; k < 2; ++k) {
    S.pos[k] = reinterpret_cast<unsigned long long*>(base + off);
    off += kRhoRankBytes;
    S.r2[k] = reinterpret_cast<int64_t*>(base + off);
    off += kRhoRankBytes;
  }
  for (int k = 0; k < 2; ++k) {
    S.tmp[k] = reinterpret_cast<int64_t*>(base + off);
    off += kRhoTmpBytes;
  }
  S.part = reinterpret_cast<long long*>(base + off);
  off += kRhoPartBytes;
  S.tot = reinterpret_cast<long long*>(base + off);
  return S;
}

hipError_t static_scratch_address(unsigned char** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<unsigned char*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

void launch_rank_correlation(const int64_t* r2a, const int64_t* r2b, int64_t n, long long* part,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_rank_corr, dim3((unsigned)rank_corr_blocks(n)), dim3(kCorrRankThreads), 0,
                     st, r2a, r2b, n, part);
}

void launch_correlation(const InstDev* inst, int64_t n, const double* xy, double w,
                        int32_t nbins, double abs_alpha, uint64_t* sum, uint64_t* cnt,
                        hipStream_t st) {
  const int64_t blocks = std::min<int64_t>(1024, std::max<int64_t>(1, (n + 255) / 256));
  hipLaunchKernelGGL(k_corr, dim3((unsigned)blocks), dim3(256), 2 * nbins * sizeof(int32_t), st,
                     inst, xy, w, nbins, abs_alpha,
                     reinterpret_cast<unsigned long long*>(sum),
                     reinterpret_cast<unsigned long long*>(cnt));
}

void launch_group_magnetization(const int8_t* s, const double* mx, const double* my,
                                const int64_t* ptr, const int32_t* idx, int64_t ngroups,
                                double* out, hipStream_t st) {
  const int64_t blocks = (ngroups + 255) / 256;
  hipLaunchKernelGGL(k_group_mag, dim3((unsigned)blocks), dim3(256), 0, st, s, mx, my, ptr, idx,
                     ngroups, out);
}

void launch_magnetization(const int8_t* s, const double* mx, const double* my, int64_t n,
                          double* part, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_mag_partial, dim3(kMagBlocks), dim3(kMagThreads), 0, st, s, mx, my, n,
                     part);
  hipLaunchKernelGGL(k_mag_final, dim3(1), dim3(kMagThreads), 0, st, part, out);
}

void launch_draw_hk(double* hk, int64_t n, double mean, double k, uint64_t seed, hipStream_t st) {
  if (n <= 0) return;
  hipLaunchKernelGGL(k_draw_hk, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, hk, n, mean, k,
                     seed);
}

void launch_inverse_hk(const double* hk, int64_t n, double b, double* g, hipStream_t st) {
  hipLaunchKernelGGL(k_inverse_hk, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, hk, n, b, g);
}

void launch_neighbour_count(const double* x, const double* y, const int32_t* cellx,
                            const int32_t* celly, const int32_t* cell_start,
                            const int32_t* cell_members, int64_t n, int64_t gx, int64_t gy,
                            double cut2, int32_t* len, int32_t* dup_flag, hipStream_t st) {
  const int bs = 256;
  const int64_t nb = (n + bs - 1) / bs;
  hipLaunchKernelGGL(k_nb_count, dim3((unsigned)nb), dim3(bs), 0, st, x, y, cellx, celly,
                     cell_start, cell_members, n, gx, gy, cut2, len, dup_flag);
}

void launch_neighbour_fill(const double* x, const double* y, const double* mx, const double* my,
                           const int32_t* cellx, const int32_t* celly, const int32_t* cell_start,
                           const int32_t* cell_members, int64_t n, int64_t gx, int64_t gy,
                           double cut2, double alpha, int32_t D, int32_t* col, double* A,
                           double* B, int32_t* rcol, double2* rAB, hipStream_t st) {
  const int bs = 128;
  const int64_t nb = (n + bs - 1) / bs;
  hipLaunchKernelGGL(k_nb_fill, dim3((unsigned)nb), dim3(bs), 0, st, x, y, mx, my, cellx, celly,
                     cell_start, cell_members, n, gx, gy, cut2, alpha, D, col, A, B, rcol, rAB);
}

void launch_field(const InstDev* insts, RunDev* runs, const int32_t* blk_inst,
                  const int32_t* blk_row0, int64_t nblocks, hipStream_t st) {
  if (nblocks <= 0) return;
  hipLaunchKernelGGL(k_field, dim3((unsigned)nblocks), dim3(kFieldBlock), 0, st, insts, runs,
                     blk_inst, blk_row0);
}

void launch_field_hd(const InstDev* inst, RunDev* run, int64_t n, int32_t rows, int32_t nch,
                     hipStream_t st) {
  const int64_t nsl = (n + 63) / 64;
  if (rows == 0 && nch > 0 && nsl < kHdSplitSlices) {
    hipLaunchKernelGGL(k_field_hd_part, dim3((unsigned)(nsl * nch)), dim3(512), 0, st, inst, run);
    hipLaunchKernelGGL(k_field_hd_comb, dim3((unsigned)((nsl + 3) / 4)), dim3(256), 0, st, inst,
                       run);
    return;
  }
  // rows per workgroup: by default the largest that still gives the device
  // about four workgroups per compute unit, at least 8
  const int R = rows ? rows
                     : nsl >= 1024 ? 64 : 2 * nsl >= 1024 ? 32 : 4 * nsl >= 1024 ? 16 : 8;
  const unsigned blocks = (unsigned)(((nsl + 7) / 8) * 8 * (64 / R));
  switch (R) {
    case 64:
      hipLaunchKernelGGL(k_field_hd<64>, dim3(blocks), dim3(512), 0, st, inst, run);
      break;
    case 32:
      hipLaunchKernelGGL(k_field_hd<32>, dim3(blocks), dim3(256), 0, st, inst, run);
      break;
    case 16:
      hipLaunchKernelGGL(k_field_hd<16>, dim3(blocks), dim3(128), 0, st, inst, run);
      break;
    default:
      hipLaunchKernelGGL(k_field_hd<8>, dim3(blocks), dim3(64), 0, st, inst, run);
      break;
  }
  if (R < 64)
    hipLaunchKernelGGL(k_slice_max, dim3((unsigned)((nsl + 3) / 4)), dim3(256), 0, st, inst, run);
}

void launch_relax(const InstDev* insts, RunDev* runs, int32_t count, int32_t waves,
                  size_t lds_bytes, RelaxPath path, hipStream_t st) {
  if (count <= 0) return;
  const dim3 g((unsigned)count), b((unsigned)(64 * waves));
  if (path == kPathLds)
    hipLaunchKernelGGL(k_relax<kPathLds>, g, b, lds_bytes, st, insts, runs);
  else if (path == kPathLdsSpec)
    hipLaunchKernelGGL(k_relax<kPathLdsSpec>, g, b, lds_bytes, st, insts, runs);
  else if (path == kPathTree)
    hipLaunchKernelGGL(k_relax<kPathTree>, g, b, lds_bytes, st, insts, runs);
  else if (path == kPathMixed)
    hipLaunchKernelGGL(k_relax<kPathMixed>, g, b, lds_bytes, st, insts, runs);
  else
    hipLaunchKernelGGL(k_relax<kPathSpec>, g, b, lds_bytes, st, insts, runs);
}

void launch_fused(const InstDev* insts, RunDev* runs, int32_t count, int32_t waves,
                  size_t lds_bytes, RelaxPath path, int64_t max_steps, int64_t budget_ticks,
                  int32_t first_ready, hipStream_t st) {
  if (count <= 0) return;
  const dim3 g((unsigned)count), b((unsigned)(64 * waves));
  if (path == kPathLds)
    hipLaunchKernelGGL(k_fused<kPathLds>, g, b, lds_bytes, st, insts, runs, max_steps,
                       budget_ticks, first_ready);
  else if (path == kPathLdsSpec)
    hipLaunchKernelGGL(k_fused<kPathLdsSpec>, g, b, lds_bytes, st, insts, runs, max_steps,
                       budget_ticks, first_ready);
  else if (path == kPathMixed)
    hipLaunchKernelGGL(k_fused<kPathMixed>, g, b, lds_bytes, st, insts, runs, max_steps,
                       budget_ticks, first_ready);
  else
    hipLaunchKernelGGL(k_fused<kPathSpec>, g, b, lds_bytes, st, insts, runs, max_steps,
                       budget_ticks, first_ready);
}

void launch_set_run(RunDev* run, int32_t* ccount, int64_t t, int64_t t_end, int32_t active,
                    int32_t reset_log, int64_t cur_step, hipStream_t st) {
  hipLaunchKernelGGL(k_set_run, dim3(1), dim3(64), 0, st, run, ccount, t, t_end, active,
                     reset_log, cur_step);
}

int32_t relax_l1_shift(int64_t n) {
  int32_t s = 6;
  while (((n + (1LL << s) - 1) >> s) > kMaxL1Tiles) ++s;
  return s;
}

namespace {
size_t batch_lds_bytes(int64_t n, int32_t D) {
  return many_fits(n, D) ? many_lds_bytes(n) : spec_lds_bytes();
}
}  // namespace

// the relax paths of a step share the space
size_t relax_lds_bytes(int64_t n, int32_t D, int32_t waves, int32_t l1_shift) {
  const size_t a = relax_tree_lds_bytes(n, l1_shift);
  return relax_may_speculate(D, waves) ? std::max(a, batch_lds_bytes(n, D)) : a;
}

size_t relax_keys_lds_bytes(int64_t n, int32_t D, int32_t waves) {
  const size_t a = flip_lds_bytes(n, 64 * waves);
  return relax_may_speculate(D, waves) ? std::max(a, batch_lds_bytes(n, D)) : a;
}

hipError_t configure_kernels() {
  // the relax kernels take more than 64 KB of dynamic LDS
  const int tree = (int)std::max({relax_tree_lds_bytes((int64_t)kMaxL1Tiles << 6, 6), spec_lds_bytes(),
                                  many_lds_bytes(kManyMaxN)});
  const int keys = (int)flip_lds_bytes(kLdsMaxN, 64 * kMaxRelaxWaves);
  const std::pair<const void*, int> k[] = {
      {reinterpret_cast<const void*>(&k_relax<kPathTree>), tree},
      {reinterpret_cast<const void*>(&k_relax<kPathSpec>), tree},
      {reinterpret_cast<const void*>(&k_relax<kPathLds>), keys},
      {reinterpret_cast<const void*>(&k_relax<kPathLdsSpec>), keys},
      {reinterpret_cast<const void*>(&k_fused<kPathLdsSpec>), keys},
      {reinterpret_cast<const void*>(&k_fused<kPathSpec>), tree},
      {reinterpret_cast<const void*>(&k_fused<kPathLds>), keys},
      {reinterpret_cast<const void*>(&k_relax<kPathMixed>), std::max(tree, keys)},
      {reinterpret_cast<const void*>(&k_fused<kPathMixed>), std::max(tree, keys)}};
  hipError_t e = hipSuccess;
  for (const auto& f : k)
    if (e == hipSuccess)
      e = hipFuncSetAttribute(f.first, hipFuncAttributeMaxDynamicSharedMemorySize, f.second);
  return e;
}

}  // namespace asi
