// Right-hand side b = chi - b_sol for F electrolyte frames (Sec. III.A, Eq. 25).
//
// b_sol,i = sum_I q_I e_iI(a_i) with e_iI the Gaussian Ewald entry (Eq. 22)
// between electrode charge i (inverse width a_i) and point charge I (mixing
// width a_i). Split as in Eq. 20:
//   reciprocal  sum_K w_K [cos(K.r_i) Re S_K + sin(K.r_i) Im S_K],
//               S_K = sum_I q_I exp(i K.r_I)  (ion structure factor)
//   real space  sum_I q_I sum_{images, d < rcut} [erfc(beta d) - erfc(a_i d)] / d
//   background  -pi / (V beta^2) Q_sol,  Q_sol = sum_I q_I.
// Phases are evaluated from the fractional coordinate t = n . (r / L)
// reduced to [-1/2, 1/2] and sincospi(2t), all in FP64 (the structure
// factors' (n_x, n_y) phases by a table of 128 roots of unity and a short
// Taylor series, phase_cs); every sum runs in a fixed order (no atomics), so
// results are bitwise reproducible.
#include "cpm_internal.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

namespace cpm {
namespace {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int RB = 256;       // threads per block
constexpr int FG = 16;        // frames per thread in the back-projection
constexpr int BP_AT = 2;      // atoms per thread in the back-projection
constexpr int BP_KCH = 32;    // k-vectors per LDS chunk in the back-projection
constexpr double kErfcZero = 6.5;   // erfc(x) < 4e-20 beyond: below any FP64 sum it enters
static_assert(kErfcIntervals == kErfcPer * 6.5, "erfc table intervals up to kErfcZero");

// erfc(x) for 0 <= x from the table (0 for x >= kErfcZero): interval j =
// floor(16 x), u = 16 x - (j + 1/2) in [-1/2, 1/2), Horner. Every lane runs
// the same instructions (no range branches); absolute error below 1.2e-16
// (twelve Taylor terms on intervals of 1/8: 1.2e-16 too, a third more reads).
// Rows of nine doubles start in all banks of LDS.
__device__ inline double erfc_pw(const double *tab, double x) {
  const double s = kErfcPer * fmin(x, kErfcZero);
  const int j = min((int)s, kErfcIntervals - 1);
  const double u = s - ((double)j + 0.5);
  const double *c = tab + j * kErfcTerms;
  double v = c[kErfcTerms - 1];
#pragma unroll
  for (int k = kErfcTerms - 2; k >= 0; --k) v = fma(v, u, c[k]);
  return x < kErfcZero ? v : 0.0;
}

__global__ void fill_zero_kernel(double *__restrict__ v, int64_t len) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < len) v[i] = 0.0;
}

// Q_sol[f] = sum_I q_I; with m1 != null also M1[f] = sum_I q_I z_I (z in [0, L_z)),
// the ion dipole that the slab correction needs.
__global__ __launch_bounds__(RB) void qsum_kernel(const double *__restrict__ q, int64_t m,
                                                  double *__restrict__ qsol,
                                                  const double *__restrict__ ion_pos, double lz,
                                                  double *__restrict__ m1) {
  __shared__ double red[2][RB];
  const int64_t f = blockIdx.x;
  double acc = 0.0, dip = 0.0;
  for (int64_t I = threadIdx.x; I < m; I += RB) {
    const double qi = q[f * m + I];
    acc += qi;
    if (m1 != nullptr) {
      const double z = ion_pos[(f * m + I) * 3 + 2];
      dip += qi * (z - lz * floor(z / lz));
    }
  }
  red[0][threadIdx.x] = acc;
  red[1][threadIdx.x] = dip;
  __syncthreads();
  for (int s = RB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      red[0][threadIdx.x] += red[0][threadIdx.x + s];
      red[1][threadIdx.x] += red[1][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    qsol[f] = red[0][0];
    if (m1 != nullptr) m1[f] = red[1][0];
  }
}

// Ion structure factors of one group of ions, S_fK = sum_I q_I exp(i K.r_I).
// One thread per (run, frame): a run is up to kRun vectors of one (n_x, n_y)
// column with consecutive n_z. The phase of the run's first vector is
// evaluated directly (sincospi of the fractional phase), the second by one
// complex product with exp(2 pi i z_I / L_z), the following ones by the
// three-term recurrence of the cosine and sine, so kRun vectors cost one
// sincospi and about kRun FMAs per part and ion. Ions stream through LDS.
// Output layout: Sg[(g * nk * f_total + k * sk + f * sf) * 2 + {0: Re, 1: Im}].
__global__ __launch_bounds__(RB) void structure_factor_kernel(
    const double *__restrict__ ion_pos, const double *__restrict__ ion_q, int64_t m, int64_t ipg,
    const int32_t *__restrict__ kinfo, const int32_t *__restrict__ runs, int64_t nruns,
    int64_t nk, double inv_lx, double inv_ly, double inv_lz, int64_t f_total, int64_t sk,
    int64_t sf, double *__restrict__ Sg) {
  __shared__ double su[RB][6];   // x/L, y/L, z/L, q, cos and sin of 2 pi z/L
  const int64_t f = blockIdx.y, g = blockIdx.z;
  const int64_t r = (int64_t)blockIdx.x * RB + threadIdx.x;
  int64_t k0 = 0;
  int len = 0;
  double nx = 0, ny = 0, nz = 0;
  if (r < nruns) {
    k0 = runs[2 * r];
    len = runs[2 * r + 1];
    nx = kinfo[4 * k0];
    ny = kinfo[4 * k0 + 1];
    nz = kinfo[4 * k0 + 2];
  }
  double ar[kRun], ai[kRun];
#pragma unroll
  for (int st = 0; st < kRun; ++st) ar[st] = ai[st] = 0.0;
  const double *pf = ion_pos + f * m * 3;
  const double *qf = ion_q + f * m;
  const int64_t i0 = g * ipg, i1 = min(m, i0 + ipg);
  for (int64_t base = i0; base < i1; base += RB) {
    const int64_t I = base + threadIdx.x;
    if (I < i1) {
      const double uz = pf[3 * I + 2] * inv_lz;
      su[threadIdx.x][0] = pf[3 * I] * inv_lx;
      su[threadIdx.x][1] = pf[3 * I + 1] * inv_ly;
      su[threadIdx.x][2] = uz;
      su[threadIdx.x][3] = qf[I];
      double zs, zc;
      sincospi(2.0 * (uz - rint(uz)), &zs, &zc);
      su[threadIdx.x][4] = zc;
      su[threadIdx.x][5] = zs;
    }
    __syncthreads();
    const int cnt = (int)((i1 - base) < RB ? (i1 - base) : RB);
    // two ions per pass: their phase evaluations and recurrences are
    // independent, so each thread keeps four FMA chains in flight; a missing
    // second ion (odd count) enters with q = 0
    for (int j = 0; j < cnt; j += 2) {
      const int j2 = (j + 1 < cnt) ? j + 1 : j;
      const double qb = (j + 1 < cnt) ? su[j2][3] : 0.0;
      double ta = nx * su[j][0] + ny * su[j][1] + nz * su[j][2];
      double tb = nx * su[j2][0] + ny * su[j2][1] + nz * su[j2][2];
      ta -= rint(ta);
      tb -= rint(tb);
      double sna, csa, snb, csb;
      sincospi(2.0 * ta, &sna, &csa);
      sincospi(2.0 * tb, &snb, &csb);
      const double qa = su[j][3];
      const double zca = su[j][4], zsa = su[j][5], zcb = su[j2][4], zsb = su[j2][5];
      // q exp(i (phi + s theta)) for s = 0, 1, ... by the three-term
      // recurrence x_{s+1} = 2 cos(theta) x_s - x_{s-1} (one FMA per part;
      // a rounding error made at step m enters step s with the factor
      // sin((s - m) theta) / sin(theta), at most s - m)
      double c0 = qa * csa, s0 = qa * sna;
      double c1 = c0 * zca - s0 * zsa, s1 = s0 * zca + c0 * zsa;
      double d0 = qb * csb, e0 = qb * snb;
      double d1 = d0 * zcb - e0 * zsb, e1 = e0 * zcb + d0 * zsb;
      const double tza = 2.0 * zca, tzb = 2.0 * zcb;
#pragma unroll
      for (int st = 0; st < kRun; st += 2) {
        ar[st] += c0 + d0;
        ai[st] += s0 + e0;
        ar[st + 1] += c1 + d1;
        ai[st + 1] += s1 + e1;
        c0 = fma(tza, c1, -c0);
        s0 = fma(tza, s1, -s0);
        d0 = fma(tzb, d1, -d0);
        e0 = fma(tzb, e1, -e0);
        c1 = fma(tza, c0, -c1);
        s1 = fma(tza, s0, -s1);
        d1 = fma(tzb, d0, -d1);
        e1 = fma(tzb, e0, -e1);
      }
    }
    __syncthreads();
  }
  if (r < nruns) {
    double *out = Sg + (g * nk * f_total + k0 * sk + f * sf) * 2;
#pragma unroll
    for (int st = 0; st < kRun; ++st)
      if (st < len) {
        out[st * sk * 2] = ar[st];
        out[st * sk * 2 + 1] = ai[st];
      }
  }
}

// Ion structure factors as a product on the FP64 matrix cores. With
// exp(i K.r) = exp(2 pi i (n_x x / L_x + n_y y / L_y)) exp(2 pi i n_z z / L_z)
// = P_c(r) Z_s(r)^(+-1) for the column c = (n_x, n_y) and s = |n_z|,
//   S(c, +s) = sum_I q_I P_c Z_s,   S(c, -s) = sum_I q_I P_c conj(Z_s).
// With q P = a + i b and Z = z + i w these are four real products over the
// ions, AZ = sum a z, BW = sum b w, AW = sum a w, BZ = sum b z:
//   S(c, +s) = (AZ - BW) + i (AW + BZ),  S(c, -s) = (AZ + BW) + i (BZ - AW),
// one pass over the ions for both signs of n_z. A workgroup takes 64
// columns (a wave each 16: the A operand rows) and NSB blocks of 16 s (the
// columns are sorted by their largest |n_z|; the body is compiled for each
// block count), and streams its ion group in chunks of SG_CH ions through
// two LDS buffers:
//   - table phase: the chunk's x / L_x, y / L_y, q and Z_s for s < 16 NSB,
//     eight threads per ion, each a run of 2 NSB consecutive s (Z_s0 by
//     sincospi of the reduced fractional phase, then Z_(s+1) = Z_s Z_1);
//     the raw positions were loaded into registers one chunk ahead;
//   - product phase: per step of 4 ions each lane forms its (column, ion)
//     entry of q P (phase_cs: a table of exp(2 pi i j / 128) and a short
//     Taylor series) and v_mfma_f64_16x16x4f64 accumulates the four
//     products for every s block.
// One barrier per chunk: the table of chunk c + 1 goes to the buffer that
// the product phase of chunk c - 1 read, and every wave has left that phase
// before the barrier of chunk c. Output: Sg as in structure_factor_kernel.
constexpr int SG_CH = 32;      // ions per LDS chunk
constexpr int SG_SB = 3;       // s blocks of 16 at most (|n_z| <= 47)

// LDS of one workgroup: two chunk buffers of Z tables (SG_CH ions x 16 NSB
// s values, sized for the largest NSB) and of x / L_x, y / L_y, q
constexpr int kTw = 128;        // entries of the table of exp(2 pi i j / kTw)
struct SfLds {
  double2 zt[2][SG_CH][16 * SG_SB];
  double su[2][SG_CH][3];
  double2 tw[kTw];
};

// (cos, sin) of 2 pi t without a library sincos: t = j / kTw + d with
// j = rint(kTw t) and |d| <= 1 / (2 kTw), and exp(2 pi i t) = exp(2 pi i j /
// kTw) exp(2 pi i d), the first factor from the table tw, the second from
// the Taylor series of cos(2 pi d) and sin(2 pi d) in d up to d^6 and d^7
// (|2 pi d| <= pi / 128: the first terms left out are below 4e-18). About
// a dozen FP64 operations, against about three times as many for sincospi;
// on this chip the FP64 vector work does not overlap the FP64 matrix-core
// products, so it adds to the kernel's time one for one.
constexpr double kTwoPi = 6.283185307179586;
constexpr double kC1 = -kTwoPi * kTwoPi / 2.0;
constexpr double kC2 = -kC1 * kTwoPi * kTwoPi / 12.0;
constexpr double kC3 = -kC2 * kTwoPi * kTwoPi / 30.0;
constexpr double kS1 = -kTwoPi * kTwoPi * kTwoPi / 6.0;
constexpr double kS2 = -kS1 * kTwoPi * kTwoPi / 20.0;
constexpr double kS3 = -kS2 * kTwoPi * kTwoPi / 42.0;
__device__ __forceinline__ void phase_cs(const double2 *tw, double t, double &c, double &s) {
  const double j = rint(t * kTw);
  const double d = fma(j, -1.0 / kTw, t);
  const double d2 = d * d;
  const double cd = fma(d2, fma(d2, fma(d2, kC3, kC2), kC1), 1.0);
  const double sd = d * fma(d2, fma(d2, fma(d2, kS3, kS2), kS1), kTwoPi);
  const double2 w = tw[(int)(int64_t)j & (kTw - 1)];
  c = fma(w.x, cd, -w.y * sd);
  s = fma(w.y, cd, w.x * sd);
}

template <int NSB>
__device__ __forceinline__ void sf_gemm_body(SfLds &L, const double *__restrict__ ion_pos,
                                             const double *__restrict__ ion_q, int64_t m,
                                             int64_t ipg, const int4 *__restrict__ kcol,
                                             int64_t cbase, int64_t f, int64_t g, double inv_lx,
                                             double inv_ly, double inv_lz, int64_t nk,
                                             int64_t f_total, int64_t sk, int64_t sf,
                                             double *__restrict__ Sg) {
  constexpr int NS = 16 * NSB;        // s values of the tables
  constexpr int PER = NS / 8;         // s values per table thread
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int lr = lane & 15, lg = lane >> 4;
  const int4 mycol = kcol[cbase + wave * 16 + lr];
  const double cnx = (double)mycol.x, cny = (double)mycol.y;
  d4 acc[NSB][4];
#pragma unroll
  for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
    for (int p = 0; p < 4; ++p) acc[sb][p] = d4{0.0, 0.0, 0.0, 0.0};
  const double *pf = ion_pos + f * m * 3;
  const double *qf = ion_q + f * m;
  const int64_t i0 = g * ipg, i1 = min(m, i0 + ipg);
  const int nchunks = (int)((i1 - i0 + SG_CH - 1) / SG_CH);
  // table thread: ion ti of the chunk, run tj of s values
  const int ti = tid >> 3, tj = tid & 7;
  double rx = 0.0, ry = 0.0, rz = 0.0, rq = 0.0;   // raw data of the next chunk
  auto fetch = [&](int c) {
    const int64_t I = i0 + (int64_t)c * SG_CH + ti;
    rx = ry = rz = rq = 0.0;   // missing ions: q = 0 (and Z = 1)
    if (I < i1) {
      rx = pf[3 * I];
      ry = pf[3 * I + 1];
      rz = pf[3 * I + 2];
      rq = qf[I];
    }
  };
  auto table = [&](int buf) {
    const double uz = rz * inv_lz;
    if (tj == 0) {
      L.su[buf][ti][0] = rx * inv_lx;
      L.su[buf][ti][1] = ry * inv_ly;
      L.su[buf][ti][2] = rq;
    }
    double t = (double)(tj * PER) * uz;
    t -= rint(t);
    double sn, cs;
    phase_cs(L.tw, t, cs, sn);
    L.zt[buf][ti][tj * PER] = make_double2(cs, sn);
    if (PER > 1) {
      double t1 = uz - rint(uz), s1, c1;
      phase_cs(L.tw, t1, c1, s1);
#pragma unroll
      for (int u = 1; u < PER; ++u) {
        const double c2 = cs * c1 - sn * s1;
        sn = sn * c1 + cs * s1;
        cs = c2;
        L.zt[buf][ti][tj * PER + u] = make_double2(cs, sn);
      }
    }
  };
  // the exp(2 pi i j / kTw) table
  if (tid < kTw) {
    double sj, cj;
    sincospi(2.0 * (double)tid / kTw, &sj, &cj);
    L.tw[tid] = make_double2(cj, sj);
  }
  if (nchunks > 0) fetch(0);
  __syncthreads();
  if (nchunks > 0) {
    table(0);
  }
  for (int c = 0; c < nchunks; ++c) {
    const int buf = c & 1;
    __syncthreads();
    if (c + 1 < nchunks) fetch(c + 1);   // in flight during the products
#pragma unroll 2
    for (int ks = 0; ks < SG_CH / 4; ++ks) {
      const int ion = ks * 4 + lg;
      double2 z[NSB];
#pragma unroll
      for (int sb = 0; sb < NSB; ++sb) z[sb] = L.zt[buf][ion][sb * 16 + lr];
      double sn, cs;
      phase_cs(L.tw, cnx * L.su[buf][ion][0] + cny * L.su[buf][ion][1], cs, sn);
      const double q = L.su[buf][ion][2];
      const double a = q * cs, b = q * sn;
#pragma unroll
      for (int sb = 0; sb < NSB; ++sb) {
        acc[sb][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, z[sb].x, acc[sb][0], 0, 0, 0);
        acc[sb][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(b, z[sb].y, acc[sb][1], 0, 0, 0);
        acc[sb][2] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, z[sb].y, acc[sb][2], 0, 0, 0);
        acc[sb][3] = __builtin_amdgcn_mfma_f64_16x16x4f64(b, z[sb].x, acc[sb][3], 0, 0, 0);
      }
    }
    if (c + 1 < nchunks) table(buf ^ 1);
  }
  // D[i][j] (column i, s = j of the block) in lane j + 16 (i % 4), register i / 4
#pragma unroll
  for (int sb = 0; sb < NSB; ++sb) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int4 col = kcol[cbase + wave * 16 + 4 * v + lg];
      const int sv = sb * 16 + lr;
      if (col.z < 0 || sv > col.z) continue;
      const double AZ = acc[sb][0][v], BW = acc[sb][1][v], AW = acc[sb][2][v],
                   BZ = acc[sb][3][v];
      const bool half = col.x == 0 && col.y == 0;   // n_z = 1..m only
      if (!(half && sv == 0)) {
        double *o = Sg + (g * nk * f_total + (col.w + sv) * sk + f * sf) * 2;
        o[0] = AZ - BW;
        o[1] = AW + BZ;
      }
      if (!half && sv > 0) {
        double *o = Sg + (g * nk * f_total + (col.w - sv) * sk + f * sf) * 2;
        o[0] = AZ + BW;
        o[1] = BZ - AW;
      }
    }
  }
}

// One launch for every tile: grid (frames * ion groups, tiles), so that the
// dispatch order starts with the first tiles (the most s blocks, the longest
// workgroups) and ends with the tiles of one s block; the s-block count of a
// tile is set by its first column (the columns are sorted by their largest
// |n_z|) and selects the body compiled for it.
__global__ __launch_bounds__(256, 2) void sf_gemm_kernel(
    const double *__restrict__ ion_pos, const double *__restrict__ ion_q, int64_t m, int64_t ipg,
    const int4 *__restrict__ kcol, double inv_lx, double inv_ly, double inv_lz, int64_t nk,
    int64_t f_total, int64_t sk, int64_t sf, double *__restrict__ Sg) {
  __shared__ SfLds L;
  const int64_t f = blockIdx.x % f_total, g = blockIdx.x / f_total;
  const int64_t cbase = (int64_t)blockIdx.y * kSfTile;
  const int nsb = (kcol[cbase].z + 16) / 16;
  if (nsb >= 3)
    sf_gemm_body<3>(L, ion_pos, ion_q, m, ipg, kcol, cbase, f, g, inv_lx, inv_ly, inv_lz, nk,
                    f_total, sk, sf, Sg);
  else if (nsb == 2)
    sf_gemm_body<2>(L, ion_pos, ion_q, m, ipg, kcol, cbase, f, g, inv_lx, inv_ly, inv_lz, nk,
                    f_total, sk, sf, Sg);
  else
    sf_gemm_body<1>(L, ion_pos, ion_q, m, ipg, kcol, cbase, f, g, inv_lx, inv_ly, inv_lz, nk,
                    f_total, sk, sf, Sg);
}

// ---- ion structure factors through a grid (non-uniform FFT of type 1)
//
// The direct product costs 4 n_k M flops per frame. For many ions and
// vectors the same sums come cheaper from a regular grid: with phi the
// "exponential of semicircle" window exp(beta (sqrt(1 - (2 t / w)^2) - 1)),
// |t| < w / 2 (Barnett, Magland, af Klinteberg, SIAM J. Sci. Comput. 41,
// C479 (2019)),
//   g[j] = sum_I q_I prod_d phi(j_d - u_Id),  u = r G / L,
//   S_K  = sum_j g[j] exp(2 pi i sum_d n_d j_d / G_d) / prod_d Phi_d(n_d),
// Phi_d(n) = integral of phi(t) cos(2 pi n t / G_d). With w = 16, beta =
// 36.8 and G at least 2 (2 n_max + 1) the aliasing error is 2e-15 of |S|,
// below the rounding error of the direct sum's phases (5e-15): measured in
// long double for n_max 27..48. Every sum runs in a fixed order.
//
// nu_spread_kernel: one wave per 16^3 grid points and frame. The ions that
//   reach the tile are taken from the cell list in order (filtered by
//   ballot), 32 at a time; each ion's 3 x 16 window values (polynomials in
//   its offset, coefficients in registers) go to LDS, and the tile is the
//   product sum_I [q phi_x phi_y] phi_z on the FP64 matrix cores: 16 row
//   blocks (one y each, rows x) of v_mfma_f64_16x16x4f64. An ion reaches 8
//   tiles, so 7/8 of the products are with zeros; that is still 65.5 kflop
//   per ion against 4 n_k (482 kflop for 120 000 vectors).
//   A step of 4 ions multiplies only the y that one of them reaches (the
//   cell list keeps ions of about one y together: 11 of 16 on average),
//   positions are scaled by reciprocals, and the window's points l and 15 - l
//   share the even and odd parts of one polynomial (they are mirror images):
//   50000 ions, 8 frames 750 us without these, 587 now, of which 205 are
//   matrix-core products and 110 vector instructions.
// nu_dftz_kernel, nu_dfty_kernel, nu_dftx_kernel: the three transforms, each
//   a product with a dense (cos, sin) matrix on the FP64 matrix cores that
//   computes only the wanted n (z: n >= 0; y and x: both signs from the same
//   four real products) and any G; the transform axis of each result is
//   written as the contiguous axis of the next.
// nu_dftx_kernel divides by Phi and writes S in the k-vector order (the half
//   space; S(-K) = conj(S(K))).
// 50 000 ions x 32 frames, 120 500 vectors (box 79 x 136 x 120 A): structure
// factors 19.0 -> 4.3 ms; 20 000 ions x 64 frames: 15.6 -> 5.6 ms. Error of b
// against the same sums in long double at 2592 atoms, 12 000 ions and 38 000
// vectors: 6.7e-16 of max|b|, with the direct product 1.0e-15.
constexpr int NU_W = 16;              // support of the window (grid points)
constexpr int NU_DEG = 13;            // degree of its polynomials per interval
constexpr double NU_BETA = 2.3 * NU_W;
constexpr int NU_T = 16;              // edge of a grid tile
constexpr int NU_CH = 32;             // ions per table
constexpr int NU_RZ = 6;              // row blocks of the z transform per wave
constexpr int NU_K2 = 2;              // blocks of n of the y and x transforms per wave

__device__ inline void cell_span(double lo, double hi, double invh, int nc, int &a, int &b);
__device__ inline int wrap_cell(int c, int nc);

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void nu_spread_kernel(
    const double4 *__restrict__ sorted, const int32_t *__restrict__ cstart, int64_t m, int ncx,
    int ncy, int ncz, double lx, double ly, double lz, int gx, int gy, int gz,
    const double *__restrict__ coef, double *__restrict__ grid) {
  __shared__ double lst[4][NU_CH + 64];   // (x, y, z) in grid points from the tile's origin, q
  __shared__ double tab[3][NU_CH][NU_T + 2];
  __shared__ unsigned rows[NU_CH / 4];   // the y of the tile that a step's ions reach
  const int lane = threadIdx.x, lr = lane & 15, lg = lane >> 4;
  int t = blockIdx.x;
  const int oz = t % (gz / NU_T) * NU_T;
  t /= gz / NU_T;
  const int oy = t % (gy / NU_T) * NU_T, ox = t / (gy / NU_T) * NU_T;
  const int64_t f = blockIdx.y;
  // window polynomial of support point l8; point 15 - l8 has its mirror image
  const int l8 = lane & 7, li = lane >> 3;
  double cf[NU_DEG + 1];
#pragma unroll
  for (int d = 0; d <= NU_DEG; ++d) cf[d] = coef[l8 * (NU_DEG + 1) + d];
  d4 acc[NU_T];
#pragma unroll
  for (int r = 0; r < NU_T; ++r) acc[r] = d4{0.0, 0.0, 0.0, 0.0};
  // cells that hold ions within w / 2 of the tile (and a hair)
  const double hx = lx / gx, hy = ly / gy, hz = lz / gz;
  constexpr double kLo = -0.5 * NU_W - 1e-6, kHi = NU_T - 1 + 0.5 * NU_W + 1e-6;
  int xa, xb, ya, yb, za, zb;
  cell_span((ox + kLo) * hx, (ox + kHi) * hx, ncx / lx, ncx, xa, xb);
  cell_span((oy + kLo) * hy, (oy + kHi) * hy, ncy / ly, ncy, ya, yb);
  cell_span((oz + kLo) * hz, (oz + kHi) * hz, ncz / lz, ncz, za, zb);
  const int32_t *cs = cstart + f * ((int64_t)ncx * ncy * ncz + 1);
  const double4 *sf = sorted + f * m;
  const int xlen = xb - xa + 1, xw0 = wrap_cell(xa, ncx);
  // the ion's coordinate from the tile's origin, nearest image to its centre
  const double ilx = 1.0 / lx, ily = 1.0 / ly, ilz = 1.0 / lz;
  const double igx = 1.0 / gx, igy = 1.0 / gy, igz = 1.0 / gz;
  auto local = [&](double x, double il, double g, double ig, int o) {
    double w = x * il;
    w -= floor(w);
    const double u = w * g - o;
    return u - g * rint((u - 7.5) * ig);
  };
  // the product of the first `cnt` listed ions, cnt <= NU_CH (padded with q = 0)
  auto flush = [&](int cnt) {
    const int steps = (cnt + 3) >> 2, pairs = (cnt + 7) >> 3;
    if (lane < 8 * pairs && lane >= cnt) {
      lst[0][lane] = lst[2][lane] = 7.5;
      lst[1][lane] = 1000.0;   // reaches no y
      lst[3][lane] = 0.0;
    }
    __syncthreads();
    for (int s = 0; s < pairs; ++s) {
      const int ion = 8 * s + li;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        // support point l is grid point j = i0 + l; the 16 j fill the 16
        // slots j mod 16, those outside the tile with 0 (a position that is
        // not a number stays one)
        const double u = lst[d][ion], i0 = ceil(u - 0.5 * NU_W);
        const double x = 2.0 * (i0 - (u - 0.5 * NU_W)) - 1.0, x2 = x * x;
        double ev = cf[NU_DEG - 1], od = cf[NU_DEG];   // even and odd part
#pragma unroll
        for (int e = NU_DEG - 3; e >= 0; e -= 2) {
          ev = fma(ev, x2, cf[e]);
          od = fma(od, x2, cf[e + 1]);
        }
        if (d == 1) {
          const double q = lst[3][ion];
          ev *= q;
          od *= q;
          const int i = (int)fmin(fmax(i0, -16.0), 16.0);
          unsigned m = u != u ? 0xffffu : (i < 0 ? 0xffffu >> -i : (0xffffu << i) & 0xffffu);
          m |= __shfl_xor(m, 8, 64);
          m |= __shfl_xor(m, 16, 64);
          if ((lane & 31) == 0) rows[2 * s + (lane >> 5)] = m;
        }
        const int ja = (int)i0 + l8, jb = (int)i0 + 15 - l8;
        const bool nan = u != u;
        tab[d][ion][ja & (NU_T - 1)] = ((unsigned)ja < (unsigned)NU_T) | nan ? fma(od, x, ev) : 0.0;
        tab[d][ion][jb & (NU_T - 1)] = ((unsigned)jb < (unsigned)NU_T) | nan ? fma(-od, x, ev) : 0.0;
      }
    }
    __syncthreads();
    for (int s = 0; s < steps; ++s) {
      const int ion = 4 * s + lg;
      const double fx = tab[0][ion][lr], fz = tab[2][ion][lr];
      d2 fy[NU_T / 2];
#pragma unroll
      for (int r = 0; r < NU_T / 2; ++r) fy[r] = *reinterpret_cast<const d2 *>(&tab[1][ion][2 * r]);
      const unsigned m = __builtin_amdgcn_readfirstlane(rows[s]);
#pragma unroll
      for (int r = 0; r < NU_T; ++r)
        if (m >> r & 1)
          acc[r] = __builtin_amdgcn_mfma_f64_16x16x4f64(fx * fy[r / 2][r & 1], fz, acc[r], 0, 0, 0);
    }
    __syncthreads();
  };
  int cnt = 0;   // listed ions
  for (int cz = za; cz <= zb; ++cz) {
    const int czw = wrap_cell(cz, ncz);
    for (int cy = ya; cy <= yb; ++cy) {
      const int64_t row = ((int64_t)czw * ncy + wrap_cell(cy, ncy)) * ncx;
      for (int part = 0; part < 2; ++part) {
        const int c0 = part == 0 ? xw0 : 0, c1 = part == 0 ? min(ncx, xw0 + xlen) : xw0 + xlen - ncx;
        if (c1 <= c0) break;
        const int64_t s0 = cs[row + c0], s1 = cs[row + c1];
        for (int64_t base = s0; base < s1; base += 64) {
          const double4 ion = sf[min(base + lane, s1 - 1)];
          const double ux = local(ion.x, ilx, gx, igx, ox), uy = local(ion.y, ily, gy, igy, oy),
                       uz = local(ion.z, ilz, gz, igz, oz);
          constexpr double kReach = 0.5 * (NU_T - 1 + NU_W);   // |u - 7.5| below this
          const bool in = base + lane < s1 && !(fabs(ux - 7.5) >= kReach) &&
                          !(fabs(uy - 7.5) >= kReach) && !(fabs(uz - 7.5) >= kReach);
          const uint64_t mask = __ballot(in);
          if (in) {
            const int at = cnt + __popcll(mask & ((1ull << lane) - 1));
            lst[0][at] = ux;
            lst[1][at] = uy;
            lst[2][at] = uz;
            lst[3][at] = ion.w;
          }
          cnt += __popcll(mask);
          while (cnt >= NU_CH) {
            flush(NU_CH);
            // the rest to the front (at most 63 entries, one per lane)
            double k0 = 0, k1 = 0, k2 = 0, k3 = 0;
            cnt -= NU_CH;
            if (lane < cnt) {
              k0 = lst[0][NU_CH + lane];
              k1 = lst[1][NU_CH + lane];
              k2 = lst[2][NU_CH + lane];
              k3 = lst[3][NU_CH + lane];
            }
            __syncthreads();
            if (lane < cnt) {
              lst[0][lane] = k0;
              lst[1][lane] = k1;
              lst[2][lane] = k2;
              lst[3][lane] = k3;
            }
            __syncthreads();
          }
        }
      }
    }
  }
  if (cnt > 0) flush(cnt);
  // acc[r][v]: grid point (x = 4 v + lg, y = r, z = lr) of the tile
#pragma unroll
  for (int r = 0; r < NU_T; ++r)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      grid[((f * gx + ox + 4 * v + lg) * gy + oy + r) * gz + oz + lr] = acc[r][v];
}

// z transform: out[f][n][part][x][y] = sum_z grid[f][x][y][z] (cos, sin)(2 pi n z / gz),
// row 2 n + part of the matrix. Wave: 32 consecutive (x, y) and RT blocks of
// 16 rows; lane (lr, lg) takes k = 16 st + 4 lg + t of both operands, the
// next 16 k loaded during the products.
template <int RT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void nu_dftz_kernel(
    const double *__restrict__ grid, int64_t lines, int gz, const double *__restrict__ mat, int nz,
    double *__restrict__ out) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int64_t f = blockIdx.y, l0 = ((int64_t)blockIdx.x * 4 + wave) * 32;
  const int row0 = blockIdx.z * RT * 16;
  const double *B = grid + (f * lines + l0 + lr) * gz + 4 * lg;
  const double *A = mat + (int64_t)(row0 + lr) * gz + 4 * lg;
  const int64_t step = (int64_t)16 * gz;
  d4 a[2][RT], b[2][2], acc[RT][2];
#pragma unroll
  for (int i = 0; i < RT; ++i) acc[i][0] = acc[i][1] = d4{0.0, 0.0, 0.0, 0.0};
  auto load = [&](auto buf, int k) {
#pragma unroll
    for (int i = 0; i < RT; ++i) a[buf.value][i] = *reinterpret_cast<const d4 *>(A + i * step + k);
#pragma unroll
    for (int i = 0; i < 2; ++i) b[buf.value][i] = *reinterpret_cast<const d4 *>(B + i * step + k);
  };
  auto mul = [&](auto buf) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[buf.value][i][q], b[buf.value][j][q],
                                                           acc[i][j], 0, 0, 0);
  };
  const std::integral_constant<int, 0> even;
  const std::integral_constant<int, 1> odd;
  load(even, 0);
  for (int k = 0; k < gz; k += 32) {
    load(odd, min(k + 16, gz - 16));
    __builtin_amdgcn_sched_barrier(0);
    mul(even);
    load(even, min(k + 32, gz - 16));
    __builtin_amdgcn_sched_barrier(0);
    if (k + 16 < gz) mul(odd);
  }
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = row0 + i * 16 + 4 * v + lg;
      if (row < 2 * nz) {
        double *o = out + (f * 2 * nz + row) * lines + l0 + lr;
        o[0] = acc[i][0][v];
        o[16] = acc[i][1][v];
      }
    }
}

// One wave's products of the y and x transforms: NU_K2 blocks of 16 n >= 0
// (cos rows at C, sin rows at C + sin_off) with 16 complex lines (real parts
// at re, imaginary at im), contraction length g (a multiple of 16):
// acc[i][0..3] = sum re cos, sum im sin, sum re sin, sum im cos.
__device__ __forceinline__ void nu_products(const double *C, int64_t sin_off, const double *re,
                                            const double *im, int g, d4 (&acc)[NU_K2][4]) {
  d4 c[2][NU_K2], s[2][NU_K2], x[2], y[2];
  const int64_t step = (int64_t)16 * g;
  auto load = [&](auto buf, int k) {
#pragma unroll
    for (int i = 0; i < NU_K2; ++i) {
      c[buf.value][i] = *reinterpret_cast<const d4 *>(C + i * step + k);
      s[buf.value][i] = *reinterpret_cast<const d4 *>(C + sin_off + i * step + k);
    }
    x[buf.value] = *reinterpret_cast<const d4 *>(re + k);
    y[buf.value] = *reinterpret_cast<const d4 *>(im + k);
  };
  auto mul = [&](auto buf) {
    constexpr int b = decltype(buf)::value;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < NU_K2; ++i) {
        acc[i][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[b][i][q], x[b][q], acc[i][0], 0, 0, 0);
        acc[i][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(s[b][i][q], y[b][q], acc[i][1], 0, 0, 0);
        acc[i][2] = __builtin_amdgcn_mfma_f64_16x16x4f64(s[b][i][q], x[b][q], acc[i][2], 0, 0, 0);
        acc[i][3] = __builtin_amdgcn_mfma_f64_16x16x4f64(c[b][i][q], y[b][q], acc[i][3], 0, 0, 0);
      }
  };
  const std::integral_constant<int, 0> even;
  const std::integral_constant<int, 1> odd;
#pragma unroll
  for (int i = 0; i < NU_K2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[i][q] = d4{0.0, 0.0, 0.0, 0.0};
  load(even, 0);
  for (int k = 0; k < g; k += 32) {
    load(odd, min(k + 16, g - 16));
    __builtin_amdgcn_sched_barrier(0);
    mul(even);
    load(even, min(k + 32, g - 16));
    __builtin_amdgcn_sched_barrier(0);
    if (k + 16 < g) mul(odd);
  }
}

// y transform: out[f][nz][ny][part][x] from in[f][nz][part][x][y]; wave: 16 x,
// one n_z, a pass of NU_K2 blocks of n_y >= 0 (both signs written). Grid
// (waves / 4, frames); waves = gx / 16 * passes * nz.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 3))) void nu_dfty_kernel(
    const double *__restrict__ in, int gx, int gy, int nz, int my, int passes,
    const double *__restrict__ mat, double *__restrict__ out) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), f = blockIdx.y;
  const int xt = (int)(w % (gx / 16)), pass = (int)(w / (gx / 16) % passes);
  const int64_t kz = w / ((int64_t)(gx / 16) * passes);
  if (kz >= nz) return;   // no barriers: a wave may leave alone
  const double *re = in + (((f * nz + kz) * 2) * gx + xt * 16 + lr) * (int64_t)gy + 4 * lg;
  const int n0 = pass * NU_K2 * 16, ny = 2 * my + 1;
  d4 acc[NU_K2][4];
  nu_products(mat + (int64_t)(n0 + lr) * gy + 4 * lg, (int64_t)passes * NU_K2 * 16 * gy, re,
              re + (int64_t)gx * gy, gy, acc);
  double *o = out + ((f * nz + kz) * ny + my) * 2 * gx + xt * 16 + lr;
#pragma unroll
  for (int i = 0; i < NU_K2; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int n = n0 + i * 16 + 4 * v + lg;
      if (n > my) continue;
      const double ac = acc[i][0][v], bs = acc[i][1][v], as = acc[i][2][v], bc = acc[i][3][v];
      double *a = o + (int64_t)n * 2 * gx, *b = o - (int64_t)n * 2 * gx;
      a[0] = ac - bs;
      a[gx] = as + bc;
      if (n > 0) {
        b[0] = ac + bs;
        b[gx] = bc - as;
      }
    }
}

// x transform of in[f][nz][ny][part][x], division by the windows' transforms
// and S[k][frame]: wave: 16 n_y, one n_z, a pass of NU_K2 blocks of n_x >= 0.
// col[n_x * ny + n_y + my] = (k index of n_z = 0, largest |n_z|) of the
// half-space columns (largest -1: none). inv: 1 / Phi_x, 1 / Phi_y, 1 / Phi_z
// at 0, off_y, off_z.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 3))) void nu_dftx_kernel(
    const double *__restrict__ in, int gx, int nz, int mx, int my, int passes,
    const double *__restrict__ mat, const double *__restrict__ inv, int off_y, int off_z,
    const int2 *__restrict__ col, int64_t f0, int64_t f_total, double *__restrict__ S) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int ny = 2 * my + 1, tiles = (ny + 15) / 16;
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), f = blockIdx.y;
  const int yt = (int)(w % tiles), pass = (int)(w / tiles % passes);
  const int64_t kz = w / ((int64_t)tiles * passes);
  if (kz >= nz) return;   // no barriers: a wave may leave alone
  const int yi = yt * 16 + lr, n0 = pass * NU_K2 * 16;
  const double *re = in + ((f * nz + kz) * ny + min(yi, ny - 1)) * 2 * gx + 4 * lg;
  d4 acc[NU_K2][4];
  nu_products(mat + (int64_t)(n0 + lr) * gx + 4 * lg, (int64_t)passes * NU_K2 * 16 * gx, re,
              re + gx, gx, acc);
  if (yi >= ny) return;
  const int n_y = yi - my, n_z = (int)kz;
  const double iyz = inv[off_y + (n_y < 0 ? -n_y : n_y)] * inv[off_z + n_z];
  auto put = [&](int64_t k, double re_, double im_) {
    double *o = S + (k * f_total + f0 + f) * 2;
    o[0] = re_;
    o[1] = im_;
  };
#pragma unroll
  for (int i = 0; i < NU_K2; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int n = n0 + i * 16 + 4 * v + lg;
      if (n > mx) continue;
      const double ac = acc[i][0][v], bs = acc[i][1][v], as = acc[i][2][v], bc = acc[i][3][v];
      const double wgt = inv[n] * iyz;
      // S(n, n_y, n_z), or for n = 0, n_y < 0 its conjugate S(0, -n_y, -n_z)
      const bool own = n > 0 || n_y > 0 || (n_y == 0 && n_z > 0);
      const int2 c = col[n * ny + my + (own ? n_y : -n_y)];
      if (n_z <= c.y && (own || n_z > 0))
        put(own ? (int64_t)c.x + n_z : (int64_t)c.x - n_z, (ac - bs) * wgt,
            (own ? as + bc : -(as + bc)) * wgt);
      // S(-n, n_y, n_z) = conj S(n, -n_y, -n_z)
      if (n > 0 && n_z > 0) {
        const int2 d = col[n * ny + my - n_y];
        if (n_z <= d.y) put((int64_t)d.x - n_z, (ac + bs) * wgt, -(bc - as) * wgt);
      }
    }
}

// S[k][f] = sum_g Sg[g][f][k] over the ion groups (fixed order). The groups
// are written by frame, where the k-vectors of a column are contiguous, and
// read by k-vector, where the frames are: 32 vectors by 16 frames per
// workgroup through LDS. (Written as [k][f], every 16-byte value of a group
// was a line of its own: 13 frames of 1999 ions with 17 groups, 93 us for the
// product then, 80 now.)
constexpr int SGT_K = 32, SGT_F = 16;
__global__ __launch_bounds__(256) void sum_groups_kernel(const double2 *__restrict__ Sg,
                                                         int groups, int64_t nk, int64_t f_total,
                                                         double2 *__restrict__ S) {
  __shared__ double2 t[SGT_F][SGT_K + 1];
  const int64_t k0 = (int64_t)blockIdx.x * SGT_K, f0 = (int64_t)blockIdx.y * SGT_F;
  const int kk = threadIdx.x % SGT_K;
#pragma unroll
  for (int h = 0; h < SGT_F * SGT_K / 256; ++h) {
    const int ff = threadIdx.x / SGT_K + h * (256 / SGT_K);
    const int64_t k = min(k0 + kk, nk - 1), f = min(f0 + ff, f_total - 1);
    const double2 *src = Sg + f * nk + k;
    double re = 0.0, im = 0.0;
#pragma unroll 4
    for (int g = 0; g < groups; ++g) {
      const double2 v = src[(int64_t)g * nk * f_total];
      re += v.x;
      im += v.y;
    }
    t[ff][kk] = make_double2(re, im);
  }
  __syncthreads();
  const int nf = (int)min((int64_t)SGT_F, f_total - f0);
  for (int e = threadIdx.x; e < SGT_K * nf; e += 256) {
    const int k = e / nf, f = e - k * nf;
    if (k0 + k < nk) S[(k0 + k) * f_total + f0 + f] = t[f][k];
  }
}

// Back-projection of the ion structure factors onto the electrode atoms,
// split over k ranges: part[ks][f][i] = sum_{K in range ks} w_K (c_iK Re S_fK
// + s_iK Im S_fK). Each thread takes AT atoms (i = block base + thread +
// RB a) and FG frames; K data and S_f.K of BP_KCH vectors at a time are
// staged in LDS and read by all lanes at the same address. The phase of
// (i, K) is evaluated directly at the start of every run (and of the range)
// and by the n_z recurrence inside a run. Grid (atom blocks, k splits,
// frame groups).
template <int AT>
__global__ __launch_bounds__(RB) void backproject_kernel(
    const double *__restrict__ pos, int64_t n, const int32_t *__restrict__ kinfo,
    const double *__restrict__ kw, int64_t nk, int64_t kper, double inv_lx, double inv_ly,
    double inv_lz, const double *__restrict__ S, int64_t f_total, double *__restrict__ part) {
  __shared__ int4 sk[BP_KCH];
  __shared__ double sw[BP_KCH];
  __shared__ double2 ss[BP_KCH][FG];
  const int64_t ibase = (int64_t)blockIdx.x * RB * AT + threadIdx.x;
  const int64_t kbeg = (int64_t)blockIdx.y * kper;
  const int64_t kend = min(nk, kbeg + kper);
  const int64_t f0 = (int64_t)blockIdx.z * FG;
  const int nf = (int)((f_total - f0) < FG ? (f_total - f0) : FG);
  double ux[AT], uy[AT], uz[AT], zs[AT], zc[AT], cs[AT], sn[AT];
#pragma unroll
  for (int a = 0; a < AT; ++a) {
    const int64_t i = ibase + RB * a;
    ux[a] = uy[a] = uz[a] = 0.0;
    if (i < n) {
      ux[a] = pos[3 * i] * inv_lx;
      uy[a] = pos[3 * i + 1] * inv_ly;
      uz[a] = pos[3 * i + 2] * inv_lz;
    }
    sincospi(2.0 * (uz[a] - rint(uz[a])), &zs[a], &zc[a]);
    cs[a] = 1.0;
    sn[a] = 0.0;
  }
  double acc[AT][FG];
#pragma unroll
  for (int a = 0; a < AT; ++a)
#pragma unroll
    for (int g = 0; g < FG; ++g) acc[a][g] = 0.0;
  const int4 *ki4 = reinterpret_cast<const int4 *>(kinfo);
  for (int64_t k0 = kbeg; k0 < kend; k0 += BP_KCH) {
    const int cnt = (int)((kend - k0) < BP_KCH ? (kend - k0) : BP_KCH);
    for (int t = threadIdx.x; t < BP_KCH * FG; t += RB) {
      const int kk = t / FG, g = t % FG;
      double2 v = make_double2(0.0, 0.0);
      if (kk < cnt && g < nf) v = *reinterpret_cast<const double2 *>(S + ((k0 + kk) * f_total + f0 + g) * 2);
      ss[kk][g] = v;
    }
    if (threadIdx.x < cnt) {
      sk[threadIdx.x] = ki4[k0 + threadIdx.x];
      sw[threadIdx.x] = kw[k0 + threadIdx.x];
    }
    __syncthreads();
    for (int kk = 0; kk < cnt; ++kk) {
      const int4 ki = sk[kk];
      const double w = sw[kk];
      if (ki.w != 0 || k0 + kk == kbeg) {
#pragma unroll
        for (int a = 0; a < AT; ++a) {
          double t = (double)ki.x * ux[a] + (double)ki.y * uy[a] + (double)ki.z * uz[a];
          t -= rint(t);
          sincospi(2.0 * t, &sn[a], &cs[a]);
        }
      } else {
#pragma unroll
        for (int a = 0; a < AT; ++a) {
          const double c2 = cs[a] * zc[a] - sn[a] * zs[a];
          sn[a] = cs[a] * zs[a] + sn[a] * zc[a];
          cs[a] = c2;
        }
      }
      double wc[AT], ws[AT];
#pragma unroll
      for (int a = 0; a < AT; ++a) {
        wc[a] = w * cs[a];
        ws[a] = w * sn[a];
      }
#pragma unroll
      for (int g = 0; g < FG; ++g) {
        const double2 sv = ss[kk][g];
#pragma unroll
        for (int a = 0; a < AT; ++a) {
          acc[a][g] = fma(wc[a], sv.x, acc[a][g]);
          acc[a][g] = fma(ws[a], sv.y, acc[a][g]);
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int a = 0; a < AT; ++a) {
    const int64_t i = ibase + RB * a;
    if (i < n) {
#pragma unroll
      for (int g = 0; g < FG; ++g)
        if (g < nf) part[((int64_t)blockIdx.y * f_total + f0 + g) * n + i] = acc[a][g];
    }
  }
}

// Factored back-projection for electrode atoms in few thin layers. With
// exp(i K.r) = P_c(x, y) Z_nz(z), P_c = exp(2 pi i (n_x x / L_x + n_y y / L_y)),
// Z_nz = exp(2 pi i n_z z / L_z), for the column c = (n_x, n_y):
//   sum_K w_K Re(exp(-i K.r_i) S_fK) = sum_c Re(conj(P_c(r_i)) T_f(z_i, c)),
//   T_f(z, c) = sum_nz w_(c, nz) conj(Z_nz(z)) S_f(c, nz).
// The n_z sums are taken once per (node, column, frame) instead of once per
// atom: the node of an exact plane is its z; a layer of finite thickness D
// has nodes at the Chebyshev points of its z range, and
//   T_f(z_i, c) = sum_j l_j(z_i) T_f(z_j, c)
// with the Lagrange polynomials l_j. T is band-limited to k = 2 pi smax / L_z,
// so n nodes leave an error of at most 2 (k D / 4)^n / n! of the sum, below
// 1e-17 by the choice of n.
//
// layer_tables_kernel (system set-up): Z_s of every node, zt[s][node], and
// l_j of every tile's atoms, lw[tile offset + j][atom] (1 for an exact plane;
// the barycentric form, whose weights at the Chebyshev points are
// (-1)^j sin((j + 1/2) pi / n)).
__global__ void layer_tables_kernel(const double *__restrict__ pos, double inv_lz,
                                    const int4 *__restrict__ tile,
                                    const int32_t *__restrict__ tile_atom, int64_t ntiles,
                                    const double *__restrict__ node_z, int nodes, int nodes_pad,
                                    int smax, double2 *__restrict__ zt, double *__restrict__ lw) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nz = (int64_t)(smax + 1) * nodes_pad;
  if (e < nz) {
    const int64_t sv = e / nodes_pad;
    const int node = (int)(e - sv * nodes_pad);
    double sn = 0.0, cs = 0.0;
    if (node < nodes) {
      double t = (double)sv * (node_z[node] * inv_lz);
      t -= rint(t);
      sincospi(2.0 * t, &sn, &cs);
    }
    zt[e] = make_double2(cs, sn);
  }
  if (e < ntiles * kPlaneTile) {
    const int4 tl = tile[e / kPlaneTile];
    const int32_t a = tile_atom[e];
    const double z = a >= 0 ? pos[3 * (int64_t)a + 2] : node_z[tl.x];
    double *w = lw + (int64_t)tl.z * kPlaneTile + e % kPlaneTile;
    int hit = tl.y == 1 ? 0 : -1;
    double sum = 0.0;
    for (int j = 0; j < tl.y; ++j) {
      const double d = z - node_z[tl.x + j];
      if (d == 0.0) hit = j;
      const double q = (j & 1 ? -1.0 : 1.0) * sinpi((j + 0.5) / tl.y) / d;
      w[j * kPlaneTile] = q;
      sum += q;
    }
    for (int j = 0; j < tl.y; ++j)
      w[j * kPlaneTile] = hit < 0 ? w[j * kPlaneTile] / sum : (j == hit ? 1.0 : 0.0);
  }
}

// T as Re / Im arrays [node][column][frame] (zero for the padding columns):
// per column the product [nodes x n_z] . [n_z x frames] of conj(Z) and w S as
// four real products on the FP64 matrix cores. One wave per column, 16 nodes
// and 16 frames; every lane's loads are in bounds and unconditional (n_z
// beyond the column repeat its last with weight 0), so that they overlap.
// Bound by latency: a thread per (column, frame) and plane that walked n_z
// alone took 38 us where this takes 8 (one frame, 6 planes, 448 columns).
constexpr int PT_WAVES = 4;

__global__ __launch_bounds__(64 * PT_WAVES) void plane_table_kernel(
    const double2 *__restrict__ zt, int nodes, int nodes_pad, const int4 *__restrict__ kcol,
    int64_t ncols_pad, const double *__restrict__ kw, const double2 *__restrict__ S,
    int64_t f_total, double *__restrict__ Tre, double *__restrict__ Tim) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lq = lane >> 4;
  const int64_t c = (int64_t)blockIdx.x * PT_WAVES + wave;   // ncols_pad is a multiple
  const int node0 = blockIdx.y * 16;
  const int64_t f = (int64_t)blockIdx.z * 16 + lr, fc = min(f, f_total - 1);
  const int4 col = kcol[c];
  d4 re = d4{0.0, 0.0, 0.0, 0.0}, im = re;
  if (col.z >= 0) {
    // (0, 0) holds n_z = 1..m only
    const int lo = (col.x == 0 && col.y == 0) ? 1 : -col.z;
    const double2 *zn = zt + node0 + lr;
    for (int n0 = lo; n0 <= col.z; n0 += 16) {
      d2 sv[4], z[4];
      double wk[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int nz = min(n0 + 4 * u + lq, col.z);
        const int64_t k = (int64_t)col.w + nz;
        sv[u] = *reinterpret_cast<const d2 *>(S + k * f_total + fc);
        z[u] = *reinterpret_cast<const d2 *>(zn + (int64_t)abs(nz) * nodes_pad);
        wk[u] = kw[k];
      }
      __builtin_amdgcn_sched_barrier(0);   // every load issued before the first wait
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int nz = n0 + 4 * u + lq;
        const double w = nz > col.z ? 0.0 : wk[u];
        const double zr = z[u].x, zi = min(nz, col.z) < 0 ? -z[u].y : z[u].y;   // Z_nz
        const double sr = w * sv[u].x, si = w * sv[u].y;
        // conj(Z) S = (Re Z Re S + Im Z Im S) + i (Re Z Im S - Im Z Re S)
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(zr, sr, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(zr, si, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(zi, si, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(-zi, sr, im, 0, 0, 0);
      }
    }
  }
  // D[i][j] (node i, frame j) in lane j + 16 (i % 4), register i / 4
  if (f >= f_total) return;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int node = node0 + 4 * v + lq;
    if (node >= nodes) continue;
    const int64_t o = ((int64_t)node * ncols_pad + c) * f_total + f;
    Tre[o] = re[v];
    Tim[o] = im[v];
  }
}

// part[f][i] = sum_c cos(theta_ic) Re T_f(z_i, c) + sin(theta_ic) Im T_f(z_i, c),
// theta_ic = 2 pi (n_x x_i / L_x + n_y y_i / L_y): the product
// [frames x (nodes of the columns)] . [l_j (cos, sin) x atoms] on the FP64
// matrix cores. One wave per tile of kPlaneTile atoms of one layer and up to
// 16 NF frames: per step of 4 columns, lane (r, q) forms the phase of atom r
// and column q once; per node its l_j multiples are the B operand and Re T
// and Im T of (column q, frame r) the A operand of two
// v_mfma_f64_16x16x4f64 per 16 frames. MULTI: some layer has more than one
// node; its node count is a multiple of four, whose loads overlap. Measured for 4608
// atoms: 9 us for one frame, 10 for 16 (sincospi phases, always 32 frames: 16
// and 18); 4599 atoms in layers of 8 nodes, 13 frames 38 us; 32768 atoms, 64
// frames 540 us (740).
// Grid (tiles / PB_WAVES, frames / (16 NF), column splits): split z takes the
// columns [z cper, (z + 1) cper) and writes part + z f n (summed with the
// other splits when b is assembled).
constexpr int PB_WAVES = 4;

template <int NF, bool MULTI>
__global__ __launch_bounds__(64 * PB_WAVES) void plane_backproject_kernel(
    const double *__restrict__ pos, int64_t n, const int4 *__restrict__ tile,
    const int32_t *__restrict__ tile_atom, const double *__restrict__ lw, int64_t ntiles,
    const int4 *__restrict__ kcol, int64_t ncols_pad, int64_t cper, double inv_lx, double inv_ly,
    const double *__restrict__ Tre, const double *__restrict__ Tim, int64_t f_total,
    double *__restrict__ part) {
  __shared__ double2 tw[kTw];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (threadIdx.x < kTw) {
    double sj, cj;
    sincospi(2.0 * (double)threadIdx.x / kTw, &sj, &cj);
    tw[threadIdx.x] = make_double2(cj, sj);
  }
  __syncthreads();
  const int64_t cbeg = (int64_t)blockIdx.z * cper, cend = min(ncols_pad, cbeg + cper);
  part += (int64_t)blockIdx.z * f_total * n;
  const int64_t t = (int64_t)blockIdx.x * PB_WAVES + wave;
  if (t >= ntiles) return;   // no barriers below: a wave may leave alone
  const int lr = lane & 15, lq = lane >> 4;
  const int4 tl = tile[t];
  const int32_t atom = tile_atom[t * kPlaneTile + lr];
  double ux = 0.0, uy = 0.0;
  if (atom >= 0) {
    ux = pos[3 * (int64_t)atom] * inv_lx;
    uy = pos[3 * (int64_t)atom + 1] * inv_ly;
  }
  int64_t fo[NF];
  d4 acc[NF];
#pragma unroll
  for (int h = 0; h < NF; ++h) {
    // frames beyond the last repeat it (their results are not written)
    fo[h] = min((int64_t)blockIdx.y * (16 * NF) + 16 * h + lr, f_total - 1);
    acc[h] = d4{0.0, 0.0, 0.0, 0.0};
  }
  const double *tr = Tre + (int64_t)tl.x * ncols_pad * f_total;
  const double *ti = Tim + (int64_t)tl.x * ncols_pad * f_total;
  const int64_t nstep = ncols_pad * f_total;
  const double *wl = lw + (int64_t)tl.z * kPlaneTile + lr;
  auto phase = [&](int64_t c, double &cs, double &sn) {
    const int4 col = kcol[c];
    double th = (double)col.x * ux + (double)col.y * uy;
    th -= rint(th);
    phase_cs(tw, th, cs, sn);
  };
  if (!MULTI || tl.y == 1) {
    for (int64_t c0 = cbeg; c0 < cend; c0 += 16) {   // splits are multiples of 64
      double va[4][NF], vb[4][NF], cs[4], sn[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int h = 0; h < NF; ++h) {
          const int64_t o = (c0 + 4 * u + lq) * f_total + fo[h];
          va[u][h] = tr[o];
          vb[u][h] = ti[o];
        }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 4; ++u) phase(c0 + 4 * u + lq, cs[u], sn[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int h = 0; h < NF; ++h) {
          acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(va[u][h], cs[u], acc[h], 0, 0, 0);
          acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(vb[u][h], sn[u], acc[h], 0, 0, 0);
        }
    }
  } else {
    for (int64_t c0 = cbeg; c0 < cend; c0 += 4) {
      const int64_t c = c0 + lq, o = c * f_total;
      double cs, sn;
      phase(c, cs, sn);
      for (int j0 = 0; j0 < tl.y; j0 += 4) {
        double w[4], va[4][NF], vb[4][NF];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          w[j] = wl[(j0 + j) * kPlaneTile];
#pragma unroll
          for (int h = 0; h < NF; ++h) {
            va[j][h] = tr[(j0 + j) * nstep + o + fo[h]];
            vb[j][h] = ti[(j0 + j) * nstep + o + fo[h]];
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double wc = w[j] * cs, ws = w[j] * sn;
#pragma unroll
          for (int h = 0; h < NF; ++h) {
            acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(va[j][h], wc, acc[h], 0, 0, 0);
            acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(vb[j][h], ws, acc[h], 0, 0, 0);
          }
        }
      }
    }
  }
  // D[i][j] (frame i, atom j) in lane j + 16 (i % 4), register i / 4
  if (atom < 0) return;
#pragma unroll
  for (int h = 0; h < NF; ++h)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t f = (int64_t)blockIdx.y * (16 * NF) + 16 * h + 4 * v + lq;
      if (f < f_total) part[f * n + atom] = acc[h][v];
    }
}

// b[f, i] = chi_i / k_e - sum_ks bp[ks][f][i] - sum_g rs[g][f][i] - c0 Q_f
// (fixed order over the k splits and ion groups); slab geometry (Eq. 39 in
// its definite form): - (4 pi / V) M1_f z_i.
__global__ void assemble_b_kernel(const double *__restrict__ bp, int ksplits,
                                  const double *__restrict__ rs, int rgroups, int64_t n,
                                  int64_t f_total, const double *__restrict__ chi,
                                  const double *__restrict__ qsol, double c0,
                                  const double *__restrict__ m1, double cs,
                                  const double *__restrict__ pos, double *__restrict__ b) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * f_total) return;
  const int64_t f = idx / n, i = idx % n;
  const int64_t fn = n * f_total;
  double s = 0.0;
#pragma unroll 8
  for (int ks = 0; ks < ksplits; ++ks) s += bp[ks * fn + idx];
#pragma unroll 8
  for (int g = 0; g < rgroups; ++g) s += rs[g * fn + idx];
  double v = chi[i] * (1.0 / kCoulombVA) - s - c0 * qsol[f];
  if (m1 != nullptr) v -= cs * m1[f] * pos[3 * i + 2];
  b[idx] = v;
}

// ---- real space over a cell list of the ions of each frame
//
// The box is cut into ncx x ncy x ncz cells (edges h_d = L_d / nc_d >=
// rcut / 2, at most kMaxCells cells); cell (cx, cy, cz) has index
// (cz ncy + cy) ncx + cx. Every frame's ions are put in cell order, ions of
// one cell in index order (a stable counting sort), in three steps:
//   cell_sort_chunk_kernel  per chunk of kChunk ions: keys (cell << 12 |
//                           local index) sorted in LDS (bitonic; unique keys,
//                           so the order is fixed), the chunk's count per cell
//   cell_scan_kernel        per frame: prefix sums of the counts over the
//                           chunks (per cell) and over the cells
//   cell_scatter_kernel     every ion to cell start + earlier chunks' count +
//                           its rank in its chunk, as (x, y, z, q)
// real_space_kernel<true> then gives each wavefront of 64 spatially compact
// atoms the cells that overlap its bounding box widened by rcut: one
// contiguous range of the sorted ions per (cz, cy) row (two where the x
// range wraps), so the sum runs in a fixed order.
constexpr int kChunk = 4096;            // ions per sorting chunk (12-bit local index)
constexpr int kChunkThreads = 1024;
constexpr int kMaxCells = 8192;         // 13-bit cell index; counts of a chunk fit in LDS

__device__ inline int cell_coord(double x, double L, double invh, int nc) {
  double xw = x - L * floor(x / L);
  int c = (int)(xw * invh);
  return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

__global__ __launch_bounds__(kChunkThreads) void cell_sort_chunk_kernel(
    const double *__restrict__ ion_pos, int64_t m, int64_t nchunks, double lx, double ly,
    double lz, double ihx, double ihy, double ihz, int ncx, int ncy, int ncz,
    uint32_t *__restrict__ skeys, int32_t *__restrict__ hist) {
  __shared__ uint32_t keys[kChunk];
  const int64_t chunk = blockIdx.x, f = blockIdx.y;
  const int64_t i0 = chunk * kChunk;
  const int cnt = (int)((m - i0) < kChunk ? (m - i0) : kChunk);
  const double *pf = ion_pos + (f * m + i0) * 3;
  for (int j = threadIdx.x; j < kChunk; j += kChunkThreads) {
    uint32_t key = 0xffffffffu;
    if (j < cnt) {
      const int cx = cell_coord(pf[3 * j], lx, ihx, ncx);
      const int cy = cell_coord(pf[3 * j + 1], ly, ihy, ncy);
      const int cz = cell_coord(pf[3 * j + 2], lz, ihz, ncz);
      key = ((uint32_t)((cz * ncy + cy) * ncx + cx) << 12) | (uint32_t)j;
    }
    keys[j] = key;
  }
  __syncthreads();
  for (int k = 2; k <= kChunk; k <<= 1) {
    for (int jj = k >> 1; jj > 0; jj >>= 1) {
      for (int i = threadIdx.x; i < kChunk; i += kChunkThreads) {
        const int ixj = i ^ jj;
        if (ixj > i) {
          const uint32_t a = keys[i], b = keys[ixj];
          if ((a > b) == ((i & k) == 0)) {
            keys[i] = b;
            keys[ixj] = a;
          }
        }
      }
      __syncthreads();
    }
  }
  for (int j = threadIdx.x; j < cnt; j += kChunkThreads) skeys[f * m + i0 + j] = keys[j];
  // count of cell c = first position of cell c + 1 - first position of c
  const int ncell = ncx * ncy * ncz;
  int32_t *h = hist + (f * nchunks + chunk) * ncell;
  for (int c = threadIdx.x; c < ncell; c += kChunkThreads) {
    int lo = 0, hi = cnt;
    const uint32_t t0 = (uint32_t)c << 12;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (keys[mid] < t0) lo = mid + 1;
      else hi = mid;
    }
    int lo2 = lo, hi2 = cnt;
    const uint32_t t1 = (uint32_t)(c + 1) << 12;
    while (lo2 < hi2) {
      const int mid = (lo2 + hi2) >> 1;
      if (keys[mid] < t1) lo2 = mid + 1;
      else hi2 = mid;
    }
    h[c] = lo2 - lo;
  }
}

// One workgroup per frame: off[f][chunk][c] = sum of the counts of cell c in
// the earlier chunks; cstart[f][c] = number of ions in cells before c
// (cstart[f][ncell] = m).
__global__ __launch_bounds__(kChunkThreads) void cell_scan_kernel(
    int32_t *__restrict__ hist, int64_t nchunks, int ncell, int64_t m,
    int32_t *__restrict__ cstart) {
  __shared__ int32_t tot[kMaxCells];
  __shared__ int32_t part[kChunkThreads];
  const int64_t f = blockIdx.x;
  int32_t *h = hist + f * nchunks * ncell;
  for (int c = threadIdx.x; c < ncell; c += kChunkThreads) {
    int32_t run = 0;
    for (int64_t ch = 0; ch < nchunks; ++ch) {
      const int32_t v = h[ch * ncell + c];
      h[ch * ncell + c] = run;
      run += v;
    }
    tot[c] = run;
  }
  __syncthreads();
  // exclusive scan of tot over the cells: each thread a contiguous slice
  const int per = (ncell + kChunkThreads - 1) / kChunkThreads;
  const int c0 = threadIdx.x * per, c1 = min(ncell, c0 + per);
  int32_t sum = 0;
  for (int c = c0; c < c1; ++c) sum += tot[c];
  part[threadIdx.x] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t run = 0;
    for (int t = 0; t < kChunkThreads; ++t) {
      const int32_t v = part[t];
      part[t] = run;
      run += v;
    }
  }
  __syncthreads();
  int32_t run = part[threadIdx.x];
  int32_t *cs = cstart + f * (ncell + 1);
  for (int c = c0; c < c1; ++c) {
    cs[c] = run;
    run += tot[c];
  }
  if (threadIdx.x == 0) cs[ncell] = (int32_t)m;
}

__global__ __launch_bounds__(kChunkThreads) void cell_scatter_kernel(
    const double *__restrict__ ion_pos, const double *__restrict__ ion_q, int64_t m,
    int64_t nchunks, int ncell, const uint32_t *__restrict__ skeys,
    const int32_t *__restrict__ off, const int32_t *__restrict__ cstart,
    double4 *__restrict__ sorted) {
  __shared__ uint32_t keys[kChunk];
  const int64_t chunk = blockIdx.x, f = blockIdx.y;
  const int64_t i0 = chunk * kChunk;
  const int cnt = (int)((m - i0) < kChunk ? (m - i0) : kChunk);
  for (int j = threadIdx.x; j < cnt; j += kChunkThreads) keys[j] = skeys[f * m + i0 + j];
  __syncthreads();
  const int32_t *o = off + (f * nchunks + chunk) * ncell;
  const int32_t *cs = cstart + f * (ncell + 1);
  const double *pf = ion_pos + f * m * 3;
  const double *qf = ion_q + f * m;
  for (int j = threadIdx.x; j < cnt; j += kChunkThreads) {
    const uint32_t key = keys[j];
    const int c = (int)(key >> 12);
    const int64_t I = i0 + (int64_t)(key & 0xfffu);
    int lo = 0, hi = j;   // first position of cell c in the chunk
    const uint32_t t0 = (uint32_t)c << 12;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (keys[mid] < t0) lo = mid + 1;
      else hi = mid;
    }
    const int64_t dst = (int64_t)cs[c] + o[c] + (j - lo);
    sorted[f * m + dst] = make_double4(pf[3 * I], pf[3 * I + 1], pf[3 * I + 2], qf[I]);
  }
}

// Cells [a, b] (unwrapped, a <= b) along one edge of nc cells: all of them
// once when the range covers the edge.
__device__ inline void cell_span(double lo, double hi, double invh, int nc, int &a, int &b) {
  a = (int)floor(lo * invh);
  b = (int)floor(hi * invh);
  if (b - a + 1 >= nc) {
    a = 0;
    b = nc - 1;
  }
}

__device__ inline int wrap_cell(int c, int nc) {
  c %= nc;
  return c < 0 ? c + nc : c;
}

// rs[g][f][i] = sum over the ions of group g (with the cell list: over the
// ions in its rows of cells) of q sum_images [erfc(beta d) - erfc(a_i d)] / d,
// d < rcut. One wave per 64 spatially compact atoms order[..], frame and
// group. The wave looks at 64 ions at a time, one per lane: every periodic
// image within rcut of the tile's bounding box goes to a list in LDS (ballot,
// in order), and each listed image is then paired with the 64 atoms by three
// subtractions; a box narrower than the widened tile only lists an ion more
// than once. Four waves share the table of erfc, so that LDS holds as many
// waves as the registers (with a table per wave the largest case below takes
// 750 us). Bound by the FP64 vector unit and the reads of the table (55 and
// 50 % of the time, half the lanes within rcut). Measured, before (each pair
// with its own minimum image, an atom per thread against groups of 256 ions;
// with the cell list all ions of the cells) and now: 4608 atoms, 2000 ions,
// 1 frame 64 and 12 us, 16 frames 125 and 48 us; 288 atoms, 200 ions, 1 frame
// 131 and 15 us; 8192 atoms, 32 frames of 50000 ions 1890 and 600 us.
constexpr int RS_W = 4;   // waves per workgroup, which share the table
// LDS written by this wave before is read by it after (its accesses are in order)
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
template <bool CELL>
__global__ __launch_bounds__(64 * RS_W) void real_space_kernel(
    const double *__restrict__ pos, const double *__restrict__ width,
    const int32_t *__restrict__ order, int64_t n, const double *__restrict__ ion_pos,
    const double *__restrict__ ion_q, int64_t ipg, const double4 *__restrict__ sorted,
    const int32_t *__restrict__ cstart, int64_t m, int ncx, int ncy, int ncz, double lx,
    double ly, double lz, double beta, double rcut, int64_t f_total,
    const double *__restrict__ etab, double *__restrict__ rs) {
  __shared__ double4 lists[RS_W][128];
  __shared__ double et[kErfcTab];
  const int64_t f = blockIdx.y, grp = blockIdx.z;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double4 *lst = lists[wave];
  const int64_t t = ((int64_t)blockIdx.x * RS_W + wave) * 64 + lane;
  const int64_t i = t < n ? (int64_t)order[t] : -1;
  for (int q = threadIdx.x; q < kErfcTab; q += 64 * RS_W) et[q] = etab[q];
  double xi = 0, yi = 0, zi = 0, ai = 1.0;
  if (i >= 0) {
    xi = pos[3 * i];
    yi = pos[3 * i + 1];
    zi = pos[3 * i + 2];
    ai = width[i];
  }
  const double ilx = 1.0 / lx, ily = 1.0 / ly, ilz = 1.0 / lz;
  // the images of the tile's atoms next to its first (lane 0 always holds
  // one) and their bounding box
  const double xr = __shfl(xi, 0, 64), yr = __shfl(yi, 0, 64), zr = __shfl(zi, 0, 64);
  xi -= lx * rint((xi - xr) * ilx);
  yi -= ly * rint((yi - yr) * ily);
  zi -= lz * rint((zi - zr) * ilz);
  if (i < 0) xi = xr, yi = yr, zi = zr;
  double xmin = xi, xmax = xi, ymin = yi, ymax = yi, zmin = zi, zmax = zi;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    xmin = fmin(xmin, __shfl_xor(xmin, o, 64));
    xmax = fmax(xmax, __shfl_xor(xmax, o, 64));
    ymin = fmin(ymin, __shfl_xor(ymin, o, 64));
    ymax = fmax(ymax, __shfl_xor(ymax, o, 64));
    zmin = fmin(zmin, __shfl_xor(zmin, o, 64));
    zmax = fmax(zmax, __shfl_xor(zmax, o, 64));
  }
  // its centre, half its edges and these widened by rcut (and a hair for
  // rounding; the distance test below is exact), and the most images an ion
  // can have inside
  const double rw = rcut * (1.0 + 1e-9) + 1e-9;
  const double cx = 0.5 * (xmin + xmax), cy = 0.5 * (ymin + ymax), cz = 0.5 * (zmin + zmax);
  const double bx = 0.5 * (xmax - xmin), by = 0.5 * (ymax - ymin), bz = 0.5 * (zmax - zmin);
  const double hx = bx + rw, hy = by + rw, hz = bz + rw;
  const int ma = (int)(2.0 * hx * ilx) + 1, mb = (int)(2.0 * hy * ily) + 1,
            mc = (int)(2.0 * hz * ilz) + 1;
  const double rc2 = rcut * rcut;
  const double lim0 = 2.0 * (ai - beta) * 0.56418958354775628695;
  double acc = 0.0;
  auto process = [&](int cnt) {   // the first cnt listed images
    for (int j = 0; j < cnt; ++j) {
      const double4 ion = lst[j];
      const double dx = xi - ion.x, dy = yi - ion.y, dz = zi - ion.z;
      const double d2 = fma(dz, dz, fma(dy, dy, dx * dx));
      if (!(d2 < rc2)) continue;
      // 1 / d by one third-order step from the hardware estimate
      const double e2 = d2 > 0.0 ? d2 : 1.0;
      const double y0 = __builtin_amdgcn_rsq(e2), e = fma(-e2 * y0, y0, 1.0);
      const double y = fma(y0 * e, fma(0.375, e, 0.5), y0), d = e2 * y;
      double v = erfc_pw(et, beta * d);
      if (ai * d < kErfcZero) v -= erfc_pw(et, ai * d);
      acc += ion.w * (d2 > 0.0 ? v * y : lim0);
    }
  };
  int cnt = 0;
  auto push = [&](double4 ion, bool in) {   // full lists of 64 are processed
    const uint64_t mask = __ballot(in);
    if (in) lst[cnt + __popcll(mask & ((1ull << lane) - 1))] = ion;
    cnt += __popcll(mask);
    if (cnt < 64) return;
    wave_sync();
    process(64);
    wave_sync();
    cnt -= 64;
    const double4 rest = lst[64 + lane];
    wave_sync();
    if (lane < cnt) lst[lane] = rest;
  };
  auto offer = [&](double4 ion, bool valid) {   // one ion per lane (valid: it exists)
    const double ex = ion.x - cx, ey = ion.y - cy, ez = ion.z - cz;
    const double a0 = ceil((-hx - ex) * ilx), b0 = ceil((-hy - ey) * ily),
                 c0 = ceil((-hz - ez) * ilz);
    for (int a = 0; a < ma; ++a)
      for (int b = 0; b < mb; ++b)
        for (int c = 0; c < mc; ++c) {
          const double sx = (a0 + a) * lx, sy = (b0 + b) * ly, sz = (c0 + c) * lz;
          const double gx = fmax(fabs(ex + sx) - bx, 0.0), gy = fmax(fabs(ey + sy) - by, 0.0),
                       gz = fmax(fabs(ez + sz) - bz, 0.0);   // from the box
          push(make_double4(ion.x + sx, ion.y + sy, ion.z + sz, ion.w),
               valid && fma(gx, gx, fma(gy, gy, gz * gz)) < rw * rw);
        }
  };
  __syncthreads();
  if ((t & ~(int64_t)63) >= n) return;
  if constexpr (CELL) {
    // cells meeting the widened box
    int xa, xb, ya, yb, za, zb;
    cell_span(cx - hx, cx + hx, ncx * ilx, ncx, xa, xb);
    cell_span(cy - hy, cy + hy, ncy * ily, ncy, ya, yb);
    cell_span(cz - hz, cz + hz, ncz * ilz, ncz, za, zb);
    const int32_t *cs = cstart + f * ((int64_t)ncx * ncy * ncz + 1);
    const double4 *sf = sorted + f * m;
    int turn = (int)(gridDim.z - grp) - 1;   // the group takes each gridDim.z-th row
    const int xlen = xb - xa + 1, xw0 = wrap_cell(xa, ncx);
    for (int az = za; az <= zb; ++az) {
      const int azw = wrap_cell(az, ncz);
      for (int ay = ya; ay <= yb; ++ay) {
        if (++turn < (int)gridDim.z) continue;
        turn = 0;
        const int64_t row = ((int64_t)azw * ncy + wrap_cell(ay, ncy)) * ncx;
        for (int part = 0; part < 2; ++part) {
          const int c0 = part == 0 ? xw0 : 0;
          const int c1 = part == 0 ? min(ncx, xw0 + xlen) : xw0 + xlen - ncx;
          if (c1 <= c0) break;
          const int64_t s0 = cs[row + c0], s1 = cs[row + c1];
          for (int64_t base = s0; base < s1; base += 64)
            offer(sf[min(base + lane, s1 - 1)], base + lane < s1);
        }
      }
    }
  } else {
    const double *pf = ion_pos + f * m * 3;
    const double *qf = ion_q + f * m;
    const int64_t i0 = grp * ipg, i1 = min(m, i0 + ipg);
    for (int64_t base = i0; base < i1; base += 64) {
      const int64_t I = min(base + lane, i1 - 1);
      offer(make_double4(pf[3 * I], pf[3 * I + 1], pf[3 * I + 2], qf[I]), base + lane < i1);
    }
  }
  wave_sync();
  process(cnt);
  if (i >= 0) rs[(grp * f_total + f) * n + i] = acc;
}

}  // namespace

// doubles of one frame in the grid path's scratch: the grid, (n_z, part, x,
// y) and (n_z, n_y, part, x)
int64_t nu_frame_elems(const cpm_system *s) {
  const NuGrid &g = s->nu;
  const int64_t nz = g.m[2] + 1;
  return (int64_t)g.g[0] * g.g[1] * g.g[2] + 2 * nz * g.g[0] * g.g[1] +
         2 * nz * (2 * g.m[1] + 1) * g.g[0];
}

namespace {

// Work split of one cpm_rhs call over f frames of m ions, and the layout of
// its scratch buffer:
//   S   [nk][f][2]             structure factors
//   Sg  [sf_groups][f][nk][2]  per ion group (only when sf_groups > 1)
//   bp  [ksplit][f][n]         back-projection partials
//   T   [2][nodes][cols][f]    n_z sums per layer node (factored back-projection)
//   rs  [rs_groups][f][n]      real-space partials
//   nu  grid, y and x lines of nu_frames frames (structure factors through a grid)
struct RhsPlan {
  int64_t sf_groups = 1, sf_ipg = 0, ksplit = 0, kper = 0, rs_groups = 0, rs_ipg = 0;
  bool sf_gemm = false;         // structure factors on the matrix cores (|n_z| <= 47)
  bool bp_plane = false;        // factored back-projection over the atoms' layers
  bool rs_cell = false;         // real space over the cell list of the ions
  bool nu = false;              // structure factors through a grid, nu_frames frames at a time
  int64_t nu_frames = 0, off_nu = 0;
  int nc[3] = {1, 1, 1};        // cells per box edge
  int64_t nchunks = 0;          // sorting chunks per frame
  int64_t off_sg = 0, off_bp = 0, off_tp = 0, off_rs = 0, off_m1 = 0, off_sorted = 0, off_keys = 0,
          off_hist = 0, off_cstart = 0, total = 0;
};

// From this many ions per frame they are sorted into cells: the spreading of
// the grid path needs the list, so this is also where grids begin. For the
// real-space sums alone the line lies too low: the whole call without k-vectors,
// list and all pairs, takes 168 and 58 us at 2304 atoms and 8192 ions of one
// frame, 228 and 152 at 8192 atoms and 16 frames, and all pairs are ahead up to
// 20 000 ions at every size measured (8192 atoms, 16 frames: 351 and 317 us).
constexpr int64_t kCellMinIons = 8192;

// Cells of edge >= rcut / 2 (widened until there are at most kMaxCells).
void cell_grid(const double box[3], double rcut, int nc[3]) {
  double h = 0.5 * rcut;
  for (;;) {
    int64_t tot = 1;
    for (int d = 0; d < 3; ++d) {
      nc[d] = std::max(1, (int)std::floor(box[d] / h));
      tot *= nc[d];
    }
    if (tot <= kMaxCells) return;
    h *= 1.25;
  }
}

constexpr int64_t kTargetBlocks = 2048;          // workgroups that fill the chip several times
constexpr int64_t kPartialCap = (int64_t)1 << 27;  // doubles per partial buffer

// cost model of nu_pays in seconds per flop (per grid point; fixed per call).
// A system's first such call also makes its tables, 0.15 ms, which the model
// leaves out: with 130 us fixed, a system that serves one call saves 0.1 ms
// (9000 ions x 8 frames, 38 000 vectors: 0.63 against 0.72 ms, after 5 ms of
// assembly) and one that serves many loses up to 0.18 ms on each (12 000 x 8 in
// a box of 60 x 60 x 120 A: 0.85 against 0.67 ms).
constexpr double kNuDirect = 1.0 / 38e12, kNuSpread = 1.0 / 33e12, kNuPoint = 2.5e-12,
                 kNuDft = 1.0 / 38e12, kNuFixed = 30e-6, kNuWave = 0.4e-6;

// groups of at least RB items each, enough for ~kTargetBlocks workgroups,
// at most 64 and at most cap
int64_t groups_for(int64_t blocks, int64_t items, int64_t cap, int64_t &per) {
  int64_t g = (kTargetBlocks + blocks - 1) / std::max<int64_t>(1, blocks);
  g = std::min<int64_t>({g, std::max<int64_t>(1, items / RB), 64, std::max<int64_t>(1, cap)});
  g = std::max<int64_t>(1, g);
  per = (items + g - 1) / g;
  return per > 0 ? (items + per - 1) / per : 1;
}

// the same for workgroups of one wave: with work as uneven as the real-space
// sums of atoms near and far from the ions, two waves for each of the ~4096
// that are resident (13 frames of 1999 ions and 4599 atoms: 131 us with 2048
// waves, 100 with 4096, 78 with 8192, 71 with 16384, 81 with 32768; 16 frames
// of 2000 and 4608: 90, 70, 60, 62, 76; a table per wave in all of them)
int64_t wave_groups(int64_t waves, int64_t items, int64_t least, int64_t cap, int64_t &per) {
  int64_t g = (8192 + waves - 1) / std::max<int64_t>(1, waves);
  g = std::min<int64_t>({g, std::max<int64_t>(1, items / least), 64, std::max<int64_t>(1, cap)});
  g = std::max<int64_t>(1, g);
  per = (items + g - 1) / g;
  return per > 0 ? (items + per - 1) / per : 1;
}

// Whether the grid path beats the direct product, from the time of both at
// the rates each was measured at. With few frames the densest tile's wave
// sets the spreading time (an ion reaches 8 tiles; a slit's electrolyte is
// about 2.5 times denser than the box on average). Measured (us per call,
// direct / grid, whole right-hand side, 1 + 1 graphite layers, box height
// 120 A): 37 700 vectors, 12 000 ions x 16 frames 1924 / 1753, x 1 frame
// 1154 / 1276; 56 500 vectors, 50 000 ions x 16 8391 / 5043, x 1 3342 / 3416;
// 120 500 vectors, 8192 ions x 1 638 / 626, 50 000 x 16 11835 / 4187.
bool nu_pays(const cpm_system *s, int64_t m, int64_t f) {
  const NuGrid &g = s->nu;
  const double nk = (double)s->kset.nk, nz = g.m[2] + 1, ny = 2 * g.m[1] + 1;
  const double gx = g.g[0], gy = g.g[1], gz = g.g[2];
  auto up = [](double v, int b) { return std::ceil(v / b) * b; };
  const double direct = 4.0 * nk * (double)m * kNuDirect;
  const double spread = (double)m * 65536.0 * kNuSpread + gx * gy * gz * kNuPoint;
  const double tile_wave = 8.0 * (double)m / (gx * gy * gz / (NU_T * NU_T * NU_T)) * kNuWave;
  const double dft = 2.0 * gx * gy * gz * up(2.0 * nz, 16) +
                     8.0 * gx * gy * nz * up(g.m[1] + 1, 16 * NU_K2) +
                     8.0 * gx * nz * up(ny, 16) * up(g.m[0] + 1, 16 * NU_K2);
  return direct * (double)f > std::max(spread * (double)f, tile_wave) + dft * kNuDft * (double)f + kNuFixed;
}

}  // namespace

bool rhs_grid_pays(const cpm_system *s, int64_t m, int64_t f) {
  return s->kset.nk > 0 && m >= kCellMinIons && nu_pays(s, m, f);
}

namespace {

// cap_* > 0 bound the ion groups of the structure factor, the k splits of
// the back-projection and the ion groups of the real-space sum (fewer
// partial buffers, less parallelism)
RhsPlan rhs_plan_capped(const cpm_system *s, int64_t m, int64_t f, int64_t cap_sf,
                        int64_t cap_ks, int64_t cap_rs, bool planes, bool grid) {
  RhsPlan p;
  const int64_t n = s->n, nk = std::max<int64_t>(s->kset.nk, 1);
  const int64_t rblocks = (s->kset.nruns + RB - 1) / RB;
  const int64_t fgroups = (f + FG - 1) / FG;
  const int64_t bblocks = (n + RB * BP_AT - 1) / (RB * BP_AT);
  if (m > 0 && s->kset.nk > 0) {
    p.sf_gemm = s->kset.smax < SG_SB * 16;
    const int64_t sf_blocks = p.sf_gemm ? (s->kset.ncols_pad / kSfTile) * f
                                        : std::max<int64_t>(1, rblocks) * f;
    p.nu = grid && s->nu.elems >= nu_frame_elems(s) && rhs_grid_pays(s, m, f);
    const int64_t cap = std::max<int64_t>(1, std::min(cap_sf, kPartialCap / (2 * nk * f)));
    if (p.sf_gemm) {
      // whole chunks of ions per group, for about 1024 workgroups (three per
      // CU are resident): one frame of 2000 ions, 7 tiles: 43 us with 7 groups
      // of 286 ions, 17 with 32, 16 with 63, whose sum costs 3 us more; 13
      // frames: 80 us and 8 for the sum with 7 groups, 78 and 10 with 12,
      // 78 and 13 with 17
      const int64_t chunks = (m + SG_CH - 1) / SG_CH;
      const int64_t g = std::max<int64_t>(
          1, std::min<int64_t>({(1024 + sf_blocks - 1) / sf_blocks, chunks, 32, cap}));
      p.sf_ipg = (chunks + g - 1) / g * SG_CH;
      p.sf_groups = (m + p.sf_ipg - 1) / p.sf_ipg;
    } else {
      p.sf_groups = groups_for(sf_blocks, m, cap, p.sf_ipg);
    }
    // k splits of the back-projection: as many as fill every SIMD with three
    // wavefronts (its occupancy) without a fourth on some, at least 32 k each
    const int64_t per = bblocks * fgroups * (RB / 64);
    int64_t ks = std::max<int64_t>(1, (3 * 1024) / per);
    ks = std::min<int64_t>({ks, std::max<int64_t>(1, nk / 32),
                            std::max<int64_t>(1, kPartialCap / (f * n)), cap_ks});
    p.kper = (nk + ks - 1) / ks;
    p.ksplit = (nk + p.kper - 1) / p.kper;
    if (planes && s->layer.nodes > 0) {
      // column splits (multiples of 64 columns) until about 1024 workgroups
      p.bp_plane = true;
      const int64_t wgs = (s->layer.ntiles + 3) / 4 * ((f + 31) / 32);
      const int64_t units = s->kset.ncols_pad / 64;
      int64_t cs = std::min<int64_t>({std::max<int64_t>(1, (1024 + wgs - 1) / wgs), units,
                                      std::max<int64_t>(1, kPartialCap / (f * n)), cap_ks});
      cs = std::max<int64_t>(1, cs);
      p.kper = (units + cs - 1) / cs * 64;   // columns per split
      p.ksplit = (s->kset.ncols_pad + p.kper - 1) / p.kper;
    }
  }
  if (p.nu) {
    p.sf_gemm = false;
    p.sf_groups = 1;
    p.nu_frames = std::min<int64_t>(f, s->nu.elems / nu_frame_elems(s));
  }
  if (m >= kCellMinIons) {
    p.rs_cell = true;
    cell_grid(s->box, s->rcut, p.nc);
    p.nchunks = (m + kChunk - 1) / kChunk;
    p.rs_groups = wave_groups((n + 63) / 64 * f, (int64_t)p.nc[1] * p.nc[2], 4,
                              std::min(cap_rs, kPartialCap / (f * n)), p.rs_ipg);
  } else if (m > 0) {
    p.rs_groups = wave_groups((n + 63) / 64 * f, m, 16, std::min(cap_rs, kPartialCap / (f * n)),
                              p.rs_ipg);
  }
  const int64_t ncell = (int64_t)p.nc[0] * p.nc[1] * p.nc[2];
  p.off_sg = 2 * nk * f;
  p.off_bp = p.off_sg + (p.sf_groups > 1 ? p.sf_groups * 2 * nk * f : 0);
  p.off_tp = p.off_bp + p.ksplit * f * n;
  p.off_rs = p.off_tp + (p.bp_plane ? 2 * (int64_t)s->layer.nodes * s->kset.ncols_pad * f : 0);
  p.off_m1 = p.off_rs + p.rs_groups * f * n;
  p.off_sorted = (p.off_m1 + f + 3) / 4 * 4;   // 32-byte aligned (double4)
  p.off_keys = p.off_sorted + (p.rs_cell ? 4 * f * m : 0);
  p.off_hist = p.off_keys + (p.rs_cell ? (f * m + 1) / 2 : 0);
  p.off_cstart = p.off_hist + (p.rs_cell ? (f * p.nchunks * ncell + 1) / 2 : 0);
  p.off_nu = (p.off_cstart + (p.rs_cell ? (f * (ncell + 1) + 1) / 2 : 0) + 3) / 4 * 4;
  p.total = p.off_nu + (p.nu ? p.nu_frames * nu_frame_elems(s) : 0);
  return p;
}

constexpr int64_t kNoCap = (int64_t)1 << 40;

// the default plan, or with limit > 0 the most parallel plan whose scratch
// holds at most limit doubles (halving the largest partial count first)
RhsPlan rhs_plan(const cpm_system *s, int64_t m, int64_t f, int64_t limit = 0) {
  // the factored back-projection first; without it when its per-node sums
  // do not fit the limit
  for (int planes = 1;; planes = 0) {
    RhsPlan p = rhs_plan_capped(s, m, f, kNoCap, kNoCap, kNoCap, planes != 0, limit <= 0);
    int64_t csf = p.sf_groups, cks = std::max<int64_t>(1, p.ksplit), crs = p.rs_groups;
    while (limit > 0 && p.total > limit && (csf > 1 || cks > 1 || crs > 1)) {
      const int64_t nk = std::max<int64_t>(s->kset.nk, 1);
      const int64_t wsf = csf > 1 ? csf * 2 * nk * f : 0, wks = cks > 1 ? cks * f * s->n : 0,
                    wrs = crs > 1 ? crs * f * s->n : 0;
      if (wsf >= wks && wsf >= wrs) csf = std::max<int64_t>(1, csf / 2);
      else if (wks >= wrs) cks = std::max<int64_t>(1, cks / 2);
      else crs = std::max<int64_t>(1, crs / 2);
      p = rhs_plan_capped(s, m, f, csf, cks, crs, planes != 0, false);
    }
    if (limit <= 0 || p.total <= limit || !p.bp_plane) return p;
  }
}

// ---- cpm_rhs_noalloc: the scratch in a fixed device array
//
// kStaticRhsScratch doubles (32 MiB) per GPU, held by the code object until
// the process ends. Host code takes its device address from
// hipGetSymbolAddress (per device, on first use): the array's name in host
// code is not a device address.
constexpr int64_t kStaticRhsScratch = (int64_t)1 << 22;

}  // namespace

static __device__ __align__(256) double scratch[kStaticRhsScratch];

int64_t rhs_scratch_elems(const cpm_system *s, int64_t m, int64_t f) {
  return rhs_plan(s, m, f).total;
}

int64_t rhs_static_scratch_elems() { return kStaticRhsScratch; }

int64_t rhs_scratch_elems_capped(const cpm_system *s, int64_t m, int64_t f, int64_t limit) {
  return rhs_plan(s, m, f, limit).total;
}

hipError_t rhs_static_scratch(double **ptr) {
  static std::mutex mu;
  static std::vector<double *> per_device;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lock(mu);
  if ((int)per_device.size() <= dev) per_device.resize(dev + 1, nullptr);
  if (!per_device[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    per_device[dev] = static_cast<double *>(p);
  }
  *ptr = per_device[dev];
  return hipSuccess;
}

namespace {

// flops of the grid path per frame (its own products, with their padding)
double nu_flops(const cpm_system *s, int64_t m) {
  const NuGrid &g = s->nu;
  const double gx = g.g[0], gy = g.g[1], gz = g.g[2], nz = g.m[2] + 1, ny = 2 * g.m[1] + 1;
  return 65536.0 * (double)m + 4.0 * gx * gy * gz * nz + 8.0 * gx * gy * nz * (g.m[1] + 1) +
         8.0 * gx * nz * ny * (g.m[0] + 1);
}

hipError_t launch_nu(hipStream_t st, const cpm_system *s, const RhsPlan &p, int64_t m, int64_t f,
                     double *buf, double *S, hipEvent_t ea, hipEvent_t eb) {
  const NuGrid &g = s->nu;
  const int gx = g.g[0], gy = g.g[1], gz = g.g[2], nz = g.m[2] + 1, ny = 2 * g.m[1] + 1;
  const int64_t lines = (int64_t)gx * gy, tiles = lines / (NU_T * NU_T) * (gz / NU_T);
  const double4 *sorted = reinterpret_cast<const double4 *>(buf + p.off_sorted);
  const int32_t *cstart = reinterpret_cast<const int32_t *>(buf + p.off_cstart);
  const int64_t ncell = (int64_t)p.nc[0] * p.nc[1] * p.nc[2];
  double *grid = buf + p.off_nu, *o1 = grid + p.nu_frames * lines * gz,
         *o2 = o1 + p.nu_frames * 2 * nz * lines;
  for (int64_t f0 = 0; f0 < f; f0 += p.nu_frames) {
    const unsigned fc = (unsigned)std::min<int64_t>(p.nu_frames, f - f0);
    hipExtLaunchKernelGGL(nu_spread_kernel, dim3((unsigned)tiles, fc), dim3(64), 0, st,
                          f0 == 0 ? ea : nullptr, nullptr, 0, sorted + f0 * m,
                          cstart + f0 * (ncell + 1), m, p.nc[0], p.nc[1], p.nc[2], s->box[0],
                          s->box[1], s->box[2], gx, gy, gz, (const double *)g.coef, grid);
    const int zp = g.zpasses, rt = g.zrows / 16 / zp;
    auto kz = rt == 1   ? nu_dftz_kernel<1>
              : rt == 2 ? nu_dftz_kernel<2>
              : rt == 3 ? nu_dftz_kernel<3>
              : rt == 4 ? nu_dftz_kernel<4>
              : rt == 5 ? nu_dftz_kernel<5>
                        : nu_dftz_kernel<NU_RZ>;
    hipLaunchKernelGGL(kz, dim3((unsigned)(lines / 128), fc, (unsigned)zp), dim3(256), 0, st,
                       (const double *)grid, lines, gz, (const double *)g.mat[2], nz, o1);
    const int64_t wy = (int64_t)(gx / 16) * g.passes[1] * nz;
    hipLaunchKernelGGL(nu_dfty_kernel, dim3((unsigned)((wy + 3) / 4), fc), dim3(256), 0, st,
                       (const double *)o1, gx, gy, nz, g.m[1], g.passes[1],
                       (const double *)g.mat[1], o2);
    const int64_t wx = (int64_t)((ny + 15) / 16) * g.passes[0] * nz;
    hipExtLaunchKernelGGL(nu_dftx_kernel, dim3((unsigned)((wx + 3) / 4), fc), dim3(256), 0, st,
                          nullptr, f0 + fc == f ? eb : nullptr, 0, (const double *)o2, gx, nz,
                          g.m[0], g.m[1], g.passes[0], (const double *)g.mat[0],
                          (const double *)g.inv, g.m[0] + 1, g.m[0] + g.m[1] + 2, g.col, f0, f, S);
  }
  return hipGetLastError();
}

}  // namespace

void nu_sizes(cpm_system *s) {
  NuGrid &g = s->nu;
  for (int d = 0; d < 3; ++d) {
    g.m[d] = s->kset.nmax[d];
    // at least two points per mode, whole tiles, and room for a tile and its
    // reach (so that an ion meets a tile through one image only)
    g.g[d] = (int)round_up(std::max(2 * (2 * g.m[d] + 1), NU_T + NU_W), NU_T);
  }
  const int zt = (2 * (g.m[2] + 1) + 15) / 16;
  g.zpasses = (zt + NU_RZ - 1) / NU_RZ;
  g.zrows = (zt + g.zpasses - 1) / g.zpasses * g.zpasses * 16;
  for (int d = 0; d < 2; ++d) g.passes[d] = (g.m[d] + 1 + 16 * NU_K2 - 1) / (16 * NU_K2);
  // Grids at a time: the more frames a launch has, the less its last waves
  // count (8192 atoms, 32 frames of 7.0 M doubles: 5.0 ms with 256 MB, 4.6 with
  // 512, 4.2 with 1 GB, 4.0 with 2 GB). But the scratch stays with the system,
  // and once a process has been through the device's memory the driver clears
  // what is released at some 0.03 TB/s: 300 systems of 1024 atoms in a row that
  // each take 32 frames need 15 ms a system with 512 MB and 59 with 2 GB
  // (single waits of 2 s). So at most four times E (whose assembly takes the
  // longer the larger it is), at least 512 MB and at most 2 GB; or one grid.
  const int64_t frame = nu_frame_elems(s);
  g.full = std::min<int64_t>((int64_t)1 << 28, std::max<int64_t>((int64_t)1 << 26, 4 * s->ld * s->ld));
  g.full = std::max(g.full, frame);
}

bool rhs_uses_grid(const cpm_system *s, int64_t m, int64_t f) { return rhs_plan(s, m, f).nu; }

// ---- tables of the grid path

namespace {

// The window phi of the spreading, its polynomials (coef[s][d]: phi on
// [-w/2 + s, -w/2 + s + 1] as monomials of x = 2 delta - 1, through the
// Chebyshev points) and Gauss-Legendre nodes on (0, w/2) with weights 2 phi
// for its transform Phi (phi falls to exp(-beta) = 1e-16 at the ends).
// Constants of the program: made once per process, 0.15 ms of long double
// (2.3 ms when every system made them, with a cosine per term and 128 nodes;
// 40 give Phi to 5e-19, 32 to 3e-18).
struct NuWindow {
  static constexpr int N = NU_DEG + 1, Q = 40;
  double coef[NU_W * N];
  long double node[Q], weight[Q];
  NuWindow() {
    typedef long double ld;
    const ld pi = 3.14159265358979323846264338327950288L, beta = (ld)NU_BETA, half = 0.5L * NU_W;
    auto phi = [&](ld t) {
      const ld z = 1.0L - (t / half) * (t / half);
      return z > 0.0L ? std::exp(beta * (std::sqrt(z) - 1.0L)) : 0.0L;
    };
    ld cosine[N][N];   // T_j at the Chebyshev points
    for (int j = 0; j < N; ++j)
      for (int k = 0; k < N; ++k) cosine[j][k] = std::cos(pi * j * (k + 0.5L) / N);
    for (int si = 0; si < NU_W; ++si) {
      ld mono[N] = {}, t0[N] = {}, t1[N] = {}, fx[N];
      for (int k = 0; k < N; ++k) fx[k] = phi(-half + si + 0.5L * (cosine[1][k] + 1.0L));
      t0[0] = 1.0L;
      t1[1] = 1.0L;
      for (int j = 0; j < N; ++j) {   // t0 = T_j
        ld c = 0.0L;
        for (int k = 0; k < N; ++k) c += fx[k] * cosine[j][k];
        c *= (j == 0 ? 1.0L : 2.0L) / N;
        for (int k = 0; k < N; ++k) mono[k] += c * t0[k];
        ld t2[N] = {};
        for (int k = 0; k + 1 < N; ++k) t2[k + 1] = 2.0L * t1[k];
        for (int k = 0; k < N; ++k) {
          t2[k] -= t0[k];
          t0[k] = t1[k];
          t1[k] = t2[k];
        }
      }
      for (int k = 0; k < N; ++k) coef[si * N + k] = (double)mono[k];
    }
    for (int i = 0; i < Q / 2; ++i) {   // the nodes come in pairs +-x
      ld x = std::cos(pi * (i + 0.75L) / (Q + 0.5L)), dp = 0.0L;
      for (int it = 0; it < 6; ++it) {
        ld p0 = 1.0L, p1 = x;
        for (int j = 2; j <= Q; ++j) {
          const ld p2 = ((2 * j - 1) * x * p1 - (j - 1) * p0) / j;
          p0 = p1;
          p1 = p2;
        }
        dp = Q * (x * p1 - p0) / (x * x - 1.0L);
        x -= p1 / dp;
      }
      const ld w = 2.0L / ((1.0L - x * x) * dp * dp);
      for (int k : {i, Q - 1 - i}) {
        node[k] = 0.5L * half * ((k == i ? x : -x) + 1.0L);
        weight[k] = half * phi(node[k]) * w;
      }
    }
  }
};

// mat (rows of one axis by g): row n of the cosines at n * cos_step, of the
// sines at n * cos_step + sin_off, zero for n > m; cs: (cos, sin)(2 pi j / g).
// Grid (rows, axes).
struct NuAxis {
  double *mat;
  const double2 *cs;
  int g, m, rows, step, sin_off;
};
struct NuAxes {
  NuAxis a[3];
};
__global__ __launch_bounds__(128) void nu_matrix_kernel(NuAxes axes) {
  const NuAxis &a = axes.a[blockIdx.y];
  const int row = blockIdx.x;
  if (row >= a.rows) return;
  const bool sine = a.step == 2 ? row & 1 : row >= a.sin_off;
  const int n = a.step == 2 ? row >> 1 : row - (sine ? a.sin_off : 0);
  for (int j = threadIdx.x; j < a.g; j += 128) {
    const double2 v = a.cs[(int64_t)n * j % a.g];
    a.mat[(int64_t)row * a.g + j] = n > a.m ? 0.0 : sine ? v.y : v.x;
  }
}

}  // namespace

// The tables of one system on the device (on its first call that takes the
// grid): the transform matrices, expanded there from (cos, sin)(2 pi j / G),
// the window's polynomials, 1 / Phi and the column table. Of the host's work
// 1 / Phi is the largest part: exp(2 pi i n t / G) at the quadrature nodes by
// repeated rotation (2e-18).
cpm_status ensure_nu(cpm_system *s) {
  NuGrid &g = s->nu;
  if (g.coef) return CPM_OK;
  static const NuWindow win;
  typedef long double ld;
  const ld two_pi = 6.28318530717958647692528676655900577L;
  std::vector<double> h(win.coef, win.coef + NU_W * NuWindow::N);
  for (int d = 0; d < 3; ++d) {
    ld c[NuWindow::Q], sn[NuWindow::Q], rc[NuWindow::Q], rs[NuWindow::Q];
    for (int i = 0; i < NuWindow::Q; ++i) {
      c[i] = win.weight[i];
      sn[i] = 0.0L;
      rc[i] = std::cos(two_pi * win.node[i] / g.g[d]);
      rs[i] = std::sin(two_pi * win.node[i] / g.g[d]);
    }
    for (int n = 0; n <= g.m[d]; ++n) {
      ld v = 0.0L;
      for (int i = 0; i < NuWindow::Q; ++i) {
        v += c[i];
        const ld t = c[i] * rc[i] - sn[i] * rs[i];
        sn[i] = sn[i] * rc[i] + c[i] * rs[i];
        c[i] = t;
      }
      h.push_back((double)(1.0L / v));
    }
  }
  if (h.size() & 1) h.push_back(0.0);   // pairs from here on
  const size_t cs_off = h.size();
  for (int d = 0; d < 3; ++d) {
    const int G = g.g[d], q = G / 4;   // G is a multiple of 16
    std::vector<double> cq(q + 1);
    for (int j = 0; j < q; ++j) cq[j] = (double)std::cos(two_pi * j / G);
    cq[q] = 0.0;
    for (int j = 0; j < G; ++j) {
      const int k = j % q;
      const double c = cq[k], sv = cq[q - k];
      const double cs[4][2] = {{c, sv}, {-sv, c}, {-c, -sv}, {sv, -c}};
      h.insert(h.end(), cs[j / q], cs[j / q] + 2);
    }
  }
  const size_t col_off = h.size();
  const int ny = 2 * g.m[1] + 1;
  std::vector<int2> col((size_t)(g.m[0] + 1) * ny, make_int2(0, -1));
  for (int64_t c = 0; c < s->kset.ncols; ++c) {
    const int32_t *k = s->kset.cols.data() + 4 * c;
    col[(size_t)k[0] * ny + g.m[1] + k[1]] = make_int2(k[3], k[2]);
  }
  static_assert(sizeof(int2) == sizeof(double), "the column table in the block of doubles");
  h.resize(col_off + col.size());
  std::memcpy(h.data() + col_off, col.data(), sizeof(int2) * col.size());
  NuAxes axes;
  size_t moff[3], mats = 0;   // the matrices first: rows of 16 k are 128-byte aligned
  int rows = 0;
  for (int d = 0; d < 3; ++d) {
    NuAxis &a = axes.a[d];
    a.g = g.g[d];
    a.m = g.m[d];
    a.rows = d == 2 ? g.zrows : 2 * g.passes[d] * NU_K2 * 16;
    a.step = d == 2 ? 2 : 1;
    a.sin_off = d == 2 ? 1 : a.rows / 2;
    moff[d] = mats;
    mats += (size_t)a.rows * a.g;
    rows = std::max(rows, a.rows);
  }
  const size_t nd = mats + h.size();
  double *dev = nullptr;
  if (hipMalloc((void **)&dev, sizeof(double) * nd) != hipSuccess) {
    (void)hipGetLastError();
    set_error("structure-factor table allocation failed");
    return CPM_ENOMEM;
  }
  double *small = dev + mats;
  size_t cs_at = cs_off;
  for (int d = 0; d < 3; ++d) {
    axes.a[d].mat = dev + moff[d];
    axes.a[d].cs = reinterpret_cast<const double2 *>(small + cs_at);
    cs_at += 2 * (size_t)g.g[d];
  }
  hipError_t e = hipMemcpyAsync(small, h.data(), sizeof(double) * h.size(), hipMemcpyHostToDevice,
                                s->stream);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(nu_matrix_kernel, dim3((unsigned)rows, 3), dim3(128), 0, s->stream, axes);
    e = hipGetLastError();
  }
  const hipError_t done = hipStreamSynchronize(s->stream);   // the host copy goes out of scope
  if (e != hipSuccess || done != hipSuccess) {
    (void)hipFree(dev);
    set_error("structure-factor table copy failed");
    return CPM_EDEVICE;
  }
  for (int d = 0; d < 3; ++d) g.mat[d] = dev + moff[d];
  g.tab = dev;
  g.coef = small;
  g.inv = small + NU_W * NuWindow::N;
  g.col = reinterpret_cast<const int2 *>(small + col_off);
  s->device_bytes += (int64_t)(sizeof(double) * nd);
  return CPM_OK;
}

hipError_t launch_rhs(hipStream_t st, const cpm_system *s, const double *ion_pos,
                      const double *ion_q, int64_t m, int64_t f, const double *chi, double *buf,
                      double *b_out, double *qsol_out, int64_t limit) {
  const double ilx = 1.0 / s->box[0], ily = 1.0 / s->box[1], ilz = 1.0 / s->box[2];
  const int64_t nk = s->kset.nk, n = s->n;
  const double c0 = -M_PI / (s->vol * s->beta * s->beta);
  const RhsPlan p = rhs_plan(s, m, f, limit);
  double *S = buf, *bp = buf + p.off_bp, *rs = buf + p.off_rs;
  const int64_t fgroups = (f + FG - 1) / FG;
  double *m1 = s->slab ? buf + p.off_m1 : nullptr;
  if (m > 0) {
    hipLaunchKernelGGL(qsum_kernel, dim3((unsigned)f), dim3(RB), 0, st, ion_q, m, qsol_out, ion_pos,
                       s->box[2], m1);
  } else {
    // zeros by a kernel (no memset node when the caller captures the stream)
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((f + 255) / 256)), dim3(256), 0, st,
                       qsol_out, f);
    if (m1)
      hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((f + 255) / 256)), dim3(256), 0, st,
                         m1, f);
  }
  // the cell list of the ions (real space, and the grid path)
  if (p.rs_cell) {
    double4 *sorted = reinterpret_cast<double4 *>(buf + p.off_sorted);
    uint32_t *keys = reinterpret_cast<uint32_t *>(buf + p.off_keys);
    int32_t *hist = reinterpret_cast<int32_t *>(buf + p.off_hist);
    int32_t *cstart = reinterpret_cast<int32_t *>(buf + p.off_cstart);
    const int ncell = p.nc[0] * p.nc[1] * p.nc[2];
    hipLaunchKernelGGL(cell_sort_chunk_kernel, dim3((unsigned)p.nchunks, (unsigned)f),
                       dim3(kChunkThreads), 0, st, ion_pos, m, p.nchunks, s->box[0], s->box[1],
                       s->box[2], p.nc[0] * ilx, p.nc[1] * ily, p.nc[2] * ilz, p.nc[0], p.nc[1],
                       p.nc[2], keys, hist);
    hipLaunchKernelGGL(cell_scan_kernel, dim3((unsigned)f), dim3(kChunkThreads), 0, st, hist,
                       p.nchunks, ncell, m, cstart);
    hipLaunchKernelGGL(cell_scatter_kernel, dim3((unsigned)p.nchunks, (unsigned)f),
                       dim3(kChunkThreads), 0, st, ion_pos, ion_q, m, p.nchunks, ncell,
                       (const uint32_t *)keys, (const int32_t *)hist, (const int32_t *)cstart,
                       sorted);
  }
  if (p.ksplit > 0) {
    double *Sg = p.sf_groups > 1 ? buf + p.off_sg : S;
    const int64_t sk = p.sf_groups > 1 ? 1 : f, sf = p.sf_groups > 1 ? nk : 1;
    const int64_t rblocks = (s->kset.nruns + RB - 1) / RB;
    // live timing (cpm_profile_enable): algorithmic flops 4 n_k m f
    hipEvent_t ea = nullptr, eb = nullptr;
    if (s->prof.sample(4)) {
      Profile::Rec &r = s->prof.add(4, p.nu ? nu_flops(s, m) * (double)f
                                            : 4.0 * (double)nk * (double)m * (double)f);
      ea = r.a;
      eb = r.b;
    }
    if (p.nu) {
      const hipError_t e = launch_nu(st, s, p, m, f, buf, S, ea, eb);
      if (e != hipSuccess) return e;
    } else if (p.sf_gemm)
      hipExtLaunchKernelGGL(sf_gemm_kernel,
                            dim3((unsigned)(f * p.sf_groups),
                                 (unsigned)(s->kset.ncols_pad / kSfTile)),
                            dim3(256), 0, st, ea, eb, 0, ion_pos, ion_q, m, p.sf_ipg,
                            reinterpret_cast<const int4 *>(s->kcol), ilx, ily, ilz, nk, f, sk,
                            sf, Sg);
    else
      hipExtLaunchKernelGGL(structure_factor_kernel,
                            dim3((unsigned)rblocks, (unsigned)f, (unsigned)p.sf_groups), dim3(RB),
                            0, st, ea, eb, 0, ion_pos, ion_q, m, p.sf_ipg, s->kinfo, s->krun,
                            s->kset.nruns, nk, ilx, ily, ilz, f, sk, sf, Sg);
    if (p.sf_groups > 1)
      hipLaunchKernelGGL(sum_groups_kernel,
                         dim3((unsigned)((nk + SGT_K - 1) / SGT_K),
                              (unsigned)((f + SGT_F - 1) / SGT_F)),
                         dim3(256), 0, st, reinterpret_cast<const double2 *>(Sg),
                         (int)p.sf_groups, nk, f, reinterpret_cast<double2 *>(S));
    if (p.bp_plane) {
      const int64_t ncp = s->kset.ncols_pad;
      const Layers &ly = s->layer;
      double *Tre = buf + p.off_tp, *Tim = Tre + (int64_t)ly.nodes * ncp * f;
      const int4 *kcol = reinterpret_cast<const int4 *>(s->kcol);
      hipLaunchKernelGGL(plane_table_kernel,
                         dim3((unsigned)(ncp / PT_WAVES), (unsigned)(ly.nodes_pad / 16),
                              (unsigned)((f + 15) / 16)),
                         dim3(64 * PT_WAVES), 0, st, reinterpret_cast<const double2 *>(ly.zt),
                         ly.nodes, ly.nodes_pad, kcol, ncp, (const double *)s->kw,
                         reinterpret_cast<const double2 *>(S), f, Tre, Tim);
      const int nf = f > 16 ? 2 : 1;
      const dim3 grid((unsigned)((ly.ntiles + PB_WAVES - 1) / PB_WAVES),
                      (unsigned)((f + 16 * nf - 1) / (16 * nf)), (unsigned)p.ksplit);
#define CPM_PLANE_BP(NF, MULTI)                                                                  \
  hipLaunchKernelGGL((plane_backproject_kernel<NF, MULTI>), grid, dim3(64 * PB_WAVES), 0, st,    \
                     (const double *)s->pos, n, reinterpret_cast<const int4 *>(ly.tile), ly.atom, \
                     (const double *)ly.lw, ly.ntiles, kcol, ncp, p.kper, ilx, ily,              \
                     (const double *)Tre, (const double *)Tim, f, bp)
      if (nf == 1 && ly.multi) CPM_PLANE_BP(1, true);
      else if (nf == 1) CPM_PLANE_BP(1, false);
      else if (ly.multi) CPM_PLANE_BP(2, true);
      else CPM_PLANE_BP(2, false);
#undef CPM_PLANE_BP
    } else {
      const int64_t bblocks = (n + RB * BP_AT - 1) / (RB * BP_AT);
      hipLaunchKernelGGL(backproject_kernel<BP_AT>,
                         dim3((unsigned)bblocks, (unsigned)p.ksplit, (unsigned)fgroups), dim3(RB),
                         0, st, s->pos, n, s->kinfo, s->kw, nk, p.kper, ilx, ily, ilz, S, f, bp);
    }
  }
  if (p.rs_cell) {
    const double4 *sorted = reinterpret_cast<const double4 *>(buf + p.off_sorted);
    const int32_t *cstart = reinterpret_cast<const int32_t *>(buf + p.off_cstart);
    hipLaunchKernelGGL(real_space_kernel<true>,
                       dim3((unsigned)((n + 64 * RS_W - 1) / (64 * RS_W)), (unsigned)f,
                            (unsigned)p.rs_groups),
                       dim3(64 * RS_W), 0, st, s->pos, s->rs_width, s->atom_order, n, ion_pos, ion_q,
                       (int64_t)0, sorted, cstart, m, p.nc[0], p.nc[1], p.nc[2], s->box[0],
                       s->box[1], s->box[2], s->beta, s->rcut, f, (const double *)s->erfc_tab, rs);
  } else if (p.rs_groups > 0) {
    hipLaunchKernelGGL(real_space_kernel<false>,
                       dim3((unsigned)((n + 64 * RS_W - 1) / (64 * RS_W)), (unsigned)f,
                            (unsigned)p.rs_groups),
                       dim3(64 * RS_W), 0, st, s->pos, s->rs_width, s->atom_order, n, ion_pos, ion_q,
                       p.rs_ipg, (const double4 *)nullptr, (const int32_t *)nullptr, m, 1, 1, 1,
                       s->box[0], s->box[1], s->box[2], s->beta, s->rcut, f,
                       (const double *)s->erfc_tab, rs);
  }
  hipLaunchKernelGGL(assemble_b_kernel, dim3((unsigned)((n * f + 255) / 256)), dim3(256), 0, st,
                     bp, (int)p.ksplit, rs, (int)p.rs_groups, n, f, chi, qsol_out, c0,
                     (const double *)m1, 4.0 * M_PI / s->vol, s->pos, b_out);
  return hipGetLastError();
}

// One device block for a system's layers: tiles, atoms, node z, tables.
static int64_t layers_fixed(const LayerPlan &lp) {
  const int64_t nt = (int64_t)lp.tile.size() / 4, nodes = (int64_t)lp.node_z.size();
  return (2 * nt + nt * kPlaneTile / 2 + nodes + 1) / 2 * 2;
}
int64_t layers_elems(const LayerPlan &lp, int smax) {
  const int64_t npad = ((int64_t)lp.node_z.size() + 15) / 16 * 16;
  return layers_fixed(lp) + 2 * (smax + 1) * npad + lp.weights * kPlaneTile;
}
hipError_t set_layers(cpm_system *s, hipStream_t st, const LayerPlan &lp, double *d) {
  const int64_t nt = (int64_t)lp.tile.size() / 4, nodes = (int64_t)lp.node_z.size();
  const int64_t npad = (nodes + 15) / 16 * 16, smax = s->kset.smax;
  std::vector<double> h(layers_fixed(lp), 0.0);
  const int64_t oa = 2 * nt, oz = oa + nt * kPlaneTile / 2;
  std::memcpy(h.data(), lp.tile.data(), sizeof(int32_t) * 4 * nt);
  std::memcpy(h.data() + oa, lp.atom.data(), sizeof(int32_t) * kPlaneTile * nt);
  std::memcpy(h.data() + oz, lp.node_z.data(), sizeof(double) * nodes);
  Layers &out = s->layer;
  out.tile = reinterpret_cast<int32_t *>(d);
  out.atom = reinterpret_cast<int32_t *>(d + oa);
  out.zt = d + h.size();
  out.lw = out.zt + 2 * (smax + 1) * npad;
  out.ntiles = nt;
  out.nodes = (int)nodes;
  out.nodes_pad = (int)npad;
  out.multi = lp.weights > nt;
  hipError_t e =
      hipMemcpyAsync(d, h.data(), sizeof(double) * h.size(), hipMemcpyHostToDevice, st);
  if (e != hipSuccess) return e;
  const int64_t work = std::max((smax + 1) * npad, nt * kPlaneTile);
  hipLaunchKernelGGL(layer_tables_kernel, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, st,
                     (const double *)s->pos, 1.0 / s->box[2],
                     reinterpret_cast<const int4 *>(out.tile), (const int32_t *)out.atom, nt,
                     (const double *)(d + oz), (int)nodes, (int)npad, (int)smax,
                     reinterpret_cast<double2 *>(out.zt), out.lw);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return hipStreamSynchronize(st);   // the host copy goes out of scope
}

// Coefficients of erfc_pw. About x_j = (j + 1/2) / kErfcPer: c_0 = erfc(x_j)
// and, from d^(k+1)/dx^(k+1) erfc(x) = -(2/sqrt(pi)) (-1)^k H_k(x) exp(-x^2)
// with the Hermite recurrence H_(k+1) = 2 x H_k - 2 k H_(k-1), c_(k+1) = that
// derivative / ((k+1)! kErfcPer^(k+1)), taken to degree NT - 1 in long double
// and reduced to kErfcTerms terms one degree at a time: subtract the multiple
// of the Chebyshev polynomial T_n(2u) that cancels u^n (it adds at most
// |c_n| / 2^(2n-1) on [-1/2, 1/2]).
void erfc_table(double *out) {
  constexpr int NT = 16;
  const long double c2 = 2.0L / std::sqrt(3.14159265358979323846264338327950288L);
  long double cheb[NT][NT] = {};   // T_n(2u) in powers of u
  cheb[0][0] = 1.0L;
  cheb[1][1] = 2.0L;
  for (int n = 2; n < NT; ++n)
    for (int k = 0; k <= n; ++k)
      cheb[n][k] = (k > 0 ? 4.0L * cheb[n - 1][k - 1] : 0.0L) - cheb[n - 2][k];
  for (int j = 0; j < kErfcIntervals; ++j) {
    const long double x = ((long double)j + 0.5L) / kErfcPer;
    const long double e = std::exp(-x * x);
    long double c[NT];
    c[0] = std::erfc(x);
    long double hprev = 0.0L, hcur = 1.0L, fact = 1.0L, scale = 1.0L;
    for (int k = 0; k + 1 < NT; ++k) {
      const long double sign = (k % 2 == 0) ? -1.0L : 1.0L;
      fact *= (long double)(k + 1);
      scale /= kErfcPer;
      c[k + 1] = sign * c2 * hcur * e * scale / fact;
      const long double hnext = 2.0L * x * hcur - 2.0L * (long double)k * hprev;
      hprev = hcur;
      hcur = hnext;
    }
    for (int n = NT - 1; n >= kErfcTerms; --n) {
      const long double w = c[n] / cheb[n][n];
      for (int k = 0; k <= n; ++k) c[k] -= w * cheb[n][k];
    }
    for (int k = 0; k < kErfcTerms; ++k) out[j * kErfcTerms + k] = (double)c[k];
  }
}

}  // namespace cpm
