// Device code of the MI355X likelihood engine (gfx950).
//
//   invariants_kernel   once per event set: FP64 kinematics -> structure-of-arrays
//                       columns (breakup momenta, sines, phi as cos/sin, the Z-chain
//                       lineshape factors and angular factors of Eq. 10)
//   amp_kernel          per call: Eq. (2)-(5), (10)-(12) per event, -2 ln L terms and
//                       the adjoint of S with respect to every coupling and the
//                       floating masses/widths, reduced per block
//   reduce_final        fixed-order compensated sum of the block partials
//   generators          Philox4x32-10 phase space, and accept-reject samples of the model (toys)
//
// Wavefronts are 64 lanes.  Every reduction is atomic-free and in a fixed order,
// so results are bitwise reproducible run to run.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kpsi_internal.h"
#include "kpsi_math.h"

namespace kpsi {

// ------------------------------------------------------------------ math helpers
// rcp_, rsq_, fma_, the barrier polynomials and the angular functions: kpsi_math.h
// Smallest density a data event may have (exclusive): the FP32 path counts an event whose density
// is below the smallest normal float as a bad event.
template <typename T> __device__ __forceinline__ constexpr T pos_floor() {
  if constexpr (std::is_same_v<T, float>) return 1.17549435e-38f;
  else return T(0);
}

template <typename T> __device__ __forceinline__ T ldnt(const T* p) { return __builtin_nontemporal_load(p); }
// Load at a uniform base plus a 32-bit per-lane byte offset: this maps onto the
// scalar-base + vector-offset address form, so no per-lane 64-bit address arithmetic.  The
// 32-byte FP64 column groups are loaded non-temporally; everything else with plain loads, which
// measured 3% faster than non-temporal ones in the FP32 kernel (and 1% slower in the FP64 one).
template <typename T> __device__ __forceinline__ T ldoff(const T* base, uint32_t off_bytes) {
  const T* p = (const T*)((const char*)base + off_bytes);
  if constexpr (sizeof(T) == 4 * sizeof(double)) return __builtin_nontemporal_load(p);
  else return *p;
}

template <typename P> using lds_ptr = __attribute__((address_space(3))) P*;   // LDS (32-bit address)

// FP64: x added to this thread's own LDS slot by an LDS add without a returned value, so nothing
// waits for the slot.  (The FP32 kernel reads, adds and writes: the LDS add of a float runs at a
// tenth of the rate here, 570 against 50 us for 3e6 events.)
__device__ __forceinline__ void lds_add(lds_ptr<double> p, double x) { __builtin_amdgcn_ds_atomic_fadd_f64(p, x); }

// ------------------------------------------------------------------ invariants
// Columns written per event (type T, in groups of four at col_at(k, e, ld)):
//   K* chain  : m, q(m), p_B(m), cos/sin theta_K*, cos/sin theta_J/psi, cos/sin phi, and
//               q/m (column 10)
//   Z chain   : m^2_Jpsi pi (column 9), gZ = q/m_Jpsi pi (column 11), and the complex angular
//               factors Zang[l'][xi = +1] of Eq. (10) for l' = 0 (columns 12-13) and l' = +-1
//               combined through Eq. 11 (columns 14-15), each multiplied by
//               nZ = (p_B/M_B) / sqrt(1 + (r_B p_B)^2), the factor common to every Z amplitude.
//               The xi = -1 factors are (-Re, Im) of the xi = +1 ones and are not stored.
//               With free Z helicities (zfree), columns 14-15 hold F++ = Zang[+1][+1] and
//               16-17 F+- = Zang[+1][-1]; the l' = -1 factors are Zang[-1][+1] = -conj(F+-)
//               and Zang[-1][-1] = -conj(F++).
// All arithmetic in double.
__device__ __forceinline__ void invariants(const Kin& k, double m, double cK, double cJ, double ph, bool with_z,
                                           bool zfree, double* c, double* diag) {
  // One-time kinematics without contraction: at the threshold and end point of m_Kpi the
  // breakup momenta then round to exactly zero, as the plain double-precision definition does.
#pragma clang fp contract(off)
  const double mB = k.mB, mJ = k.mJ, mK = k.mK, mP = k.mPi;
  // two-body momenta in the K pi frame and in the B frame
  const double s = m * m;
  const double q2 = (s - (mK + mP) * (mK + mP)) * (s - (mK - mP) * (mK - mP));
  const double q = q2 > 0.0 ? sqrt(q2) / (2.0 * m) : 0.0;
  const double mB2 = mB * mB;
  const double pb2 = (mB2 - (mJ + m) * (mJ + m)) * (mB2 - (mJ - m) * (mJ - m));
  const double pB = pb2 > 0.0 ? sqrt(pb2) / (2.0 * mB) : 0.0;
  const double sK = sqrt(fmax(0.0, (1.0 - cK) * (1.0 + cK)));
  const double sJ = sqrt(fmax(0.0, (1.0 - cJ) * (1.0 + cJ)));
  double sph, cph;
  sincos(ph, &sph, &cph);
  c[0] = m;
  c[1] = q;
  c[2] = pB;
  c[3] = cK;
  c[4] = sK;
  c[5] = cJ;
  c[6] = sJ;
  c[7] = cph;
  c[8] = sph;
  c[10] = (q / m);
  if (!with_z && !diag) return;

  // J/psi rest frame, reached by a boost along z from the B frame, in which the K pi
  // system moves along +z and the J/psi along -z.  The K pi system moves along +z in
  // the J/psi frame with gamma = p_Kpi.p_J/(m mJ) and gamma*beta = pB mB/(m mJ).
  const double EK = sqrt(mK * mK + q * q), EP = sqrt(mP * mP + q * q);
  const double g = (mB2 - s - mJ * mJ) / (2.0 * m * mJ);
  const double gb = pB * mB / (m * mJ);
  // K and pi momenta in the J/psi frame (x: K side of the hadron plane)
  const double kx = q * sK, kz = g * (q * cK) + gb * EK;
  const double px = -q * sK, pz = g * (-q * cK) + gb * EP;
  const double Epi = g * EP + gb * (-q * cK);
  // m^2_Jpsi pi = mJ^2 + mpi^2 + 2 mJ E_pi(J/psi frame)
  const double mz2 = mJ * mJ + mP * mP + 2.0 * mJ * Epi;
  const double mz = sqrt(mz2);
  // cos theta_Z from invariants: K and pi energies and momenta in the J/psi pi frame
  const double EKz = (mB2 - mz2 - mK * mK) / (2.0 * mz);
  const double EPz = (mz2 + mP * mP - mJ * mJ) / (2.0 * mz);
  const double pKz = sqrt(fmax(0.0, EKz * EKz - mK * mK)), pPz = sqrt(fmax(0.0, EPz * EPz - mP * mP));
  const double dotKP = EKz * EPz - 0.5 * (s - mK * mK - mP * mP);
  double cZ = (pKz * pPz > 0.0) ? dotKP / (pKz * pPz) : 1.0;
  cZ = fmin(1.0, fmax(-1.0, cZ));
  const double sZ = sqrt(fmax(0.0, (1.0 - cZ) * (1.0 + cZ)));
  // Z-chain frame in the J/psi frame: n2 = -pi direction, x2 = K side perpendicular to n2
  const double pn = sqrt(px * px + pz * pz);
  const double n2x = -px / pn, n2z = -pz / pn;       // (y component is zero: hadron plane is x-z)
  const double kd = kx * n2x + kz * n2z;
  double x2x = kx - kd * n2x, x2z = kz - kd * n2z;
  const double kn = sqrt(x2x * x2x + x2z * x2z);
  if (kn * kn > 1e-24 * (kx * kx + kz * kz)) { x2x /= kn; x2z /= kn; }
  else {  // collinear hadrons: take the K* frame's x axis projected off n2
    const double d1 = n2x;
    x2x = 1.0 - d1 * n2x; x2z = -d1 * n2z;
    const double nn = sqrt(x2x * x2x + x2z * x2z);
    x2x /= nn; x2z /= nn;
  }
  // y2 = n2 x x2 (only the y component survives for vectors in the x-z plane)
  const double y2y = n2z * x2x - n2x * x2z;
  // mu+ direction in the J/psi frame: theta_J/psi from n1 = -z, azimuth phi from x1 = +x,
  // right-handed about n1 (y1 = -y)
  const double ux = sJ * cph, uy = -sJ * sph, uz = -cJ;
  const double ct = ux * n2x + uz * n2z;                 // cos theta~
  const double ux2 = ux * x2x + uz * x2z;                 // sin theta~ cos phi~
  const double uy2 = uy * y2y;                            // sin theta~ sin phi~
  const double st = sqrt(ux2 * ux2 + uy2 * uy2);
  double cpt = 1.0, spt = 0.0;
  if (st > 0.0) { cpt = ux2 / st; spt = uy2 / st; }
  // muon helicity frame x axes: x' = cos(theta)(cos(phi) x + sin(phi) y) - sin(theta) n
  //  K* chain: x1 = +x, y1 = -y, n1 = -z
  const double xa_x = cJ * cph, xa_y = -cJ * sph, xa_z = sJ;
  //  Z chain
  const double xb_x = ct * (cpt * x2x) - st * n2x;
  const double xb_y = ct * (spt * y2y);
  const double xb_z = ct * (cpt * x2z) - st * n2z;
  // alpha: rotation about mu+ taking the Z-chain axis xb onto the K*-chain axis xa
  const double ca = xb_x * xa_x + xb_y * xa_y + xb_z * xa_z;
  const double crx = xb_y * xa_z - xb_z * xa_y, cry = xb_z * xa_x - xb_x * xa_z, crz = xb_x * xa_y - xb_y * xa_x;
  const double sa = crx * ux + cry * uy + crz * uz;
  if (diag) {
    diag[0] = mz; diag[1] = cZ; diag[2] = ct; diag[3] = atan2(spt, cpt); diag[4] = atan2(sa, ca);
  }
  if (!with_z) return;
  // Z lineshape factors (B -> Z K with L_B = 1, Z -> J/psi pi with L_R = 0)
  const double qz2 = (mz2 - (mJ + mP) * (mJ + mP)) * (mz2 - (mJ - mP) * (mJ - mP));
  const double qz = qz2 > 0.0 ? sqrt(qz2) / (2.0 * mz) : 0.0;
  const double pbz2 = (mB2 - (mz + mK) * (mz + mK)) * (mB2 - (mz - mK) * (mz - mK));
  const double pbz = pbz2 > 0.0 ? sqrt(pbz2) / (2.0 * mB) : 0.0;
  const double zb = k.rB * pbz * k.rB * pbz;
  const double nZ = (pbz / mB) / sqrt(1.0 + zb);
  c[9] = mz2;
  c[11] = (qz / mz);
  // Angular factors of Eq. (10): d^1_{0l'}(theta_Z) e^{i l' phi~} d^1_{l' xi}(theta~) e^{i xi alpha},
  // times nZ
  const double r2 = 0.7071067811865475244 * nZ;
  //  l' = 0:  xi = +1: cZ st/sqrt2 e^{i alpha};  xi = -1: -cZ st/sqrt2 e^{-i alpha}
  //  (xi = -1 is -z0 ca + i z0 sa: minus the real part, the same imaginary part)
  const double z0 = cZ * st * r2;
  c[12] = (z0 * ca);
  c[13] = (z0 * sa);
  //  l' = +-1 (H'_{-1} = H'_{+1}):  xi = +1: sZ/sqrt2 (ct cpt + i spt) e^{i alpha}
  //                                 xi = -1: sZ/sqrt2 (-ct cpt + i spt) e^{-i alpha}, again
  //                                 (-Re, Im) of the xi = +1 factor
  const double z1 = sZ * r2;
  if (zfree) {
    // l' = +1 alone: d^1_{0,1}(theta_Z) = sZ/sqrt2, d^1_{1,xi}(theta~) = (1 + xi ct)/2, phases
    // e^{i (phi~ + xi alpha)}
    const double up = 0.5 * z1 * (1.0 + ct), dn = 0.5 * z1 * (1.0 - ct);
    c[14] = (up * (cpt * ca - spt * sa));
    c[15] = (up * (spt * ca + cpt * sa));
    c[16] = (dn * (cpt * ca + spt * sa));
    c[17] = (dn * (spt * ca - cpt * sa));
    return;
  }
  const double pr = ct * cpt, pi_ = spt;
  c[14] = (z1 * (pr * ca - pi_ * sa));
  c[15] = (z1 * (pr * sa + pi_ * ca));
}

template <typename T>
__global__ __launch_bounds__(256) void invariants_kernel(InvArgs<T> a) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.n) return;
  double c[18];
  const double m = a.obs[0][e], ck = a.obs[1][e], cj = a.obs[2][e], ph = a.obs[3][e];
  if (a.bad) {
    const double tol = 1e-12;
    const bool ok = m >= a.lo - tol && m <= a.hi + tol && fabs(ck) <= 1.0 + tol && fabs(cj) <= 1.0 + tol &&
                    fabs(ph) <= 3.14159265358979323846 + tol;
    if (!ok) *a.bad = 1u;   // (the same value from whichever events: no atomic operation)
  }
  invariants(a.kin, m, ck, cj, ph, a.with_z, a.zfree, c, a.diag ? a.diag + 5 * e : nullptr);
#pragma unroll
  for (int k = 0; k < 18; ++k) {
    const bool z = k == 9 || k > 10;   // a Z column
    if (!z || (a.with_z && (k < 16 || a.zfree))) a.cols[col_at(k, e, a.ld)] = (T)c[k];
  }
}

// ------------------------------------------------------------------ generators
// Philox4x32-10 from its published definition (Salmon et al., SC'11).
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint64_t p0 = (uint64_t)0xD2511F53u * c[0];
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c[2];
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c[1] ^ k0;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c[3] ^ k1;
    c[1] = (uint32_t)p1;
    c[3] = (uint32_t)p0;
    c[0] = n0;
    c[2] = n2;
  }
}
__device__ __forceinline__ void u2(uint64_t e, uint32_t w2, uint32_t w3, uint64_t seed, double& ua, double& ub) {
  uint32_t c[4] = {(uint32_t)e, (uint32_t)(e >> 32), w2, w3};
  philox4x32_10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
  ua = (double)(((uint64_t)(c[0] >> 5) << 26) | (uint64_t)(c[1] >> 6)) * (1.0 / 9007199254740992.0);
  ub = (double)(((uint64_t)(c[2] >> 5) << 26) | (uint64_t)(c[3] >> 6)) * (1.0 / 9007199254740992.0);
}

// Trial t of the phase-space proposal e: m_Kpi flat in the mass range, accepted if u wmax < p_B(m)
// q(m).  The test is evaluated without contraction so it is bit-identical to a plain FP64 host; the
// squares decide it without roots and quotients where they differ by more than 1e-10 of either,
// which is far more than both forms' roundings.
__device__ __forceinline__ bool phsp_trial(const Kin& k, uint64_t seed, double wmax, uint64_t e, uint32_t t,
                                           double& m) {
#pragma clang fp contract(off)
  const double lo = k.mK + k.mPi, hi = k.mB - k.mJ;
  const double c1 = (k.mK + k.mPi) * (k.mK + k.mPi), c2 = (k.mK - k.mPi) * (k.mK - k.mPi);
  double ua, ub;
  u2(e, t, 0u, seed, ua, ub);
  m = lo + (hi - lo) * ua;
  // p_B(m) = sqrt((mB^2 - (mJ+m)^2)(mB^2 - (mJ-m)^2)) / (2 mB);  q(m) analogous
  const double s = k.mB * k.mB;
  const double pa = s - (k.mJ + m) * (k.mJ + m);
  const double pb = s - (k.mJ - m) * (k.mJ - m);
  const double px = pa * pb;
  const double mm = m * m;
  const double qa = mm - c1;
  const double qb = mm - c2;
  const double qx = qa * qb;
  if (px > 0.0 && qx > 0.0) {
    const double w = ub * wmax, l = w * w * (16.0 * s * mm), r = px * qx;
    if (l < r * (1.0 - 1e-10)) return true;
    if (l > r * (1.0 + 1e-10)) return false;
  }
  const double pB = px <= 0.0 ? 0.0 : sqrt(px) / (2.0 * k.mB);
  const double q = qx <= 0.0 ? 0.0 : sqrt(qx) / (2.0 * m);
  return ub * wmax < pB * q;
}
constexpr uint32_t kTrials = 4096;   // trials of a proposal before it counts as failed
// Angles of the proposal e from counters (e, 0, 1) and (e, 0, 2), and the number kept for the
// accept-reject test.
__device__ __forceinline__ void phsp_angles(uint64_t e, uint64_t seed, double& ck, double& cj, double& phi,
                                            double& spare) {
#pragma clang fp contract(off)
  double ua, ub;
  u2(e, 0u, 1u, seed, ua, ub);
  ck = 2.0 * ua - 1.0;
  cj = 2.0 * ub - 1.0;
  u2(e, 0u, 2u, seed, ua, spare);
  phi = 3.14159265358979323846 * (2.0 * ua - 1.0);
}

// Seeded analytic acceptance (same definition as the generator's truth efficiency):
// eps = 0.9 prod_d (1 - delta (1 - t_d)/2), t_d = sum_l a_dl P_l(u_d) / sum_l |a_dl|.
// (t_d is in [-1, 1] and delta in (0, 1): eps is at most 0.9.)
__device__ __forceinline__ double acceptance(const double* co, double delta, double lo, double hi, double m, double cK,
                                             double cJ, double ph) {
#pragma clang fp contract(off)
  const double u[4] = {2.0 * (m - lo) / (hi - lo) - 1.0, cK, cJ, ph / 3.14159265358979323846};
  double eps = 0.9;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const double x = u[d];
    const double P1 = x, P2 = 0.5 * (3.0 * x * x - 1.0), P3 = 0.5 * (5.0 * x * x * x - 3.0 * x);
    const double num = co[3 * d] * P1 + co[3 * d + 1] * P2 + co[3 * d + 2] * P3;
    const double den = fabs(co[3 * d]) + fabs(co[3 * d + 1]) + fabs(co[3 * d + 2]);
    const double t = den > 0.0 ? num / den : 0.0;
    eps *= 1.0 - delta * (1.0 - t) / 2.0;
  }
  return eps;
}

// ------------------------------------------------------------------ cross-lane exchange
// One step of a transposed butterfly at distance D = 32 or 16 on a pair of per-lane values:
// lanes whose bit log2(D) is clear end with (their lo, the partner's lo), the others with
// (the partner's hi, their hi), so lo + hi is the pair sum each lane keeps.  v_permlane32_swap
// exchanges lanes 32-63 of its first operand with lanes 0-31 of its second; v_permlane16_swap
// exchanges the odd 16-lane rows of the first with the even rows of the second.
template <int D> __device__ __forceinline__ void swap_halves(double& lo, double& hi) {
  static_assert(D == 32 || D == 16, "lane-swap distance");
  const uint64_t a = __builtin_bit_cast(uint64_t, lo), b = __builtin_bit_cast(uint64_t, hi);
  const unsigned al = (unsigned)a, ah = (unsigned)(a >> 32), bl = (unsigned)b, bh = (unsigned)(b >> 32);
  unsigned nl0, nl1, nh0, nh1;
  if constexpr (D == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    nl0 = l[0]; nl1 = l[1]; nh0 = h[0]; nh1 = h[1];
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    nl0 = l[0]; nl1 = l[1]; nh0 = h[0]; nh1 = h[1];
  }
  lo = __builtin_bit_cast(double, ((uint64_t)nh0 << 32) | nl0);
  hi = __builtin_bit_cast(double, ((uint64_t)nh1 << 32) | nl1);
}
template <int D> __device__ __forceinline__ void swap_halves(float& lo, float& hi) {
  static_assert(D == 32 || D == 16, "lane-swap distance");
  const unsigned a = __builtin_bit_cast(unsigned, lo), b = __builtin_bit_cast(unsigned, hi);
  unsigned n0, n1;
  if constexpr (D == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    n0 = r[0]; n1 = r[1];
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    n0 = r[0]; n1 = r[1];
  }
  lo = __builtin_bit_cast(float, n0);
  hi = __builtin_bit_cast(float, n1);
}
// The value of the partner lane in a butterfly step of width H = 8, 4, 2, 1 within each 16-lane
// row, by DPP: row_mirror (lane i <-> 15 - i), row_half_mirror (i <-> 7 - i in each half row),
// and the quad permutations (i <-> i ^ 2, i <-> i ^ 1).  Each pairs lanes whose bit log2(H)
// differs and whose higher bits agree, which is what the transposed butterfly needs.
template <int H> __device__ __forceinline__ unsigned dpp_partner(unsigned x) {
  static_assert(H == 8 || H == 4 || H == 2 || H == 1, "butterfly width");
  constexpr int ctrl = H == 8 ? 0x140 : (H == 4 ? 0x141 : (H == 2 ? 0x4E : 0xB1));
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xF, 0xF, false);
}
template <int H> __device__ __forceinline__ float dpp_partner(float x) {
  return __builtin_bit_cast(float, dpp_partner<H>(__builtin_bit_cast(unsigned, x)));
}
template <int H> __device__ __forceinline__ double dpp_partner(double x) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint64_t lo = dpp_partner<H>((unsigned)b), hi = dpp_partner<H>((unsigned)(b >> 32));
  return __builtin_bit_cast(double, (hi << 32) | lo);
}

// ------------------------------------------------------------------ compensated sums
__device__ __forceinline__ void neumaier(double& s, double& c, double x) {
  const double t = s + x;
  c += (fabs(s) >= fabs(x)) ? (s - t) + x : (x - t) + s;
  s = t;
}
// Merge of two compensated sums; the two-sum error term is exact, so merging (a, b) and
// (b, a) gives the same result.
__device__ __forceinline__ void two_sum_merge(double& s, double& c, double s2, double c2) {
  const double t = s + s2;
  const double bp = t - s;
  const double err = (s - (t - bp)) + (s2 - bp);
  s = t;
  c = c + c2 + err;
}

// ------------------------------------------------------------------ per-event amplitude
template <typename T> struct Cx { T re, im; };
template <typename T> __device__ __forceinline__ void cmac(Cx<T>& acc, T ar, T ai, T br, T bi) {
  acc.re = fma_(ar, br, fma_(-ai, bi, acc.re));
  acc.im = fma_(ar, bi, fma_(ai, br, acc.im));
}

// (gr, gi) += A V: the per-event gradient contribution, fused into the accumulators
template <typename T> __device__ __forceinline__ void cacc(T& gr, T& gi, const Cx<T>& A, const Cx<T>& V) {
  gr = fma_(A.re, V.re, fma_(-A.im, V.im, gr));
  gi = fma_(A.re, V.im, fma_(A.im, V.re, gi));
}

// Lineshape-parameter sums of one floating resonance.  B = 1/(M^2 - m^2 - i P g) is its bare
// Breit-Wigner and Q = sum_lambda h_lambda V_lambda its adjoint weight, so X = B Q is the
// resonance's share of dS/dA times A.  With A = K n B (K and P depending on M, P also on
// Gamma0 = P/PoG) and Z = B X:
//   dS/dM      = Re[X (kappa - (2M - i P' g) B)] = kappa Re X - 2M Re Z - P' g Im Z
//   dS/dGamma0 = Re[X i PoG g B]                 = -PoG g Im Z
// (kappa = d ln K/dM, P' = dP/dM).  The constants leave the event loop: the kernel sums Re Z and
// g Im Z, and the host combines them with sum Re X, which follows from the coupling sums
// (finish_record).  That is 9 instructions per event and floating resonance where the two
// derivatives and their routing to the slots took 20.
template <typename T> __device__ __forceinline__ void flt_sums(const Cx<T>& B, const Cx<T>& Q, T g, T& sR, T& sI) {
  const T Xr = fma_(B.re, Q.re, -B.im * Q.im), Xi = fma_(B.re, Q.im, B.im * Q.re);
  sR = fma_(Xr, B.re, fma_(-Xi, B.im, sR));
  sI = fma_(g, fma_(Xr, B.im, Xi * B.re), sI);
}

template <class Sh> __host__ __device__ constexpr int acc_base(int J) {   // accumulator offset of spin J
  int b = 3;
  for (int j = 0; j < J; ++j) b += Sh::N[j] * (j == 0 ? 2 : 6);
  return b;
}

// Accumulator indices (per block record of NACC doubles):
//   0, 1 : main sum and its (negated Kahan) compensation, total = [0] + [1]
//          (data: sum ln S; norm: sum eps S).  Gradient mode, flavour tags with the Eq. 14
//          mixture: data slot 0 is the whole sum and slot 1 the - flavour's sum of w S
//   2    : number of data events with S <= 0 or non-finite
//   then per K* slot (spin order) 2 (spin 0) or 6 (lambda = -1, 0, +1) values re/im of
//   sum w * dS/dH' with H' = K H but for constant factors (before the factor 2), then per Z slot 4 values
//   (lambda' = 0, +-1; free helicities 0, +1, -1), then 2 per floating slot (sum Re Z, sum g Im Z: flt_sums).

// The gradient kernel of the large shape asks for 4 (FP32) or 2 (FP64) wavefronts per SIMD, at
// most 128 or 256 registers; its spin-1..3 accumulators live in LDS to make room (36 values x
// 256 threads: 36 KB per block in FP32, 4 blocks per compute unit; 72 KB in FP64, 2 blocks).
// The FP64 likelihood-only and density kernels of the large shape ask for 4 (128 registers).
// The FP32 likelihood-only one without tags asks for 8 (64
// registers): it waits for memory more than it issues (33.6 against 36.9 us for 3e6 events).
template <typename T, class Sh, int MODE, bool CC> struct AmpWaves {
  static constexpr bool lds = MODE == MODE_GRAD && Sh::LDS_HI > Sh::LDS_LO;
  static constexpr bool f32 = std::is_same<T, float>::value;
  static constexpr int v = MODE == MODE_TOYS ? 2 : (lds ? (f32 ? 4 : 2) : Sh::NK == 1 ? 1 : !f32 ? 4 : CC ? 1 : 8);
};
// CC: flavour-tagged events (text after Eq. 12).  Data events carry a tag q = +-1 and are read
// with phi -> q phi, plus the other flavour with the mistag weight; the normalisation events run
// twice, as record 1 (phi) and record 2 (-phi), blocks [nb_data + nb_mc, nb_data + 2 nb_mc).
// ZF: one Z whose H'_{+1} and H'_{-1} are independent couplings (no Eq. 11 relation); its
// lambda' = -1 accumulators use the record slots of the second Z.
template <typename T, class Sh, int MODE, bool CC, bool ZF>
__global__ __launch_bounds__(256, (AmpWaves<T, Sh, MODE, CC>::v)) void amp_kernel(const typename AmpArgsOf<T, Sh, MODE>::type a) {
  constexpr int NK = Sh::NK;
  static_assert(!ZF || Sh::NZ >= 2, "free Z helicities use the second Z's record slots");
  constexpr int NZ = ZF ? 1 : Sh::NZ;   // Z slots evaluated
  constexpr bool GRAD = (MODE == MODE_GRAD);
  constexpr bool TOYS = (MODE == MODE_TOYS);   // the listed proposals of a ToyArgs chunk
  using A_t = typename AccType<T>::type;   // per-thread gradient accumulator type

  const int set = (blockIdx.x < (unsigned)a.nb_data)
                      ? 0
                      : ((!CC || blockIdx.x < (unsigned)(a.nb_data + a.nb_mc)) ? 1 : 2);
  const int src = set == 0 ? 0 : 1;   // event set read by this block
  const int64_t blk = (int64_t)blockIdx.x - (set == 0 ? 0 : (set == 1 ? a.nb_data : a.nb_data + a.nb_mc));
  const uint32_t tl = TOYS ? blockIdx.x % kToyLists : 0;   // toys: this block's list
  int64_t n = a.n[src];
  if constexpr (TOYS) n = (int64_t)a.toys.stat[kToyListed + 16 * tl];
  const T* __restrict__ col = a.cols[src];
  const int64_t ld = a.ld[src];
  auto first = [&](int64_t b) { return (b * a.per[src] + (b < a.more[src] ? b : a.more[src])) * 256; };
  const int64_t e0 = TOYS ? 0 : first(blk), e2 = TOYS ? n : first(blk + 1);
  const int64_t e1 = e2 < n ? e2 : n;

  // normalisation: Kahan pair; data: product of the terms as ms 2^mexp until the loop is done (one
  // variable for both: the FP32 likelihood kernel has no register to spare)
  double ms = set == 0 ? 1.0 : 0.0, mc = 0.0;
  int mexp = 0;
  float nbad = 0.f;   // events with a non-positive or non-finite density (exact count; the call then
                      // fails, so what they add to the sums does not matter)
  // Eq. 14 mixture on the data set: background weight k from the reduced normalisation total
  const bool mix = (set == 0) && a.bkg_data != nullptr;
  T kb = T(0), kb2 = T(0);   // background weight k (flavour tags: of the + and - flavours)
  if (mix) {
    constexpr int NR = CC ? 2 : 1;   // normalisation records: phi (and -phi with tags)
    double tot[2] = {0.0, 0.0};
    if (a.mc_part) {
      // sum eps S over the normalisation blocks in a fixed order (the same in every block):
      // strided compensated sums per lane, a butterfly of exact two-sum merges in each
      // wavefront (both partners get the same result), then the four wavefronts in order
      __shared__ double kred[4][2 * NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        double s = 0.0, c = 0.0;
        const double* mp = a.mc_part + r * a.mc_nb;
        for (int b = threadIdx.x; b < a.mc_nb; b += 256) {
          neumaier(s, c, mp[b]);
          neumaier(s, c, mp[a.pstride + b]);   // value 1: the Kahan correction
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) two_sum_merge(s, c, __shfl_xor(s, off, 64), __shfl_xor(c, off, 64));
        if ((threadIdx.x & 63) == 0) {
          kred[threadIdx.x >> 6][2 * r] = s;
          kred[threadIdx.x >> 6][2 * r + 1] = c;
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        double s = kred[0][2 * r], c = kred[0][2 * r + 1];
        for (int w = 1; w < 4; ++w) two_sum_merge(s, c, kred[w][2 * r], kred[w][2 * r + 1]);
        tot[r] = s + c;
      }
    } else {
      tot[0] = a.norm_total[0] + a.norm_total[1];
      if (CC) tot[1] = a.norm_total[NACC] + a.norm_total[NACC + 1];
    }
    if constexpr (CC) {
      // N_q = (1 - w) I(q) + w I(-q) for the event's flavour q
      const double wm = (double)a.mistag, kp = 1.0 - wm;
      kb = (T)(a.bkg_coef * (kp * tot[0] + wm * tot[1]));
      kb2 = (T)(a.bkg_coef * (kp * tot[1] + wm * tot[0]));
    } else {
      kb = (T)(a.bkg_coef * tot[0]);
    }
  }
  A_t ws = A_t(0);    // sum_i w_i S_i (mixture, gradient mode; with tags: the + flavour's events)
  A_t ws2 = A_t(0);   // with tags: the same over the - flavour's events
  // accumulators gk[LO, HI) live in this thread's LDS column accl[.][tid] (gradient kernel)
  constexpr bool LDSACC = GRAD && (Sh::LDS_HI > Sh::LDS_LO);
  constexpr int LO = LDSACC ? Sh::LDS_LO : 0, HI = LDSACC ? Sh::LDS_HI : 0;
  __shared__ A_t accl[HI > LO ? HI - LO : 1][256];
  if constexpr (LDSACC) {
#pragma unroll
    for (int i = 0; i < HI - LO; ++i) accl[i][threadIdx.x] = A_t(0);
  }
  A_t gk[Sh::NKACC > 0 ? Sh::NKACC : 1];
  A_t gz[NZ > 0 ? 4 * Sh::NZ : 1];
  static_assert(NFL == 2, "floating accumulators are named registers for two slots");
  A_t gM0 = 0, gG0 = 0, gM1 = 0, gG1 = 0;   // lineshape sums of floating slots 0 and 1 (flt_sums)
  if constexpr (GRAD) {
#pragma unroll
    for (int i = 0; i < Sh::NKACC; ++i) gk[i] = 0;
#pragma unroll
    for (int i = 0; i < 4 * Sh::NZ; ++i) gz[i] = 0;
  }

  using V4 = T __attribute__((ext_vector_type(4)));
  const V4* __restrict__ gb = (const V4*)col + e0;   // column group 0 at this block's first event
  const uint32_t n_blk = (uint32_t)(e1 > e0 ? e1 - e0 : 0);
  // Column groups of this thread's event.  The FP64 gradient kernel of the large shape (two wavefronts
  // per SIMD) fetches the next event's as soon as the current ones are used up, before the
  // accumulation (a clamped index past the last event: no branch); 108 against 111 us for 3e6 events.
  // With free helicities the last pass of a block branches over it: the kernel then needs no scratch
  // (3e6 events 114.8 against 116.3 us, 48e3 events 20.8 against 21.5; without them 110.9 against 109.2).
  // The others load them where the event begins, and the Z columns where the Z chain does: the live
  // registers cost the FP32 gradient kernel more than the latency (51.5 against 50.5 us) and the
  // likelihood-only ones wavefronts (FP32: 37 against 35 us), and the small shape reads at the
  // memory's rate (FP64 gradient: 57 against 53 us).
  constexpr int NG = NZ > 0 ? (ZF ? 5 : 4) : 3;
  constexpr bool PRE = GRAD && std::is_same_v<T, double> && NK > 1;
  V4 grp[NG];
  uint32_t prop = 0;       // toys: this thread's proposal and the number of its accept-reject test
  double spare = 0.0, eps_true = 1.0;
  auto fetch = [&](uint32_t i) {
    if constexpr (TOYS) {
      const ToyArgs& ty = a.toys;
      prop = ty.list[tl * (((uint32_t)ty.rounds << kRoundBits) / kToyLists) + i];
      const double m = ty.m[prop];
      double ck, cj, phi, c[20];
      phsp_angles((uint64_t)ty.e0 + prop, ty.seed, ck, cj, phi, spare);
      invariants(ty.kin, m, ck, cj, phi, a.cnt[5] > 0, ZF, c, nullptr);
      if (ty.acc_on)
        eps_true = acceptance(ty.coef, ty.delta, ty.kin.mK + ty.kin.mPi, ty.kin.mB - ty.kin.mJ, m, ck, cj, phi);
#pragma unroll
      for (int k = 0; k < NG; ++k)
        if (k < 3 || a.cnt[5] > 0) grp[k] = V4{(T)c[4 * k], (T)c[4 * k + 1], (T)c[4 * k + 2], (T)c[4 * k + 3]};
      return;
    }
    const uint32_t ob4 = i * (uint32_t)sizeof(V4);
#pragma unroll
    for (int k = 0; k < (PRE ? NG : 3); ++k)
      if (k < 3 || a.cnt[5] > 0) grp[k] = ldoff(gb + k * ld, ob4);
  };
  if (PRE && threadIdx.x < n_blk) fetch(threadIdx.x);
  // (Issue-bound kernels only: where memory is waited for, FP32 likelihood and small shape, the fixed
  // order cost 2 us of 23.)
  // Wavefronts further from their block's end issue first.  Left to the hardware, the oldest ready
  // wavefront issues first, so of the blocks sharing a compute unit (all with the same number of
  // events) one ends early and the last runs with idle issue slots: on average 3.5 of 4 (FP32) and
  // 1.7 of 2 (FP64) wavefronts per SIMD were left.  Lowering a wavefront's priority as it nears its end
  // lets the others catch up.
  constexpr bool PRIO = NK > 1 && (GRAD || std::is_same_v<T, double>) && !TOYS;
  if constexpr (PRIO) __builtin_amdgcn_s_setprio(3);
  uint32_t left = (n_blk + 255) / 256;   // passes of this block still to do
  for (uint32_t i = TOYS ? blockIdx.x / kToyLists * 256 + threadIdx.x : threadIdx.x; i < n_blk;
       i += TOYS ? gridDim.x / kToyLists * 256 : 256) {
    if constexpr (PRIO) {
      if (left == 6) __builtin_amdgcn_s_setprio(2);
      else if (left == 3) __builtin_amdgcn_s_setprio(1);
      else if (left == 1) __builtin_amdgcn_s_setprio(0);
      --left;
    }
    const int64_t e = e0 + i;
    const uint32_t ob = i * (uint32_t)sizeof(T);
    const auto& ka = *kernarg_laundered<AmpArgs<T, Sh>>();
    if constexpr (!PRE) fetch(i);
    // this thread's LDS accumulator column, re-derived opaquely each event so the compiler keeps
    // the accumulators in LDS instead of promoting them back into registers across the loop
    lds_ptr<A_t> accb = (lds_ptr<A_t>)&accl[0][threadIdx.x];
    if constexpr (LDSACC) asm volatile("" : "+v"(accb));
    const T m = grp[0].x, q = grp[0].y, pB = grp[0].z, cK = grp[0].w;
    const T sK = grp[1].x, cJ = grp[1].y, sJ = grp[1].z, cph = grp[1].w;
    const T sph = grp[2].x, qm = grp[2].z;   // q/m from the event columns

    const T qq = q * q;
    const T zR = ka.rR2 * qq;
    const T zB = ka.rB2 * (pB * pB);

    // ---- K* lineshapes (Eq. 2-3) and coupling sums T_{J lambda}
    // Each resonance's amplitude is K n_J(m) B_R(m) with B_R = 1/(M^2 - m^2 - i P g_J(m)) the
    // bare Breit-Wigner, K the per-resonance constant and n_J the per-spin barrier and momentum
    // factor.  K is folded into the couplings on the host and n_J into the angular
    // factors of its spin, so each resonance costs one complex reciprocal: Amp holds B_R.
    Cx<T> Amp[NK > 0 ? NK : 1];
    T gJv[5] = {T(0), T(0), T(0), T(0), T(0)};   // g_J(m) per spin (width derivative)
    T nJv[5] = {T(0), T(0), T(0), T(0), T(0)};   // n_J(m) per spin (without the 1/M_B of p_B: host)
    Cx<T> Tl[5][3];
#pragma unroll
    for (int J = 0; J < 5; ++J)
#pragma unroll
      for (int l = 0; l < 3; ++l) Tl[J][l] = Cx<T>{T(0), T(0)};

    // The constants of a resonance are one scalar load (AC).  In FP64 (two wavefronts per SIMD)
    // it is taken one resonance ahead: the load of the next one is issued when the current one's
    // values have arrived (the empty asm is their first use), and the scheduling barrier, which
    // only arithmetic may cross, keeps it there.  Scalar loads return out of order, so every wait
    // is for all of them; loaded where they are used, each resonance waited for its own.  The four
    // wavefronts of FP32 hide those waits, and the fixed order costs more than it gives there
    // (tagged step 90 against 85 us); so it does in the tagged FP64 gradient kernel, whose second
    // reading leaves no registers for the order (3e6 events 187 against 179 us, 28e3 events 21.2 against
    // 19.6, and no scratch).
    using C8 = T __attribute__((ext_vector_type(8)));
    const kconst_ptr<C8> cp = (kconst_ptr<C8>)&ka.cs[0];
    constexpr bool AHEAD = std::is_same_v<T, double> && !(CC && GRAD);
    C8 ahead{};
    if constexpr (AHEAD) ahead = cp[0];
    auto constants = [&](int k) -> C8 {
      if constexpr (AHEAD) {
        asm volatile("" : "+s"(ahead));
        const C8 c = ahead;
        if (k + 1 < NK + Sh::NZ) ahead = cp[k + 1];
        __builtin_amdgcn_sched_barrier(1);
        return c;
      } else {
        return cp[k];
      }
    };
    // Every K* slot of the shape is evaluated: the host gives the slots the model leaves empty
    // zero couplings and the constants M^2 = P = 0 (a finite 1/D = -1/m^2), so they add nothing
    // and need no per-event test (the Z slots keep theirs: models often use one of the two).
    const int lass = ka.lass;
    // LASS (Eq. 7-8): with u = q cot(delta_B) = 1/a + b q^2/2 (finite at threshold),
    // (m/q) sin(delta_B) e^{i delta_B} = m (u + i q)/(u^2 + q^2) and
    // e^{2 i delta_B} = (u + i q)^2/(u^2 + q^2); the resonant term is the
    // Breit-Wigner B times P = M^2 Gamma0/q0 and e^{2 i delta_B}
    auto lass_amp = [&](int k, T P, const Cx<T>& B) -> Cx<T> {
      if (!(lass & (1 << k))) return B;
      const T u = fma_(ka.lhb[k], qq, ka.lai[k]);
      const T dn = rcp_(fma_(u, u, qq));
      const T er = (u * u - qq) * dn, ei = T(2) * u * q * dn;
      const T md = m * dn;
      return Cx<T>{fma_(md, u, P * (er * B.re - ei * B.im)), fma_(md, q, P * (er * B.im + ei * B.re))};
    };
    auto do_spin = [&](auto Jc) {
      constexpr int J = decltype(Jc)::value;
      if constexpr (Sh::N[J] > 0) {
        {
          constexpr int LB = LBof<J>::v;
          const T BR = bpoly<J>(zR), BB = bpoly<LB>(zB);
          const T rJ = rsq_(BR * BB);
          const T nJ = ipow<T, LB>(pB) * ipow<T, J>(qm) * rJ;
          // 1/B_J(z_R) = rJ^2 B_LB(z_B): no second reciprocal
          T gJ = qm;
          if constexpr (J > 0) gJ = qm * ipow<T, J>(qq) * (rJ * rJ * BB);
          gJv[J] = gJ;
          nJv[J] = nJ;
          constexpr int sb = slot_base<Sh>(J);
#pragma unroll
          for (int j = 0; j < Sh::N[J]; ++j) {
            {
              const C8 rc = constants(sb + j);   // M2, P, h
              const T dre = pole_gap_m(rc[0], ka.M2lo[sb + j], m);
              const T dim = rc[1] * gJ;   // M Gamma(m)
              const T inv = rcp_(fma_(dre, dre, dim * dim));
              Cx<T> A{dre * inv, dim * inv};
              if constexpr (J == 0) {
                if (lass) A = lass_amp(sb + j, rc[1], A);
              }
              Amp[sb + j] = A;
              if constexpr (J == 0) {
                cmac(Tl[0][1], rc[4], rc[5], A.re, A.im);
              } else {
#pragma unroll
                for (int l = 0; l < 3; ++l) cmac(Tl[J][l], rc[2 + 2 * l], rc[3 + 2 * l], A.re, A.im);
              }
            }
          }
        }
      }
    };
    do_spin(std::integral_constant<int, 0>{});
    do_spin(std::integral_constant<int, 1>{});
    do_spin(std::integral_constant<int, 2>{});
    do_spin(std::integral_constant<int, 3>{});
    do_spin(std::integral_constant<int, 4>{});

    // ---- angular sums (Eq. 4) and the muon amplitudes rotated to X = (a_+ + a_-)/sqrt2, Y = (a_+ - a_-)/sqrt2
    // (S = |X|^2 + |Y|^2): with the helicity sums U_+- and U_0,
    //   X = e^{i phi} U_+ - e^{-i phi} U_- + Z terms
    //   Y = cos th_J (e^{i phi} U_+ + e^{-i phi} U_-) + sin th_J U_0 + Z terms
    // (d^J_{-10} = -d^J_{10}; the constants are in the couplings): fewer instructions than a_+-1
    // themselves, by about 25% in this part and half in the Z chain, whose factors are real or imaginary.
    // The couplings stay by helicity: as rounded sums and differences, a small one beside a large one would
    // be off by the large one's rounding in every event.
    // (n_J times the angular functions; the n_J of spins absent from the model are zero)
    T dd0[5], dd1[5];
    auto do_ang = [&](auto Jc) {
      constexpr int J = decltype(Jc)::value;
      dd0[J] = nJv[J] * ang0<J>(cK);
      dd1[J] = J > 0 ? nJv[J] * sK * ang1<J>(cK) : T(0);
    };
    do_ang(std::integral_constant<int, 0>{});
    do_ang(std::integral_constant<int, 1>{});
    do_ang(std::integral_constant<int, 2>{});
    do_ang(std::integral_constant<int, 3>{});
    do_ang(std::integral_constant<int, 4>{});
    Cx<T> U0{T(0), T(0)}, Um{T(0), T(0)}, Up{T(0), T(0)};
#pragma unroll
    for (int J = 0; J < 5; ++J) {
      if (Sh::N[J] == 0) continue;
      U0.re = fma_(dd0[J], Tl[J][1].re, U0.re);
      U0.im = fma_(dd0[J], Tl[J][1].im, U0.im);
      if (J > 0) {
        Um.re = fma_(dd1[J], Tl[J][0].re, Um.re);
        Um.im = fma_(dd1[J], Tl[J][0].im, Um.im);
        Up.re = fma_(dd1[J], Tl[J][2].re, Up.re);
        Up.im = fma_(dd1[J], Tl[J][2].im, Up.im);
      }
    }
    // Amplitudes X, Y of the event read with phi -> f phi.  f = -1 is the charge-conjugate decay:
    // sin phi changes its sign, and the Z-chain azimuths phi~ and alpha reverse, which conjugates
    // the Z angular factors.
    auto kstar_at = [&](T f, Cx<T>& X_, Cx<T>& Y_) {
      const T sp = f * sph;
      const Cx<T> p{fma_(cph, Up.re, -sp * Up.im), fma_(cph, Up.im, sp * Up.re)};   // e^{i phi} U_+
      X_ = Cx<T>{fma_(-cph, Um.re, fma_(-sp, Um.im, p.re)), fma_(-cph, Um.im, fma_(sp, Um.re, p.im))};
      const Cx<T> y{fma_(cph, Um.re, fma_(sp, Um.im, p.re)), fma_(cph, Um.im, fma_(-sp, Um.re, p.im))};
      Y_ = Cx<T>{fma_(cJ, y.re, sJ * U0.re), fma_(cJ, y.im, sJ * U0.im)};
    };
    // Z chain: X += i z0i T0 + i z1i T1 (+ z2r T2), Y += z0r T0 + z1r T1 (+ i z2i T2), T2 with free
    // helicities only; the imaginary parts carry f
    T z0r = T(0), z0i = T(0), z1r = T(0), z1i = T(0), z2r = T(0), z2i = T(0);
    auto z_add = [&](T f, const Cx<T>& T0, const Cx<T>& T1, const Cx<T>& T2, Cx<T>& X_, Cx<T>& Y_) {
      const T a0 = f * z0i, a1 = f * z1i;
      X_.re = fma_(-a0, T0.im, fma_(-a1, T1.im, X_.re));
      X_.im = fma_(a0, T0.re, fma_(a1, T1.re, X_.im));
      Y_.re = fma_(z0r, T0.re, fma_(z1r, T1.re, Y_.re));
      Y_.im = fma_(z0r, T0.im, fma_(z1r, T1.im, Y_.im));
      if constexpr (ZF) {
        const T a2 = f * z2i;
        X_.re = fma_(z2r, T2.re, X_.re);
        X_.im = fma_(z2r, T2.im, X_.im);
        Y_.re = fma_(-a2, T2.im, Y_.re);
        Y_.im = fma_(a2, T2.re, Y_.im);
      }
    };
    // flavour of this reading: the tag of a data event, + / - for the two normalisation records
    T f1 = T(1);
    if constexpr (CC) f1 = set == 0 ? ldoff(a.tag + e0, ob) : (set == 1 ? T(1) : T(-1));
    Cx<T> X, Y;
    kstar_at(f1, X, Y);

    // ---- Z chain (Eq. 10-12)
    // (AZ holds the bare Breit-Wigner; the Z barrier factor n_Z is in the angular columns)
    Cx<T> AZ[NZ > 0 ? NZ : 1];
    T gzv = T(0);
    Cx<T> T0k{T(0), T(0)}, T1k{T(0), T(0)}, T2k{T(0), T(0)};   // Z coupling sums, kept for a second reading
    if constexpr (NZ > 0) {
      if (a.cnt[5] > 0) {
        if constexpr (!PRE && !TOYS) {
#pragma unroll
          for (int k = 3; k < NG; ++k) grp[k] = ldoff(gb + k * ld, i * (uint32_t)sizeof(V4));
        }
        const T mz2 = grp[2].y;
        gzv = grp[2].w;
        // The xi = -1 factors are (-Re, Im) of the xi = +1 ones (columns 12-15), so Im enters X and
        // Re enters Y
        const V4 g3 = grp[3];
        z0r = g3.x;
        z0i = g3.y;
        if constexpr (ZF) {
          // F++ (14-15) and F+- (16-17): the sum and difference couplings take the real and
          // imaginary parts of F++ +- F+-
          const V4 g4 = grp[4];
          z1r = g3.z - g4.x;
          z1i = g3.w + g4.y;
          z2r = g3.z + g4.x;
          z2i = g3.w - g4.y;
        } else {
          z1r = g3.z;
          z1i = g3.w;
        }
        Cx<T> T0{T(0), T(0)}, T1{T(0), T(0)}, T2{T(0), T(0)};
#pragma unroll
        for (int z = 0; z < NZ; ++z) {
          if (z < a.cnt[5]) {
            const C8 rc = constants(NK + z);
            const T dre = pole_gap(rc[0], ka.M2lo[NK + z], mz2);
            const T dim = rc[1] * gzv;
            const T inv = rcp_(fma_(dre, dre, dim * dim));
            AZ[z] = Cx<T>{dre * inv, dim * inv};
            cmac(T0, rc[2], rc[3], AZ[z].re, AZ[z].im);
            cmac(T1, rc[4], rc[5], AZ[z].re, AZ[z].im);
            if constexpr (ZF) cmac(T2, rc[6], rc[7], AZ[z].re, AZ[z].im);
          }
        }
        if constexpr (ZF) {   // sum and difference of lambda' = +1 and -1
          const Cx<T> p = T1, m = T2;
          T1 = Cx<T>{p.re + m.re, p.im + m.im};
          T2 = Cx<T>{p.re - m.re, p.im - m.im};
        }
        z_add(f1, T0, T1, T2, X, Y);
        if constexpr (CC) {
          T0k = T0;
          T1k = T1;
          if constexpr (ZF) T2k = T2;
        }
      }
    }

    const T S = fma_(X.re, X.re, X.im * X.im) + fma_(Y.re, Y.re, Y.im * Y.im);

    if constexpr (MODE == MODE_DENSITY) {
      a.s_out[set][e] = (double)S;
      continue;
    }
    if constexpr (TOYS) {
      const ToyArgs& ty = a.toys;
      const double s = ty.acc_on ? (double)S * eps_true : (double)S;
      if (s > ty.smax) atomicAdd(&ty.stat[kToyOver + (prop >> kRoundBits)], 1u);
      if (spare * ty.smax < s) atomicOr(&ty.mask[prop >> 6], 1ull << (prop & 63));
      continue;
    }

    // ---- likelihood terms
    T w;
    T w2 = T(0);                  // mistag: adjoint weight of the other-flavour reading
    Cx<T> X2{T(0), T(0)}, Y2{T(0), T(0)};
    if (set == 0) {
      T arg = S;   // the quantity whose logarithm is summed
      if constexpr (CC) {
        T S2 = T(0);
        if (a.mistag > T(0)) {
          // t = (1 - w) S(q phi) + w S(-q phi)
          kstar_at(-f1, X2, Y2);
          if constexpr (NZ > 0) {
            if (a.cnt[5] > 0) z_add(-f1, T0k, T1k, T2k, X2, Y2);
          }
          S2 = fma_(X2.re, X2.re, X2.im * X2.im) + fma_(Y2.re, Y2.re, Y2.im * Y2.im);
          arg = fma_(a.keep, S, a.mistag * S2);
        }
        // Eq. 14 with tags: t = p eps [(1 - w) S(q phi) + w S(-q phi)] + k_q b, k_q of the
        // event's flavour; d ln t / dS = p eps (1 - w) / t
        T pe = T(1);
        if (mix) {
          pe = a.purity * (a.eps_data ? ldoff(a.eps_data + e0, ob) : T(1));
          arg = fma_(pe, arg, (f1 > T(0) ? kb : kb2) * ldoff(a.bkg_data + e0, ob));
        }
        if (!(arg > pos_floor<T>()) || !(arg < T(INFINITY))) nbad += 1.f;
        const T r = pe * rcp_(arg);
        if (a.mistag > T(0)) {
          w = a.keep * r;
          w2 = a.mistag * r;
        } else {
          w = r;
        }
        if (mix) {
          const A_t c = (A_t)fma_(w, S, w2 * S2);
          if (f1 > T(0)) ws += c;
          else ws2 += c;
        }
      } else if (mix) {
        // Eq. 14: t = p eps S + k b; d ln t / dS = p eps / t
        const T pe = a.purity * (a.eps_data ? ldoff(a.eps_data + e0, ob) : T(1));
        arg = fma_(pe, S, kb * ldoff(a.bkg_data + e0, ob));
        if (!(arg > pos_floor<T>()) || !(arg < T(INFINITY))) nbad += 1.f;
        w = pe * rcp_(arg);
        ws += (A_t)(w * S);
      } else {
        if (!(S > pos_floor<T>()) || !(S < T(INFINITY))) nbad += 1.f;
        w = rcp_(S);
      }
      // ln of the product of the terms, kept as the product of their mantissas (each in [1/2, 1): at
      // most 1024 passes, so it stays representable) and the sum of their exponents; one logarithm per
      // thread after the loop.  Its roundings (2^-53 per event) are below those of a logarithm per event:
      // the rms error of 64 terms is 3.7e-16 whatever their scale, that of a compensated sum of
      // correctly rounded logarithms 6e-16 for terms near 1 and 4e-15 for terms near 1e3 or 1e-4.
      if constexpr (std::is_same_v<T, float>) {
        ms *= (double)__builtin_amdgcn_frexp_mantf(arg);
        mexp += __builtin_amdgcn_frexp_expf(arg);
      } else {
        ms *= __builtin_amdgcn_frexp_mant(arg);
        mexp += __builtin_amdgcn_frexp_exp(arg);
      }
    } else {
      const T eps = a.eps ? ldoff(a.eps + e0, ob) : T(1);
      const double x = (double)(eps * S);
      const double y = x - mc;
      const double t = ms + y;
      mc = (t - ms) - y;
      ms = t;
      w = eps;
    }

    if constexpr (GRAD) {
      // adjoint of S = |X|^2 + |Y|^2: bX = w conj(X), bY = w conj(Y); the weights of U_+-, e^{+-i phi}
      // (cos th_J bY +- bX), and of U_0, sin th_J bY, summed over the readings of the event.  (By helicity: as
      // sums over the weights of U_+ +- U_-, the gradient of a small helicity beside a large one would be the
      // difference of two sums of the large one's size.)
      Cx<T> W0, Wp, Wm;
      Cx<T> bX, bY, bX2{T(0), T(0)}, bY2{T(0), T(0)};
      auto adj_w = [&](auto first, T wt, T f, const Cx<T>& X_, const Cx<T>& Y_, Cx<T>& bX_, Cx<T>& bY_) {
        constexpr bool F = decltype(first)::value;
        bX_ = Cx<T>{wt * X_.re, -wt * X_.im};
        bY_ = Cx<T>{wt * Y_.re, -wt * Y_.im};
        const T sp = f * sph;
        const Cx<T> s{fma_(cJ, bY_.re, bX_.re), fma_(cJ, bY_.im, bX_.im)};
        const Cx<T> d{fma_(cJ, bY_.re, -bX_.re), fma_(cJ, bY_.im, -bX_.im)};
        if constexpr (F) {
          Wp = Cx<T>{fma_(cph, s.re, -sp * s.im), fma_(cph, s.im, sp * s.re)};
          Wm = Cx<T>{fma_(cph, d.re, sp * d.im), fma_(cph, d.im, -sp * d.re)};
          W0 = Cx<T>{sJ * bY_.re, sJ * bY_.im};
        } else {
          Wp.re = fma_(cph, s.re, fma_(-sp, s.im, Wp.re));
          Wp.im = fma_(cph, s.im, fma_(sp, s.re, Wp.im));
          Wm.re = fma_(cph, d.re, fma_(sp, d.im, Wm.re));
          Wm.im = fma_(cph, d.im, fma_(-sp, d.re, Wm.im));
          W0.re = fma_(sJ, bY_.re, W0.re);
          W0.im = fma_(sJ, bY_.im, W0.im);
        }
      };
      adj_w(std::true_type{}, w, f1, X, Y, bX, bY);
      const bool two = CC && set == 0 && a.mistag > T(0);
      if constexpr (CC) {
        if (two) adj_w(std::false_type{}, w2, -f1, X2, Y2, bX2, bY2);
      }
      // weights of the Z coupling sums over the readings: WZ0 = i z0i bX + z0r bY, WZ1 alike, and
      // with free helicities WZ2 = z2r bX + i z2i bY
      Cx<T> WZ0{T(0), T(0)}, WZ1{T(0), T(0)}, WZ2{T(0), T(0)};
      auto wz = [&](auto first, T f, const Cx<T>& bX_, const Cx<T>& bY_) {
        constexpr bool F = decltype(first)::value;
        const T a0 = f * z0i, a1 = f * z1i;
        Cx<T> y0{z0r * bY_.re, z0r * bY_.im}, y1{z1r * bY_.re, z1r * bY_.im};
        if constexpr (!F) {
          y0.re += WZ0.re; y0.im += WZ0.im;
          y1.re += WZ1.re; y1.im += WZ1.im;
        }
        WZ0 = Cx<T>{fma_(-a0, bX_.im, y0.re), fma_(a0, bX_.re, y0.im)};
        WZ1 = Cx<T>{fma_(-a1, bX_.im, y1.re), fma_(a1, bX_.re, y1.im)};
        if constexpr (ZF) {
          const T a2 = f * z2i;
          WZ2.re = fma_(z2r, bX_.re, fma_(-a2, bY_.im, WZ2.re));
          WZ2.im = fma_(z2r, bX_.im, fma_(a2, bY_.re, WZ2.im));
        }
      };
      auto z_weights = [&]() {
        wz(std::true_type{}, f1, bX, bY);
        if constexpr (CC) {
          if (two) wz(std::false_type{}, -f1, bX2, bY2);
        }
      };
      // V_{J lambda}: the angular functions times the weights
      auto V_of = [&](auto Jc, Cx<T>& Vm, Cx<T>& V0, Cx<T>& Vp) {
        constexpr int J = decltype(Jc)::value;
        V0 = Cx<T>{dd0[J] * W0.re, dd0[J] * W0.im};
        if constexpr (J > 0) {
          Vm = Cx<T>{dd1[J] * Wm.re, dd1[J] * Wm.im};
          Vp = Cx<T>{dd1[J] * Wp.re, dd1[J] * Wp.im};
        }
      };
      if constexpr (NZ > 0) {
        if (a.cnt[5] > 0) {
          z_weights();
          if constexpr (ZF) {   // lambda' = +1 and -1 of the sum and difference
            const Cx<T> s = WZ1, d = WZ2;
            WZ1 = Cx<T>{s.re + d.re, s.im + d.im};
            WZ2 = Cx<T>{s.re - d.re, s.im - d.im};
          }
        }
      }
      if constexpr (PRE) {
        if (!ZF || left != 0) fetch(i + 256 < n_blk ? i + 256 : i);
      }
      auto grad_spin = [&](auto Jc) {
        constexpr int J = decltype(Jc)::value;
        if constexpr (Sh::N[J] > 0) {
          constexpr int sb = slot_base<Sh>(J);
          constexpr int ab = acc_base<Sh>(J) - 3;
          Cx<T> Vm, V0, Vp;
          V_of(Jc, Vm, V0, Vp);
#pragma unroll
          for (int j = 0; j < Sh::N[J]; ++j) {
            const Cx<T> A = Amp[sb + j];
            if constexpr (J == 0) {
              // accumulators += A V as two fused multiply-adds per component
              cacc(gk[ab + 2 * j], gk[ab + 2 * j + 1], A, V0);
            } else if constexpr (LDSACC && J >= 1 && J <= 3) {
              // ab + 6 j lies in [LO, HI): this thread's own LDS slots
              lds_ptr<A_t> g = accb + 256 * (ab + 6 * j - LO);
              if constexpr (std::is_same_v<A_t, double>) {
                auto add = [&](int l, const Cx<T>& V) {
                  lds_add(g + 512 * l, fma_(A.re, V.re, -A.im * V.im));
                  lds_add(g + 512 * l + 256, fma_(A.re, V.im, A.im * V.re));
                };
                add(0, Vm);
                add(1, V0);
                add(2, Vp);
              } else {
                A_t v[6];
#pragma unroll
                for (int q = 0; q < 6; ++q) v[q] = g[256 * q];
                cacc(v[0], v[1], A, Vm);
                cacc(v[2], v[3], A, V0);
                cacc(v[4], v[5], A, Vp);
#pragma unroll
                for (int q = 0; q < 6; ++q) g[256 * q] = v[q];
              }
            } else {
              A_t* g = gk + ab + 6 * j;
              cacc(g[0], g[1], A, Vm);
              cacc(g[2], g[3], A, V0);
              cacc(g[4], g[5], A, Vp);
            }
          }
        }
      };
      grad_spin(std::integral_constant<int, 0>{});
      grad_spin(std::integral_constant<int, 1>{});
      grad_spin(std::integral_constant<int, 2>{});
      grad_spin(std::integral_constant<int, 3>{});
      grad_spin(std::integral_constant<int, 4>{});

      if constexpr (NZ > 0) {
        if (a.cnt[5] > 0) {
#pragma unroll
          for (int z = 0; z < NZ; ++z) {
            if (z < a.cnt[5]) {
              const Cx<T> A = AZ[z];
              A_t* g = gz + 4 * z;
              cacc(g[0], g[1], A, WZ0);
              cacc(g[2], g[3], A, WZ1);
              if constexpr (ZF) cacc(g[4], g[5], A, WZ2);   // the second Z's lambda' = 0 slots
            }
          }
        }
      }

      // Lineshape sums of the floating slots: the slot's Breit-Wigner, adjoint weight and width
      // factor are picked by uniform branches (the slot numbers are re-read each event, so the
      // comparisons are not hoisted into scalar registers the loop needs), then one piece of code
      // sums them.
      auto flt_slot = [&](int slot, T& sR, T& sI) {
        const auto& h = ka.cs[slot].h;
        Cx<T> B{T(0), T(0)}, Q{T(0), T(0)};
        T g = T(0);
        auto pick = [&](auto Jc) {
          constexpr int J = decltype(Jc)::value;
          constexpr int sb = slot_base<Sh>(J);
#pragma unroll
          for (int j = 0; j < Sh::N[J]; ++j) {
            if (slot != sb + j) continue;
            Cx<T> Vm, V0, Vp;
            V_of(Jc, Vm, V0, Vp);
            if constexpr (J > 0) cmac(Q, h[0][0], h[0][1], Vm.re, Vm.im);
            cmac(Q, h[1][0], h[1][1], V0.re, V0.im);
            if constexpr (J > 0) cmac(Q, h[2][0], h[2][1], Vp.re, Vp.im);
            B = Amp[sb + j];
            g = gJv[J];
          }
        };
        pick(std::integral_constant<int, 0>{});
        pick(std::integral_constant<int, 1>{});
        pick(std::integral_constant<int, 2>{});
        pick(std::integral_constant<int, 3>{});
        pick(std::integral_constant<int, 4>{});
        if constexpr (NZ > 0) {
#pragma unroll
          for (int z = 0; z < NZ; ++z) {
            if (slot != NK + z) continue;
            cmac(Q, h[0][0], h[0][1], WZ0.re, WZ0.im);
            cmac(Q, h[1][0], h[1][1], WZ1.re, WZ1.im);
            if constexpr (ZF) cmac(Q, h[2][0], h[2][1], WZ2.re, WZ2.im);
            B = AZ[z];
            g = gzv;
          }
        }
        flt_sums(B, Q, g, sR, sI);
      };
      const int fs0 = ka.flt[0], fs1 = ka.flt[1];   // (the first is filled first)
      if (fs0 >= 0) {
        flt_slot(fs0, gM0, gG0);
        if (fs1 >= 0) flt_slot(fs1, gM1, gG1);
      }
    }
  }

  if constexpr (MODE == MODE_DENSITY || TOYS) return;

  if (set == 0) {
    // ln(ms 2^mexp) as the pair ms - mc: mexp ln2 in two parts, the first exact (29 bits times
    // at most 24) so that the pair carries the full product.  FP32: the logarithm of the mantissa is
    // the hardware's (an error of 1e-7 per thread, where each event's was), corrected for what its
    // argument leaves out; the double precision one cost 1.5 us of the 35 of 3e6 events.
    constexpr double L2H = 0x1.62e42ff000000p-1, L2L = -0x1.718432a1b0e26p-35;
    mexp += __builtin_amdgcn_frexp_exp(ms);
    const double mprod = __builtin_amdgcn_frexp_mant(ms);
    double ln;
    if constexpr (std::is_same_v<T, float>) {
      const float hi = (float)mprod;
      ln = (double)(__builtin_amdgcn_logf(hi) * 0.693147180559945309f + (float)(mprod - (double)hi) * rcp_(hi));
    } else {
      ln = log(mprod);
    }
    ms = (double)mexp * L2H;
    mc = -((double)mexp * L2L + ln);
  }
  // ---- block reduction: wave transpose-butterfly, then the 4 waves in order
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __shared__ double red[4][NACC];
  if constexpr (GRAD) {
    // accumulator i >= 2 of this lane at its accumulation type (compile-time index after
    // unrolling); 0 and 1 are the FP64 likelihood sums
    auto accf = [&](int i) -> A_t {
      if (i == 2) return (A_t)nbad;
      if (LDSACC && i >= 3 + LO && i < 3 + HI) return accl[i - 3 - LO][threadIdx.x];
      if (i < 3 + Sh::NKACC) return gk[i - 3];
      if (i < 3 + Sh::NKACC + 4 * Sh::NZ) return gz[i - 3 - Sh::NKACC];
      const int f = i - 3 - Sh::NKACC - 4 * Sh::NZ;
      if (f == 0) return gM0;
      if (f == 1) return gG0;
      if (f == 2) return gM1;
      if (f == 3) return gG1;
      if (f == 4) return ws;
      return A_t(0);
    };
    // Transpose butterfly: after the step of width h, lane l keeps h values, each summed
    // with its partner lane's; after the last step lane l holds the wave sum of value l.
    // The steps of width 32 and 16 use the lane-swap instructions (swap_halves), the rest DPP
    // row permutations (dpp_partner).  Slots 0 and 1 carry the FP64 likelihood sums and every value merged into
    // them (as double); the other slots move the accumulators at their own type (FP32 sums of
    // the wave's FP32 thread accumulators in the FP32 kernel).
    if constexpr (CC) {
      // tagged mixture: slot 1 carries the - flavour's sum of w S (the Kahan correction is
      // folded into slot 0 first)
      if (mix) {
        ms = ms - mc;
        mc = -(double)ws2;
      }
    }
    double d[2];
    A_t v[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      if (i < 2) {
        double lo = (i == 0) ? ms : -mc;   // Kahan: the running sum exceeds the exact one by mc
        double hi = (double)accf(i + 32);
        swap_halves<32>(lo, hi);
        d[i] = lo + hi;
      } else {
        A_t lo = accf(i), hi = accf(i + 32);
        swap_halves<32>(lo, hi);
        v[i] = lo + hi;
      }
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i < 2) {
        double lo = d[i], hi = (double)v[i + 16];
        swap_halves<16>(lo, hi);
        d[i] = lo + hi;
      } else {
        A_t lo = v[i], hi = v[i + 16];
        swap_halves<16>(lo, hi);
        v[i] = lo + hi;
      }
    }
    auto narrow = [&](auto Hc) {
      constexpr int half = decltype(Hc)::value;
      const bool up = lane & half;
#pragma unroll
      for (int i = 0; i < half; ++i) {
        if (i < 2) {
          const double hv = (i + half < 2) ? d[i + half] : (double)v[i + half];
          const double keep = up ? hv : d[i];
          const double send = up ? d[i] : hv;
          d[i] = keep + dpp_partner<half>(send);
        } else {
          // (the empty asm keeps the two slots as values, so that the selects below stay
          // selects instead of becoming a lane-dependent index into the slot array)
          A_t a0 = v[i], a1 = v[i + half];
          asm("" : "+v"(a0), "+v"(a1));
          const A_t keep = up ? a1 : a0;
          const A_t send = up ? a0 : a1;
          v[i] = keep + dpp_partner<half>(send);
        }
      }
    };
    narrow(std::integral_constant<int, 8>{});
    narrow(std::integral_constant<int, 4>{});
    narrow(std::integral_constant<int, 2>{});
    narrow(std::integral_constant<int, 1>{});
    red[wave][lane] = d[0];
  } else {
    double v0 = ms, v1 = -mc, v2 = (double)nbad;
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
      v0 += __shfl_xor(v0, s, 64);
      v1 += __shfl_xor(v1, s, 64);
      v2 += __shfl_xor(v2, s, 64);
    }
    if (lane < NACC) red[wave][lane] = (lane == 0) ? v0 : (lane == 1 ? v1 : (lane == 2 ? v2 : 0.0));
  }
  __syncthreads();
  if (wave == 0) {
    const double t = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    // value-major layout: value v of block b at partial[v * gridDim.x + b]
    if (GRAD || lane < 3) a.partial[(int64_t)lane * a.pstride + a.poff + blockIdx.x] = t;
  }
}

// Fixed-order compensated sum of the block partials.  Block (set, v) sums value v over the
// blocks of one set: each thread runs a Neumaier sum over a strided subset, the pairs are merged
// in a butterfly within each wavefront and the four wavefronts in order.  Output goes to
// out[set*NACC + v] (mapped pinned host memory).  The partial rows hold the data blocks, then n_mc_sets runs of
// nb_mc normalisation blocks (records 1, 2).

__global__ __launch_bounds__(256) void reduce_final(const double* __restrict__ partial, int nb_data, int nb_mc,
                                                    int n_mc_sets, int nv, double* __restrict__ out, int first_set) {
  const int set = first_set + (int)blockIdx.x / nv, v = blockIdx.x % nv;
  const int64_t nbt = nb_data + (int64_t)n_mc_sets * nb_mc;   // row stride of the partials
  const int b0 = set == 0 ? 0 : nb_data + (set - 1) * nb_mc;
  const int nb = set ? nb_mc : nb_data;
  const double* __restrict__ p = partial + (int64_t)v * nbt + b0;
  double s = 0.0, c = 0.0;
  // blocks tid, tid + 256, ... in that order; four loads are issued before their sums, so a
  // thread waits for memory once per four values rather than once per value
  for (int b0 = threadIdx.x; b0 < nb; b0 += 4 * 256) {
    double x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = b0 + k * 256 < nb ? p[b0 + k * 256] : 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (b0 + k * 256 < nb) neumaier(s, c, x[k]);
  }
  // butterfly of exact two-sum merges in each wavefront (every lane ends with the wavefront's
  // total), then the four wavefronts in order
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) two_sum_merge(s, c, __shfl_xor(s, off, 64), __shfl_xor(c, off, 64));
  __shared__ double S[4], Cc[4];
  if ((threadIdx.x & 63) == 0) {
    S[threadIdx.x >> 6] = s;
    Cc[threadIdx.x >> 6] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = S[0], tc = Cc[0];
    for (int w = 1; w < 4; ++w) two_sum_merge(t, tc, S[w], Cc[w]);
    out[set * NACC + v] = t + tc;
  }
}

// ------------------------------------------------------------------ efficiency histogram
__global__ __launch_bounds__(256) void hist_lookup_kernel(HistArgs a) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.n) return;
  int64_t idx = 0;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const double x = a.obs[d][e];
    int b = (int)floor((x - a.lo[d]) / (a.hi[d] - a.lo[d]) * a.nb[d]);
    b = b < 0 ? 0 : (b >= a.nb[d] ? a.nb[d] - 1 : b);
    idx = idx * a.nb[d] + b;
  }
  a.out_f64[e] = (double)a.table[idx];
}

// ------------------------------------------------------------------ 2D x 2D templates
__global__ __launch_bounds__(256) void template_kernel(TplArgs a) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.n) return;
  int b[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const double x = a.obs[d][e];
    int k = (int)floor((x - a.lo[d]) / (a.hi[d] - a.lo[d]) * a.nb[d]);
    b[d] = k < 0 ? 0 : (k >= a.nb[d] ? a.nb[d] - 1 : k);
  }
  a.out[e] = (double)a.t1[b[0] * a.nb[1] + b[1]] * (double)a.t2[b[2] * a.nb[3] + b[3]];
}

// ------------------------------------------------------------------ generators
__global__ __launch_bounds__(256) void phsp_kernel(GenArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const uint64_t e = (uint64_t)(a.e0 + i);
  double m, ck, cj, phi, spare;
  uint32_t t = 0;
  while (t < kTrials && !phsp_trial(a.kin, a.seed, a.wmax, e, t, m)) ++t;
  if (t == kTrials) { a.flag[i] = 0; a.out[0][i] = NAN; return; }
  phsp_angles(e, a.seed, ck, cj, phi, spare);
  a.out[0][i] = m;
  a.out[1][i] = ck;
  a.out[2][i] = cj;
  a.out[3][i] = phi;
  a.flag[i] = 1;
}

// Accept-reject toys.  Of the proposals flat in phase space about one in 200 is kept, so the density
// is evaluated only where it can matter:
//   bound_kernel    once per call: an upper bound of eps S in each of kBins mass bins
//   propose_kernel  the masses of the proposals, and the list of those whose accept-reject number
//                   lies below the bound of their bin (the others are rejected whatever their angles)
//   amp_kernel      (MODE_TOYS) angles, density, acceptance and the accept bits of the listed ones
//   count_kernel, collect_kernel   the accepted ones in the order of the proposals
// Every step is a pure function of the proposal's number, so the sample does not depend on how the
// proposals are split.  All columns, flags and densities of every proposal went through memory
// before (phase space, invariants, density, acceptance, two scans and a copy: 205 us per 2^20
// proposals, now 18 us).

// Upper bound of eps S for m_Kpi in bin b.  With the sums of kernel amplitudes P, M, U_0 of the
// angular part of amp_kernel, the K* chain alone gives S <= |P|^2 + |M|^2 + |U_0|^2 (the rotations
// by phi and theta_J are unitary), and the Z chain adds at most zmax to sqrt(S).  Each sum is at most
// the sum of its terms' magnitudes, and over an interval of the mass
//   |1/D|  <= 1 / sqrt(dist(M^2, [s1, s2])^2 + (P g(s1))^2)        (g grows with the mass)
//   n_J    <= p_B(m1)^L_B (q/m)(m2)^J / sqrt(B_J(q1) B_LB(p_B2))   (p_B falls, q and q/m grow)
//   |ang0| <= ang0(1),   |sin ang1| <= 2 ang1(1) / (J + 1)         (Legendre; Bernstein's inequality)
// The Z angular factors are at most n_Z / sqrt2 in size.  The intervals overlap by 1e-9 of the range
// and the bound is raised by 1e-6, which covers every rounding.
template <class Sh> __global__ __launch_bounds__(kBins) void bound_kernel(const ToyAmpArgs<Sh> a) {
  const ToyArgs& ty = a.toys;
  const Kin& k = ty.kin;
  auto span = [&](double lo, double hi, double& x1, double& x2) {
    x1 = fmax(lo, lo + (hi - lo) * ((double)threadIdx.x / kBins - 1e-9));
    x2 = fmin(hi, lo + (hi - lo) * ((threadIdx.x + 1.0) / kBins + 1e-9));
  };
  // breakup momentum of mass M into m1 and m2
  auto mom = [](double M, double m1, double m2) {
    return sqrt(fmax(0.0, (M * M - (m1 + m2) * (m1 + m2)) * (M * M - (m1 - m2) * (m1 - m2)))) / (2.0 * M);
  };
  auto prop = [](double M2, double P, double s1, double s2, double g1) {
    const double d = fmax(0.0, fmax(M2 - s2, s1 - M2)), w = P * g1;
    return 1.0 / sqrt(d * d + w * w);
  };
  auto mag = [](const double* h) { return sqrt(h[0] * h[0] + h[1] * h[1]); };
  auto mag2 = [](const double* h, const double* g, double s) {   // |h + s g|
    const double x = h[0] + s * g[0], y = h[1] + s * g[1];
    return sqrt(x * x + y * y);
  };
  // ---- Z chain: the bound over bin threadIdx.x of m_Jpsi pi, then the largest of the block
  __shared__ double zred[kBins / 64];
  double z = 0.0;
  if (Sh::NZ > 0 && a.cnt[5] > 0) {
    double m1, m2;
    span(k.mJ + k.mPi, k.mB - k.mK, m1, m2);
    const double g1 = mom(m1, k.mJ, k.mPi) / m1, pz = mom(k.mB, m1, k.mK);
    const double nZ = (pz / k.mB) / sqrt(1.0 + k.rB * pz * k.rB * pz);
    for (int i = 0; i < a.cnt[5]; ++i) {
      const AC<double>& rc = a.cs[Sh::NK + i];
      const double h = mag(rc.h[0]) + (a.zfree ? mag2(rc.h[1], rc.h[2], 1.0) + mag2(rc.h[1], rc.h[2], -1.0) : mag(rc.h[1]));
      if (h > 0.0) z += h * prop(rc.M2, rc.P, m1 * m1, m2 * m2, g1) * nZ * 0.70710678118654752440;
    }
  }
  for (int off = 32; off >= 1; off >>= 1) {
    const double o = __shfl_xor(z, off, 64);
    z = o > z || o != o ? o : z;   // (a NaN stays: the bound then rejects nothing)
  }
  if ((threadIdx.x & 63) == 0) zred[threadIdx.x >> 6] = z;
  __syncthreads();
  for (int w = 0; w < kBins / 64; ++w) z = zred[w] > z || zred[w] != zred[w] ? zred[w] : z;
  // ---- K* chain
  double m1, m2;
  span(k.mK + k.mPi, k.mB - k.mJ, m1, m2);
  const double q1 = mom(m1, k.mK, k.mPi), q2 = mom(m2, k.mK, k.mPi), pB1 = mom(k.mB, m1, k.mJ), pB2 = mom(k.mB, m2, k.mJ);
  double p = 0.0, mm = 0.0, u0 = 0.0;
  auto spin = [&](auto Jc) {
    constexpr int J = decltype(Jc)::value, LB = LBof<J>::v;
    const double BR = bpoly<J>(a.rR2 * q1 * q1);
    const double nJ = ipow<double, LB>(pB1) * ipow<double, J>(q2 / m2) / sqrt(BR * bpoly<LB>(a.rB2 * pB2 * pB2));
    const double gJ = q1 / m1 * ipow<double, J>(q1 * q1) / BR;
    const double e0 = nJ * ang0<J>(1.0), e1 = J > 0 ? nJ * ang1<J>(1.0) * (2.0 / (J + 1)) : 0.0;
    for (int j = 0; j < Sh::N[J]; ++j) {
      const int sl = slot_base<Sh>(J) + j;
      const AC<double>& rc = a.cs[sl];
      const double h1 = mag(rc.h[1]);   // the couplings of U_0, and of U_+ - U_- and U_+ + U_-
      const double h0 = J > 0 ? mag2(rc.h[2], rc.h[0], -1.0) : 0.0, h2 = J > 0 ? mag2(rc.h[2], rc.h[0], 1.0) : 0.0;
      if (h0 == 0.0 && h1 == 0.0 && h2 == 0.0) continue;
      double A = prop(rc.M2, rc.P, m1 * m1, m2 * m2, gJ);
      if (J == 0 && (a.lass & (1 << sl))) {
        // m / |u + i q| + P |B|, u = 1/a + b q^2/2
        const double ua = a.lai[sl] + a.lhb[sl] * q1 * q1, ub = a.lai[sl] + a.lhb[sl] * q2 * q2;
        const double u = ua * ub > 0.0 ? fmin(fabs(ua), fabs(ub)) : 0.0;
        A = m2 / sqrt(u * u + q1 * q1) + fabs(rc.P) * A;
      }
      p += e1 * h0 * A;
      mm += e1 * h2 * A;
      u0 += e0 * h1 * A;
    }
  };
  spin(std::integral_constant<int, 0>{});
  spin(std::integral_constant<int, 1>{});
  spin(std::integral_constant<int, 2>{});
  spin(std::integral_constant<int, 3>{});
  spin(std::integral_constant<int, 4>{});
  const double r = sqrt(p * p + mm * mm + u0 * u0) + z;
  ty.bound[threadIdx.x] = (ty.acc_on ? 0.9 : 1.0) * (r * r * (1.0 + 1e-6));
}

// Masses of the proposals and the list of those to evaluate.  A wavefront takes per_wave proposals
// (a multiple of 64, at most kPerWave); a lane whose proposal has found its mass takes the next one,
// so a wavefront runs for the mean number of trials (about 2) and not for the longest of 64 (about
// 7).  Bound by the integer multiplications of Philox, 11 us per 2^20 proposals in a chunk of
// four of these (44 us for the masses and angles with one proposal per lane).
constexpr int kPerWave = 1024;
// Events accepted before this chunk; true if the sample is already complete (the chunk has nothing to do).
__device__ __forceinline__ bool toys_done(const ToyArgs& a, int64_t& before) {
  before = a.kept + *reinterpret_cast<const int64_t*>(a.stat - kToyStat + kToySum);
  return before >= a.limit;
}
__global__ __launch_bounds__(256) void propose_kernel(ToyArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t before;
  if (toys_done(a, before)) return;
  __shared__ double mass[4][kPerWave];
  __shared__ unsigned long long sel[4][kPerWave / 64];
  const int W = a.per_wave;
  const uint32_t base = ((uint32_t)blockIdx.x * 4 + wave) * (uint32_t)W;   // (the grid covers the chunk)
  const uint64_t first = (uint64_t)a.e0 + base;
  if (lane < W / 64) a.mask[base / 64 + lane] = 0ull;
  int idx = lane, next = 64;
  uint32_t t = 0;
  while (__ballot(idx < W)) {
    double m = 0.0;
    bool done = false;
    if (idx < W) {
      done = phsp_trial(a.kin, a.seed, a.wmax, first + idx, t, m);
      if (!done && ++t == kTrials) {
        m = NAN;   // failed: never listed
        done = true;
      }
    }
    const unsigned long long b = __ballot(done);
    if (done) {
      mass[wave][idx] = m;
      idx = next + __popcll(b & ((1ull << lane) - 1));
      t = 0;
    }
    next += __popcll(b);
  }
  __syncthreads();
  const double lo = a.kin.mK + a.kin.mPi, hi = a.kin.mB - a.kin.mJ;
  uint32_t cnt = 0;
  for (int g = 0; g < W / 64; ++g) {
    const int j = 64 * g + lane;
    const double m = mass[wave][j];
    double ua, spare;
    u2(first + j, 0u, 2u, a.seed, ua, spare);
    int bin = (int)((m - lo) / (hi - lo) * kBins);
    bin = bin < 0 ? 0 : (bin >= kBins ? kBins - 1 : bin);
    const bool s = m == m && !(spare * a.smax >= a.bound[bin]);
    const unsigned long long b = __ballot(s);
    if (lane == 0) sel[wave][g] = b;
    cnt += __popcll(b);
  }
  // room in the block's list: one addition per block, to one of kToyLists lengths (additions to one
  // address pass one after the other, 13 ns each: with one per wavefront to a single list they took
  // all of the kernel's time)
  __shared__ uint32_t wcnt[4], room;
  if (lane == 0) wcnt[wave] = cnt;
  __syncthreads();
  const uint32_t list = blockIdx.x % kToyLists;
  if (threadIdx.x == 0) room = atomicAdd(&a.stat[kToyListed + 16 * list], (wcnt[0] + wcnt[1]) + (wcnt[2] + wcnt[3]));
  __syncthreads();
  uint32_t at = list * (((uint32_t)a.rounds << kRoundBits) / kToyLists) + room;
  for (int v = 0; v < wave; ++v) at += wcnt[v];
  for (int g = 0; g < W / 64; ++g) {
    const unsigned long long b = sel[wave][g];
    if (b >> lane & 1) {
      const uint32_t j = 64 * g + lane;
      a.m[base + j] = mass[wave][j];
      a.list[at + __popcll(b & ((1ull << lane) - 1))] = base + j;
    }
    at += __popcll(b);
  }
}

// Accepted proposals of each group.  (Counted as they are found, the 5000 atomic additions per round
// cost 7 us of the density kernel's 11; this takes one.)
__global__ __launch_bounds__(256) void count_kernel(ToyArgs a) {
  int64_t before;
  if (toys_done(a, before)) return;
  uint32_t n = __popcll(a.mask[(int64_t)blockIdx.x * 256 + threadIdx.x]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off, 64);
  __shared__ uint32_t r[4];
  if ((threadIdx.x & 63) == 0) r[threadIdx.x >> 6] = n;
  __syncthreads();
  if (threadIdx.x == 0) a.stat[kToyCounts + blockIdx.x] = (r[0] + r[1]) + (r[2] + r[3]);
}

// The accepted proposals of group blockIdx.x (one word of accept bits per thread), written behind those
// of all earlier ones while there is room; the one that completes the sample leaves its number, and
// the last group the sum so far.
__global__ __launch_bounds__(256) void collect_kernel(ToyArgs a) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int64_t before;
  const bool full = toys_done(a, before);
  const unsigned* cnt = a.stat + kToyCounts;
  static_assert((kMaxRounds << (kRoundBits - kGroupBits)) <= 256 && kGroupBits == 14, "one count and one word per thread");
  __shared__ uint32_t r[4], q[4];
  const unsigned long long w = full ? 0ull : a.mask[(int64_t)blockIdx.x * 256 + threadIdx.x];
  uint32_t n = threadIdx.x < blockIdx.x ? cnt[threadIdx.x] : 0;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off, 64);
  const uint32_t mine = __popcll(w);
  uint32_t incl = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_up(incl, off, 64);
    if (lane >= off) incl += o;
  }
  if (lane == 63) {
    r[wave] = n;
    q[wave] = incl;
  }
  __syncthreads();
  const int64_t earlier = before + ((r[0] + r[1]) + (r[2] + r[3]));
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0)
    *reinterpret_cast<int64_t*>(a.stat + kToySum) = earlier - a.kept + ((q[0] + q[1]) + (q[2] + q[3]));
  int64_t pos = earlier + (incl - mine);
  for (int v = 0; v < wave; ++v) pos += q[v];
  for (unsigned long long b = w; b; b &= b - 1, ++pos) {
    if (pos >= a.limit) return;
    const uint32_t j = 64 * (256 * blockIdx.x + threadIdx.x) + (uint32_t)__builtin_ctzll(b);
    const uint64_t e = (uint64_t)a.e0 + j;
    double ck, cj, phi, spare;
    phsp_angles(e, a.seed, ck, cj, phi, spare);
    a.out[0][pos] = a.m[j];
    a.out[1][pos] = ck;
    a.out[2][pos] = cj;
    a.out[3][pos] = phi;
    if (pos == a.limit - 1) *reinterpret_cast<uint64_t*>(a.stat + kToyLast) = e;
  }
}

// ------------------------------------------------------------------ launchers
template <typename T> hipError_t launch_invariants(const InvArgs<T>& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  const unsigned nb = (unsigned)((a.n + 255) / 256);
  hipLaunchKernelGGL(invariants_kernel<T>, dim3(nb), dim3(256), 0, st, a);
  return hipGetLastError();
}
template hipError_t launch_invariants<float>(const InvArgs<float>&, hipStream_t);
template hipError_t launch_invariants<double>(const InvArgs<double>&, hipStream_t);

template <typename T, class Sh, bool ZF>
hipError_t launch_amp_zf(const AmpArgs<T, Sh>& a, int mode, int nblocks, hipStream_t st) {
  const bool cc = a.tag != nullptr && mode != MODE_DENSITY;
  if (mode == MODE_GRAD) {
    if (cc) hipLaunchKernelGGL((amp_kernel<T, Sh, MODE_GRAD, true, ZF>), dim3(nblocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((amp_kernel<T, Sh, MODE_GRAD, false, ZF>), dim3(nblocks), dim3(256), 0, st, a);
  } else if (mode == MODE_NLL) {
    if (cc) hipLaunchKernelGGL((amp_kernel<T, Sh, MODE_NLL, true, ZF>), dim3(nblocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((amp_kernel<T, Sh, MODE_NLL, false, ZF>), dim3(nblocks), dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL((amp_kernel<T, Sh, MODE_DENSITY, false, ZF>), dim3(nblocks), dim3(256), 0, st, a);
  }
  return hipGetLastError();
}
template <typename T, class Sh>
hipError_t launch_amp(const AmpArgs<T, Sh>& a, int mode, int nblocks, hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  if constexpr (Sh::NZ >= 2) {
    if (a.zfree) {
      if (a.cnt[5] != 1) return hipErrorInvalidValue;   // refused by the host API
      return launch_amp_zf<T, Sh, true>(a, mode, nblocks, st);
    }
  } else {
    if (a.zfree) return hipErrorInvalidValue;
  }
  return launch_amp_zf<T, Sh, false>(a, mode, nblocks, st);
}
// Blocks of the per-event kernel that can be resident on one compute unit at once (from its
// register and LDS use), or 0 if the runtime cannot tell.
template <typename T, class Sh, bool ZF>
int amp_blocks_per_cu_zf(int mode, bool cc) {
  int nb = 0;
  hipError_t e;
  if (mode == MODE_GRAD)
    e = cc ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, amp_kernel<T, Sh, MODE_GRAD, true, ZF>, 256, 0)
           : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, amp_kernel<T, Sh, MODE_GRAD, false, ZF>, 256, 0);
  else if (mode == MODE_NLL)
    e = cc ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, amp_kernel<T, Sh, MODE_NLL, true, ZF>, 256, 0)
           : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, amp_kernel<T, Sh, MODE_NLL, false, ZF>, 256, 0);
  else e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, amp_kernel<T, Sh, MODE_DENSITY, false, ZF>, 256, 0);
  return (e == hipSuccess && nb > 0) ? nb : 0;
}
template <typename T, class Sh>
int amp_blocks_per_cu(int mode, bool cc, bool zfree) {
  if constexpr (Sh::NZ >= 2) {
    if (zfree) return amp_blocks_per_cu_zf<T, Sh, true>(mode, cc);
  }
  return amp_blocks_per_cu_zf<T, Sh, false>(mode, cc);
}
template int amp_blocks_per_cu<float, ShapeSmall>(int, bool, bool);
template int amp_blocks_per_cu<double, ShapeSmall>(int, bool, bool);
template int amp_blocks_per_cu<float, ShapeFull>(int, bool, bool);
template int amp_blocks_per_cu<double, ShapeFull>(int, bool, bool);

template hipError_t launch_amp<float, ShapeSmall>(const AmpArgs<float, ShapeSmall>&, int, int, hipStream_t);
template hipError_t launch_amp<double, ShapeSmall>(const AmpArgs<double, ShapeSmall>&, int, int, hipStream_t);
template hipError_t launch_amp<float, ShapeFull>(const AmpArgs<float, ShapeFull>&, int, int, hipStream_t);
template hipError_t launch_amp<double, ShapeFull>(const AmpArgs<double, ShapeFull>&, int, int, hipStream_t);

hipError_t launch_reduce_final(const double* partial, int nb_data, int nb_mc, int n_mc_sets, int nv, double* out,
                               int first_set, int n_sets, hipStream_t st) {
  if (first_set < 0 || n_sets < 1 || n_mc_sets < 1 || n_mc_sets > 2 || first_set + n_sets > 1 + n_mc_sets)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(reduce_final, dim3(n_sets * nv), dim3(256), 0, st, partial, nb_data, nb_mc, n_mc_sets, nv, out,
                     first_set);
  return hipGetLastError();
}
hipError_t launch_hist_lookup(const HistArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(hist_lookup_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_template(const TplArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(template_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_phsp(const GenArgs& a, hipStream_t st) {
  if (a.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(phsp_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}
// One chunk of toys: the proposals, the densities of the listed ones, and the accepted events.
template <class Sh> hipError_t launch_toys(const ToyAmpArgs<Sh>& a, int n_cu, hipStream_t st) {
  const ToyArgs& t = a.toys;
  const int64_t n = (int64_t)t.rounds << kRoundBits;
  const int groups = (int)(n >> kGroupBits);
  if (t.rounds < 1 || t.rounds > kMaxRounds || t.per_wave < 64 || t.per_wave > kPerWave || n % (4 * kToyLists * t.per_wave))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(propose_kernel, dim3((unsigned)(n / (4 * t.per_wave))), dim3(256), 0, st, t);
  ToyAmpArgs<Sh> b = a;
  b.nb_data = (2 * n_cu + kToyLists - 1) / kToyLists * kToyLists;   // whole blocks per list
  if constexpr (Sh::NZ >= 2) {
    if (a.zfree) {
      if (a.cnt[5] != 1) return hipErrorInvalidValue;   // refused by the host API
      hipLaunchKernelGGL((amp_kernel<double, Sh, MODE_TOYS, false, true>), dim3(b.nb_data), dim3(256), 0, st, b);
    } else {
      hipLaunchKernelGGL((amp_kernel<double, Sh, MODE_TOYS, false, false>), dim3(b.nb_data), dim3(256), 0, st, b);
    }
  } else {
    if (a.zfree) return hipErrorInvalidValue;
    hipLaunchKernelGGL((amp_kernel<double, Sh, MODE_TOYS, false, false>), dim3(b.nb_data), dim3(256), 0, st, b);
  }
  hipLaunchKernelGGL(count_kernel, dim3(groups), dim3(256), 0, st, t);
  hipLaunchKernelGGL(collect_kernel, dim3(groups), dim3(256), 0, st, t);
  return hipGetLastError();
}
template <class Sh> hipError_t launch_toy_bound(const ToyAmpArgs<Sh>& a, hipStream_t st) {
  hipLaunchKernelGGL(bound_kernel<Sh>, dim3(1), dim3(kBins), 0, st, a);
  return hipGetLastError();
}
template hipError_t launch_toys<ShapeSmall>(const ToyAmpArgs<ShapeSmall>&, int, hipStream_t);
template hipError_t launch_toys<ShapeFull>(const ToyAmpArgs<ShapeFull>&, int, hipStream_t);
template hipError_t launch_toy_bound<ShapeSmall>(const ToyAmpArgs<ShapeSmall>&, hipStream_t);
template hipError_t launch_toy_bound<ShapeFull>(const ToyAmpArgs<ShapeFull>&, hipStream_t);

}  // namespace kpsi
