// Interference matrix of the normalisation integral (gfx950 matrix cores).
//
// With a_xi = sum_k c_k B_k,xi (complex couplings c_k, per-event component amplitudes
// B_k,xi = A_R(m) x angular factor of Eq. 4 or Eq. 10), the MC normalisation sum is
//   sum_j eps_j S(y_j) = sum_kl c_k conj(c_l) I_kl,   I_kl = sum_j eps_j sum_xi B_k,xi conj(B_l,xi),
// and its derivative with respect to a lineshape parameter p of resonance R needs
//   D^p_kl = sum_j eps_j sum_xi dB_k,xi/dp conj(B_l,xi)   (k in R).
// Both are blocks of the real Gram matrix G = X^T X of the matrix X whose rows are
// (event, xi), each scaled by sqrt(eps) of its event, and whose columns are the real and
// imaginary parts of the components followed by the derivative components.  G is accumulated
// over 16x16 tiles of its upper triangle on the matrix cores: v_mfma_f32_16x16x4f32 for FP32
// rows (FP32 sums over one 64-row tile, then FP64 sums), v_mfma_f64_16x16x4f64 for FP64 rows.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "kpsi_internal.h"
#include "kpsi_math.h"

namespace kpsi {

namespace im {

template <typename T> struct cx { T re, im; };
struct four {
  double a, b, c, d;
  __device__ __forceinline__ double& operator[](int i) { return i == 0 ? a : i == 1 ? b : i == 2 ? c : d; }
};
typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));

}  // namespace im

// One wavefront per block, one event per lane, 64 events per tile.
//
// The rows of an event are its amplitudes in the transversity basis, X = (a_+ + a_-)/sqrt2 and
// Y = (a_+ - a_-)/sqrt2 (a unitary change of the two rows), and the columns of a K* of spin >= 1 are
// p ~ b_+ - b_-, m ~ b_+ + b_- and u ~ b_0 of its helicity components:
//   X: p = a1 cos phi,            m = i a1 sin phi,          u = 0
//   Y: p = i a1 cos th_J sin phi, m = a1 cos th_J cos phi,   u = a0 sin th_J
// times the lineshape n_J / D (a1 = sin ang1, a0 = ang0, as in the per-event kernel); likewise the Z
// columns (with free helicities, the sum and difference of lambda' = +-1).  Every factor is real or
// imaginary, so a column takes two products where the helicity form took four, each lane evaluates
// its event's K* lineshapes once for both rows (before, once per row), and the X rows need only the
// tiles of the p, m and Z columns, which come first.  Constant factors and the change back to
// helicity components are the host's, in double precision.
// Column order (complex): derivatives of p, m and Z columns; p and m of each K* slot; Z; u of each K*
// slot; derivatives of u.
//
// What bounds it (counters, 2e6 events of the full model in FP32): the FP32 and FP64 matrix instructions
// occupy the vector units (another wavefront's vector instructions do not overlap with them); their 304
// times 32 cycles per 64 events are 48% of the kernel's cycles, the other vector instructions 18%.  In the last
// third neither issues: the two wavefronts of a SIMD wait for LDS operands, for the columns, and for the 64
// to 80 bytes per lane of accumulators that the FP32 kernel of 80 columns keeps in scratch (41 to 55
// registers; with one wavefront per SIMD and no scratch it took 338 against 320 us).  2e6 events in FP32:
// 326 us in the helicity form (448 matrix instructions per 64 events, two evaluations of every
// lineshape), now 250 to 260 us, and the result is 5 times closer to double precision (no rounded constant
// is left in it).
// ZF: one Z whose H'_{+1} and H'_{-1} are independent couplings: three Z columns.
template <typename T, class Sh, int C, bool ZF>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 2 : 1)))
void imatrix_kernel(const ImArgs<T, Sh> a) {
  using namespace im;
  constexpr int NT = C / 16;
  constexpr int NTILE = NT * (NT + 1) / 2;
  static_assert(!ZF || Sh::NZ >= 2, "free Z helicities use the second Z's columns");
  constexpr int NK = Sh::NK, N0 = Sh::N[0];
  constexpr int NZ = ZF ? 1 : Sh::NZ;   // Z slots evaluated
  constexpr int ZN = ZF ? 3 : 2;        // columns per Z slot
  // Rows are staged at the context precision in dynamic LDS sized for the columns in use (the
  // padded width C is only the MFMA tiling): FP32 rows of the 72-column benchmark model take
  // 18.7 KB, so eight one-wavefront blocks fit per compute unit (two per SIMD).  The row stride
  // LDX = ncols + 1 is odd: the lanes writing a column hit different banks.  Column ncols of every
  // row is never written and stays zero; the matrix phase reads it in place of the columns that
  // are not there.  Each row is scaled by sqrt(eps) of its event, so the Gram product of the
  // rows with themselves carries the weight eps once.
  extern __shared__ double im_smem[];
  T* X = reinterpret_cast<T*>(im_smem);
  const int LDX = a.ncols + 1;
  const int lane = threadIdx.x;
  // (in FP32 plain doubles: groups of eight consecutive registers are hard to place)
  using acc_t = std::conditional_t<std::is_same_v<T, float>, four, d4_t>;
  acc_t acc[NTILE];
#pragma unroll
  for (int t = 0; t < NTILE; ++t) acc[t] = acc_t{0.0, 0.0, 0.0, 0.0};

  const int64_t ntiles = (a.n + 63) / 64;
  // Every tile writes the same row positions (the columns of the model's components and
  // derivatives), so the rows are cleared once: the columns of empty slots stay zero.
  for (int i = lane; i < 64 * LDX; i += 64) X[i] = T(0);

  // The event columns of this lane's event in the next tile are fetched before the last matrix phase
  // of the current one, so their latency hides behind it.  Column groups of four (K* chain:
  // 0-11; Z angular factors: 12-15, present when the model has Z states; with free Z
  // helicities 16-17 as well).  A lane past the last event reads that event with weight zero.
  using V4 = T __attribute__((ext_vector_type(4)));
  const V4* __restrict__ gcol = reinterpret_cast<const V4*>(a.cols);
  const int64_t ld = a.ld;
  const int nz = a.cnt[5];
  const bool zon = NZ > 0 && nz > 0;
  V4 g0{}, g1{}, g2{}, g3{}, g4{};
  T wv = T(0);
  auto fetch = [&](int64_t tile) {
    if (tile >= ntiles) return;
    const int64_t i = tile * 64 + lane, e = i < a.n ? i : a.n - 1;
    g0 = gcol[e];
    g1 = gcol[ld + e];
    g2 = gcol[2 * ld + e];
    if (zon) g3 = gcol[3 * ld + e];
    if (ZF && zon) g4 = gcol[4 * ld + e];
    wv = i < a.n ? (a.eps ? a.eps[e] : T(1)) : T(0);
  };
  fetch(blockIdx.x);

  const unsigned flt = a.flt, flt1 = a.flt1;   // slots (K*, then Z) with a floating lineshape; the one of slot 1
  T* const row = X + lane * LDX;
  T* const rowA = row + 2 * a.baseA;   // p, m of the K* slots, then the Z columns
  T* const rowB = row + 2 * a.baseB;   // u of the K* slots
  // column c of this lane's row: A times the real or imaginary factor g
  auto putR = [](T* r, int c, const cx<T>& A, T g) { r[2 * c] = A.re * g; r[2 * c + 1] = A.im * g; };
  auto putI = [](T* r, int c, const cx<T>& A, T g) { r[2 * c] = -A.im * g; r[2 * c + 1] = A.re * g; };
  const int r16 = lane & 15, k4 = lane >> 4;
  // Gram tiles of the first NX column tiles of the rows: A[i][k] = X[row][16 ti + i],
  // B[k][j] = X[row][16 tj + j], row = s + 16 k; lane = i + 16 k provides A[i][k] and B[k][j = i]
  // (with the odd row stride, the four rows of a read lie in different quarters of the banks).
  // The A and B operands of a row group are the same LDS elements, so each group loads NX values per
  // lane and feeds all tiles; consecutive MFMAs accumulate into different tiles.  The next group's
  // values are read from LDS before the current group's MFMAs are issued.  Tile (0, 0) is left at
  // zero when it holds only derivative x derivative products: nothing reads them.
  auto gram = [&](auto NXc, int live) {
    constexpr int NX = decltype(NXc)::value;
    // tile (ti, tj) of the upper triangle, in the order of the partial records
    auto index = [](int ti, int tj) constexpr { return ti * NT - ti * (ti - 1) / 2 + (tj - ti); };
    int cofs[NX];   // this lane's column of each tile, those not there mapped to the zero column
#pragma unroll
    for (int t = 0; t < NX; ++t) cofs[t] = 16 * t + r16 < live ? 16 * t + r16 : a.ncols;
    T nx[NX];
#pragma unroll
    for (int t = 0; t < NX; ++t) nx[t] = X[16 * k4 * LDX + cofs[t]];
    auto steps = [&](auto&& mma) {
#pragma unroll 2
      for (int s = 0; s < 16; ++s) {
        T v[NX];
#pragma unroll
        for (int t = 0; t < NX; ++t) v[t] = nx[t];
        if (s + 1 < 16) {
          const int rw = s + 1 + 16 * k4;
#pragma unroll
          for (int t = 0; t < NX; ++t) nx[t] = X[rw * LDX + cofs[t]];
        }
        // keep those reads ahead of the MFMAs in the instruction stream
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ti = 0; ti < NX; ++ti) {
#pragma unroll
          for (int tj = ti; tj < NX; ++tj) {
            if (ti == 0 && tj == 0 && a.skip_first) continue;
            mma(index(ti, tj), v[ti], v[tj]);
          }
        }
      }
    };
    if constexpr (std::is_same_v<T, float>) {
      // FP32 rows: FP32 matrix cores (each product of two FP32 values, summed in FP32 over 64
      // rows), then these sums are added into the FP64 accumulators.  Accumulator layout of
      // the 32-bit form: lane l, register r hold row 4 (l / 16) + r, column l % 16.
      f4_t a32[NTILE];   // (those of the first NX column tiles are used)
#pragma unroll
      for (int ti = 0; ti < NX; ++ti)
#pragma unroll
        for (int tj = ti; tj < NX; ++tj) a32[index(ti, tj)] = f4_t{0.f, 0.f, 0.f, 0.f};
      steps([&](int t, float x, float y) { a32[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, a32[t], 0, 0, 0); });
#pragma unroll
      for (int ti = 0; ti < NX; ++ti)
#pragma unroll
        for (int tj = ti; tj < NX; ++tj)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[index(ti, tj)][r] += (double)a32[index(ti, tj)][r];
    } else {
      // FP64 rows: FP64 matrix cores.  Accumulator layout of the FP64 form: lane l, register r
      // hold row l / 16 + 4 r, column l % 16.
      steps([&](int t, double x, double y) { acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc[t], 0, 0, 0); });
    }
  };

  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    // (the constants are read again for each tile: kept over the loop they would fill the registers)
    const auto& ka = *kernarg_laundered<ImArgs<T, Sh>>();
    const T m = g0.x, q = g0.y, pB = g0.z, cK = g0.w;
    const T sK = g1.x, cJ = g1.y, sJ = g1.z, cph = g1.w;
    const T sph = g2.x, qm = g2.z;   // column 10: q/m
    const T sw = sqrt_(wv);
    const T qq = q * q, zR = ka.rR2 * qq, zB = ka.rB2 * (pB * pB);
    // derivative columns of the lineshape A = n / D, D = M^2 - s - i P g: E = A / D and F = i g E.  The
    // host makes dA/dM = kappa A - 2M E + dP/dM F and dA/dGamma0 = P/Gamma0 F of their sums.
    auto derivatives = [&](const cx<T>& A, T dre, T dim, T inv, T g, cx<T>& E, cx<T>& F) {
      E = cx<T>{(A.re * dre - A.im * dim) * inv, (A.re * dim + A.im * dre) * inv};
      F = cx<T>{-g * E.im, g * E.re};
    };
    // ---- K* chain: the X row, and the u columns of the Y row, which the X rows do not use (each
    // resonance is written as soon as it is known: nothing of it is kept in registers)
    auto do_spin = [&](auto Jc) {
      constexpr int J = decltype(Jc)::value;
      if constexpr (Sh::N[J] > 0) {
        constexpr int LB = LBof<J>::v, sb = slot_base<Sh>(J);
        const T BB = bpoly<LB>(zB), rJ = rsq_(bpoly<J>(zR) * BB);
        // n_J with the row weight sqrt(eps) folded in; 1/B_J(z_R) = rJ^2 B_LB(z_B)
        const T nJ = ipow<T, LB>(pB) * ipow<T, J>(qm) * rJ * sw;
        T gJ = qm;
        if constexpr (J > 0) gJ = qm * ipow<T, J>(qq) * (rJ * rJ * BB);
        const T a0 = ang0<J>(cK) * sJ, a1 = sK * ang1<J>(cK);
        const T fp = a1 * cph, fm = a1 * sph;
        auto pm = [&](T* r, int c, const cx<T>& A) {   // columns c (p) and c + 1 (m)
          putR(r, c, A, fp);
          putI(r, c + 1, A, fm);
        };
#pragma unroll
        for (int j = 0; j < Sh::N[J]; ++j) {
          const auto& rc = ka.rc[sb + j];   // (an empty slot has M^2 = P = 0; nothing reads its columns)
          const T dre = pole_gap_m(rc.M2, rc.M2lo, m), dim = rc.P * gJ;
          const T inv = rcp_(fma_(dre, dre, dim * dim));
          const T sc = nJ * inv;
          cx<T> A{sc * dre, sc * dim};
          if constexpr (J == 0) {
            if (ka.lass >> (sb + j) & 1) {
              // LASS (Eq. 7-8): u = q cot(delta_B) = 1/a + b q^2/2; the non-resonant term is
              // m (u + i q)/(u^2 + q^2), the resonant one P e^{2 i delta_B} times the Breit-Wigner
              const T u = ka.lhb[sb + j] * qq + ka.lai[sb + j];
              const T dn = rcp_(u * u + qq);
              const T er = (u * u - qq) * dn, ei = T(2) * u * q * dn;
              const T md = m * dn * nJ;
              A = cx<T>{md * u + rc.P * (er * A.re - ei * A.im), md * q + rc.P * (er * A.im + ei * A.re)};
            }
          }
          if constexpr (J > 0) pm(rowA, 2 * (sb + j - N0), A);
          putR(rowB, sb + j, A, a0);
          if (flt >> (sb + j) & 1) {
            cx<T> E, F;
            derivatives(A, dre, dim, inv, gJ, E, F);
            const int f = flt1 >> (sb + j) & 1, cA = ka.dA[f], cB = ka.dB[f];
            if constexpr (J > 0) {
              pm(row, cA, E);
              pm(row, cA + 2, F);
            }
            putR(row, cB, E, a0);
            putR(row, cB + 1, F, a0);
          }
        }
      }
    };
    do_spin(std::integral_constant<int, 0>{});
    do_spin(std::integral_constant<int, 1>{});
    do_spin(std::integral_constant<int, 2>{});
    do_spin(std::integral_constant<int, 3>{});
    do_spin(std::integral_constant<int, 4>{});
    // ---- Z chain: columns i f0, i f1 (f2) in X and f0, f1 (i f2) in Y.  The angular columns carry the
    // Z barrier factor n_Z; the xi = -1 factors are (-Re, Im) of the xi = +1 ones, or with free
    // helicities F+- beside F++.  Evaluated for each of the two rows: kept over the matrix phase, the
    // lineshapes and derivatives would not fit the registers.
    auto z_row = [&](auto Yc, const auto& kc) {
      constexpr bool Y = decltype(Yc)::value;
      const T mz2 = g2.y, gz = g2.w;
      const T f0 = Y ? g3.x : g3.y;
      T f1 = Y ? g3.z : g3.w, f2 = T(0);
      if constexpr (ZF) {
        f1 = Y ? g3.z - g4.x : g3.w + g4.y;
        f2 = Y ? g3.w - g4.y : g3.z + g4.x;
      }
      auto zcol = [&](T* r, int c, const cx<T>& A) {
        if constexpr (Y) {
          putR(r, c, A, f0);
          putR(r, c + 1, A, f1);
          if constexpr (ZF) putI(r, c + 2, A, f2);
        } else {
          putI(r, c, A, f0);
          putI(r, c + 1, A, f1);
          if constexpr (ZF) putR(r, c + 2, A, f2);
        }
      };
#pragma unroll
      for (int z = 0; z < NZ; ++z) {
        if (z >= nz) continue;
        const auto& rc = kc.rc[NK + z];
        const T dre = pole_gap(rc.M2, rc.M2lo, mz2), dim = rc.P * gz;
        const T inv = rcp_(fma_(dre, dre, dim * dim));
        const T sc = inv * sw;
        const cx<T> A{sc * dre, sc * dim};
        zcol(rowA, 2 * (NK - N0) + ZN * z, A);
        if (flt >> (NK + z) & 1) {
          cx<T> E, F;
          derivatives(A, dre, dim, inv, gz, E, F);
          const int f = flt1 >> (NK + z) & 1, cA = kc.dA[f];
          zcol(row, cA, E);
          zcol(row, cA + ZN, F);
        }
      }
    };
    if (zon) z_row(std::false_type{}, ka);
    __syncthreads();
    // the X rows fill the first baseB columns only: at most NXM tiles (the u columns come behind them)
    constexpr int NXM = (C - 2 * NK + 15) / 16;
    if constexpr (NXM > 1) {
      if (2 * a.baseB <= 16 * (NXM - 1)) gram(std::integral_constant<int, NXM - 1>{}, 2 * a.baseB);
      else gram(std::integral_constant<int, NXM>{}, 2 * a.baseB);
    } else {
      gram(std::integral_constant<int, 1>{}, 2 * a.baseB);
    }
    __syncthreads();
    // ---- the Y row: p and m are cos th_J times the X row's m and p, so nothing of the K* chain is kept
    // over the matrix phase
    {
      const auto& kb = *kernarg_laundered<ImArgs<T, Sh>>();
      auto turn = [&](T* r, int c) {
        const T p0 = r[2 * c], p1 = r[2 * c + 1], m0 = r[2 * c + 2], m1 = r[2 * c + 3];
        r[2 * c] = cJ * m0;
        r[2 * c + 1] = cJ * m1;
        r[2 * c + 2] = cJ * p0;
        r[2 * c + 3] = cJ * p1;
      };
      auto turn_spin = [&](auto Jc) {
        constexpr int J = decltype(Jc)::value;
        constexpr int sb = slot_base<Sh>(J);
#pragma unroll
        for (int j = 0; j < Sh::N[J]; ++j) {
          turn(rowA, 2 * (sb + j - N0));
          if (!(flt >> (sb + j) & 1)) continue;
          const int f = flt1 >> (sb + j) & 1;
          turn(row, kb.dA[f]);
          turn(row, kb.dA[f] + 2);
        }
      };
      turn_spin(std::integral_constant<int, 1>{});
      turn_spin(std::integral_constant<int, 2>{});
      turn_spin(std::integral_constant<int, 3>{});
      turn_spin(std::integral_constant<int, 4>{});
      if (zon) z_row(std::true_type{}, kb);
    }
    fetch(tile + gridDim.x);
    __syncthreads();
    gram(std::integral_constant<int, NT>{}, a.ncols);
    __syncthreads();
  }
  // ---- block partial: the four accumulator registers of (tile t, lane) are values
  //      v = (t*64 + lane)*4 + r, stored as one 32-byte record per (t, lane) and block at
  //      record (t*64 + lane) * nb + block (blocks of one record group adjacent)
  const int nb = gridDim.x;
  d4_t* P = reinterpret_cast<d4_t*>(a.partial);
#pragma unroll
  for (int t = 0; t < NTILE; ++t) P[((int64_t)t * 64 + lane) * nb + blockIdx.x] = d4_t{acc[t][0], acc[t][1], acc[t][2], acc[t][3]};
}

// Fixed-order compensated sums over blocks of the 32-byte partial records: block g sums record
// group g (values 4g .. 4g+3) over the nb blocks into out[4g + r].
__global__ __launch_bounds__(256) void reduce_values(const double* __restrict__ partial, int nb, double* out) {
  using im::d4_t;
  const int g = blockIdx.x;
  const d4_t* p = reinterpret_cast<const d4_t*>(partial) + (int64_t)g * nb;
  double s[4] = {0.0, 0.0, 0.0, 0.0}, c[4] = {0.0, 0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < nb; b += 256) {
    const d4_t x4 = p[b];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double x = x4[r];
      const double t = s[r] + x;
      c[r] += (fabs(s[r]) >= fabs(x)) ? (s[r] - t) + x : (x - t) + s[r];
      s[r] = t;
    }
  }
  __shared__ double S[4][256], Cc[4][256];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    S[r][threadIdx.x] = s[r];
    Cc[r][threadIdx.x] = c[r];
  }
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (threadIdx.x < w) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double a = S[r][threadIdx.x], b = S[r][threadIdx.x + w];
        const double tt = a + b, bp = tt - a;
        const double err = (a - (tt - bp)) + (b - bp);
        S[r][threadIdx.x] = tt;
        Cc[r][threadIdx.x] = Cc[r][threadIdx.x] + Cc[r][threadIdx.x + w] + err;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x < 4) out[4 * g + threadIdx.x] = S[threadIdx.x][0] + Cc[threadIdx.x][0];
}

// dynamic LDS of a block: 64 rows of ncols + 1 values
template <typename T> size_t imatrix_smem(int ncols) { return 64 * (size_t)(ncols + 1) * sizeof(T); }

template <typename T, class Sh, int C>
hipError_t launch_imatrix_c(const ImArgs<T, Sh>& a, int nb, double* out, hipStream_t st) {
  if (a.ncols <= 0 || a.ncols > C || (a.ncols & 1) || a.n <= 0 || a.baseB + Sh::NK > a.ncols / 2) return hipErrorInvalidValue;
  if constexpr (Sh::NZ >= 2) {
    if (a.zfree) {
      if (a.cnt[5] != 1) return hipErrorInvalidValue;   // refused by the host API
      hipLaunchKernelGGL((imatrix_kernel<T, Sh, C, true>), dim3(nb), dim3(64), imatrix_smem<T>(a.ncols), st, a);
    } else {
      hipLaunchKernelGGL((imatrix_kernel<T, Sh, C, false>), dim3(nb), dim3(64), imatrix_smem<T>(a.ncols), st, a);
    }
  } else {
    if (a.zfree) return hipErrorInvalidValue;
    hipLaunchKernelGGL((imatrix_kernel<T, Sh, C, false>), dim3(nb), dim3(64), imatrix_smem<T>(a.ncols), st, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  constexpr int NT = C / 16;
  const int nv = NT * (NT + 1) / 2 * 256;
  hipLaunchKernelGGL(reduce_values, dim3(nv / 4), dim3(256), 0, st, a.partial, nb, out);
  return hipGetLastError();
}

template <typename T, class Sh, int C> int imatrix_blocks_per_cu_c(int ncols) {
  int nb = 0;
  const hipError_t e =
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, imatrix_kernel<T, Sh, C, false>, 64, imatrix_smem<T>(ncols));
  return (e == hipSuccess && nb > 0) ? nb : 0;
}
// Blocks (one wavefront each) of the interference-matrix kernel resident per compute unit.
template <typename T, class Sh> int imatrix_blocks_per_cu(int ncols) {
  if (ncols <= 16) return imatrix_blocks_per_cu_c<T, Sh, 16>(ncols);
  if (ncols <= 32) return imatrix_blocks_per_cu_c<T, Sh, 32>(ncols);
  if (ncols <= 64) return imatrix_blocks_per_cu_c<T, Sh, 64>(ncols);
  return imatrix_blocks_per_cu_c<T, Sh, 80>(ncols);
}
template int imatrix_blocks_per_cu<float, ShapeSmall>(int);
template int imatrix_blocks_per_cu<double, ShapeSmall>(int);
template int imatrix_blocks_per_cu<float, ShapeFull>(int);
template int imatrix_blocks_per_cu<double, ShapeFull>(int);

template <typename T, class Sh>
hipError_t launch_imatrix(const ImArgs<T, Sh>& a, int ncols, int nb, double* out, hipStream_t st) {
  if (ncols <= 16) return launch_imatrix_c<T, Sh, 16>(a, nb, out, st);
  if (ncols <= 32) return launch_imatrix_c<T, Sh, 32>(a, nb, out, st);
  if (ncols <= 64) return launch_imatrix_c<T, Sh, 64>(a, nb, out, st);
  if (ncols <= 80) return launch_imatrix_c<T, Sh, 80>(a, nb, out, st);
  return hipErrorInvalidValue;
}
template hipError_t launch_imatrix<float, ShapeSmall>(const ImArgs<float, ShapeSmall>&, int, int, double*, hipStream_t);
template hipError_t launch_imatrix<double, ShapeSmall>(const ImArgs<double, ShapeSmall>&, int, int, double*, hipStream_t);
template hipError_t launch_imatrix<float, ShapeFull>(const ImArgs<float, ShapeFull>&, int, int, double*, hipStream_t);
template hipError_t launch_imatrix<double, ShapeFull>(const ImArgs<double, ShapeFull>&, int, int, double*, hipStream_t);

}  // namespace kpsi
