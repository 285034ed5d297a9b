// Symmetric interior penalty DG Laplacian, matrix-free, on the affine n^3 mesh (the
// discretisation of the paper's multigrid experiment, Sec. 6.1).  Per cell the discontinuous
// Q_p basis on the GLL nodes; DoF (a,b,c) of cell K at K (p+1)^3 + a + (p+1) b + (p+1)^2 c.
//
//   a(u,v) = sum_K int_K grad u . grad v
//          + sum_F int_F ( -{d_n u}[v] - {d_n v}[u] + sigma [u][v] ),   sigma = 2 (p+1)^2 / h,
//
// interior faces with n from the lower cell L to the upper cell R, [u] = u_L - u_R, {w} the mean;
// boundary faces with the outside values zero and the inside value instead of the mean
// (homogeneous Dirichlet data imposed weakly).
//
// One kernel computes the whole operator per cell in tensor-product form (dg_kron_kernel, below):
// CPW consecutive cells of an x-row per workgroup, one lane per 1D line of a cell; each cell's
// result is written once.
#include "kernels_common.hpp"

#include <type_traits>

// Lanes per workgroup that the cells fill (one lane per 1D line): 128 up to degree 4 (5 cells of
// 25 lanes at p = 4), 256 above (at p >= 6 a 128-lane workgroup would hold a single cell).
#ifndef MFQ_DG_LANES
#define MFQ_DG_LANES(P) ((P) <= 4 ? 128 : 256)
#endif

namespace mfq {
namespace {

template <int P>
struct DgCell {
  static constexpr int N1 = P + 1;
  static constexpr int T = N1 * N1;
  static constexpr int NQ = N1 * T;
  static constexpr int CPW = MFQ_DG_LANES(P) / T > 0 ? MFQ_DG_LANES(P) / T : 1;  // cells per workgroup
  static constexpr int THREADS = CPW * T;
};

// What the kernel does with its result v = (A src)_i before storing (one pass over the vectors,
// fused with the operator):
//   kStore:    dst = v
//   kChebStep: r -= v; dnew = c1 src + c2 dinv r; x += dnew   (a Chebyshev step, src = d; dnew
//              must be another buffer since other cells still read src)
//   kResidual: r = b - v
enum DgEpilogueMode { kStore = 0, kChebStep = 1, kResidual = 2 };
template <typename Real>
struct DgEpilogue {
  int mode;
  Real* dst;
  const Real* b;
  const Real* dinv;
  Real* x;
  Real* r;
  Real* dnew;
  Real c1, c2;
};

// Tensor-product form of the whole operator.  On the affine cube mesh every term of a(u, v)
// factorises over the three directions: with the Gauss rule's 1D mass matrix M = S^T diag(w) S
// and stiffness matrix K = D^T diag(w) D on the reference interval,
//
//   A u = sum_d (M x M)_{tangential to d} w_d,   w_d = h K u + (face terms of the faces normal to d)
//
// along every line of the cell in direction d: the cell term of direction d is h (K x M x M)
// (h^3 from the cell measure, h^-2 from the two derivatives), and the terms of a face normal to d
// are h^2 (M x M) applied to sigma [u] - {d_n u} at the face layer and, from d_n v = l'_a / h, to
// -f h [u] times l'_a at the face end along the line (f = 1/2 on interior faces, 1 on boundary
// faces).  The trace of a line on a face is its GLL end node and its normal derivative a dot
// product with l'_a at the end point, so w_d needs only the cell's own line and the two
// neighbours' lines through the faces it touches.  Per cell one lane per 1D line forms w_d for the
// three directions, and the tangential mass matrices act in five 1D passes,
//
//   A u = M_z (M_y w_x + M_x w_y) + M_x M_y w_z,
//
// in place in two LDS arrays per cell (each pass reads and writes only its own lane's line, with a
// barrier between passes).  K and M are symmetric about their centre, so every 1D contraction
// uses the even-odd form: eight per line in all.
template <int P, typename Real>
struct DgKron {
  EvenOdd<P + 1, Real> K;  // sum_q w_q l_a'(zeta_q) l_b'(zeta_q)
  EvenOdd<P + 1, Real> M;  // sum_q w_q l_a(zeta_q) l_b(zeta_q)
  Real d0[P + 1];          // l_a'(0)
  Real d1[P + 1];          // l_a'(1)
};

template <int P, typename Real>
DgKron<P, Real> make_dg_kron() {
  constexpr int N1 = P + 1;
  const Tables1D& tb = tables(P);
  double K[N1 * N1], M[N1 * N1];
  for (int a = 0; a < N1; ++a)
    for (int b = 0; b < N1; ++b) {
      double k = 0, m = 0;
      for (int q = 0; q < N1; ++q) {
        k += tb.omega[q] * tb.D[q * N1 + a] * tb.D[q * N1 + b];
        m += tb.omega[q] * tb.S[q * N1 + a] * tb.S[q * N1 + b];
      }
      K[a * N1 + b] = k;
      M[a * N1 + b] = m;
    }
  DgKron<P, Real> t{};
  t.K = make_even_odd<N1, Real>(K);
  t.M = make_even_odd<N1, Real>(M);
  for (int a = 0; a < N1; ++a) {
    t.d0[a] = (Real)lagrange_derivative(tb.xi, a, 0.0);
    t.d1[a] = (Real)lagrange_derivative(tb.xi, a, 1.0);
  }
  return t;
}

// A neighbour's line, as far as this cell needs it: its end value on the shared face and its derivative
// there (both zero where the neighbour is absent).
template <typename Real>
struct DgEnd {
  Real u, du;
};
// the line's end at 1 (UPPER: at 0) ; v(a) its values
template <int N1, bool UPPER, typename Real, typename KT, class F>
__device__ __forceinline__ DgEnd<Real> dg_end(const KT& kt, F v) {
  DgEnd<Real> e{0, 0};
#pragma unroll
  for (int a = 0; a < N1; ++a) {
    const Real x = v(a);
    e.du = fmad(UPPER ? kt.d0[a] : kt.d1[a], x, e.du);
    if (a == (UPPER ? 0 : N1 - 1)) e.u = x;
  }
  return e;
}

// w = h K u + the face terms of one line's two faces, from the line u of the cell and the ends of its
// neighbours' lines below and above
template <int N1, typename Real, typename KT>
__device__ __forceinline__ void dg_line_terms(const Real (&u)[N1], const DgEnd<Real>& lo, const DgEnd<Real>& hi,
                                              bool hasLo, bool hasHi, Real h, Real ih, Real h2, Real sigma,
                                              const KT& kt, Real (&w)[N1]) {
  Real dK0 = 0, dK1 = 0;
#pragma unroll
  for (int a = 0; a < N1; ++a) {
    dK0 = fmad(kt.d0[a], u[a], dK0);
    dK1 = fmad(kt.d1[a], u[a], dK1);
  }
  // jump and mean normal derivative on the lower face (this cell its upper side) and the upper
  // face; on a boundary face the outside is zero and the inside derivative replaces the mean
  const Real jLo = lo.u - u[0], jHi = u[N1 - 1] - hi.u;
  const Real mLo = hasLo ? (Real)0.5 * ih * (lo.du + dK0) : ih * dK0;
  const Real mHi = hasHi ? (Real)0.5 * ih * (dK1 + hi.du) : ih * dK1;
  const Real fLo = hasLo ? (Real)0.5 : (Real)1, fHi = hasHi ? (Real)0.5 : (Real)1;
  const Real VLo = h2 * (sigma * jLo - mLo), DLo = -fLo * h * jLo;
  const Real VHi = h2 * (sigma * jHi - mHi), DHi = -fHi * h * jHi;
  Real ku[N1];
  eo_apply<N1, 1, false>(kt.K, u, ku);
#pragma unroll
  for (int a = 0; a < N1; ++a) {
    Real v = h * ku[a];
    if (a == 0) v -= VLo;
    if (a == N1 - 1) v += VHi;
    v = fmad(DLo, kt.d0[a], v);
    w[a] = fmad(DHi, kt.d1[a], v);
  }
}

// Rules per degree and type, from times on MI355X in us (at the sizes given, without / with):
// early: the lines beyond the row segment's ends are asked for with all others, not after the first barrier
// (one memory latency less, the ends' registers and descriptors more).  FP64 Q3 50^3 39.2 / 38.5, Q4 40^3
// 40.4 / 37.8, Q5 16^3 10.6 / 10.2 and 53^3 215 / 194, Q7 6^3 8.8 / 8.2 and 40^3 188 / 169, Q8 36^3 256 / 230;
// not Q1 160^3 188 / 209, Q2 107^3 228 / 233, Q6 (spilled scalars) 14^3 12.6 / 14.2; FP32 Q4 40^3 27.4 / 25.8,
// Q6 46^3 106 / 102, not Q8 36^3 110 / 119.
constexpr bool dg_early(int p, bool fp64) { return fp64 ? p >= 3 && p != 6 : p <= 7; }
// phases: the scheduler does not carry work over the points between the x and y terms (fewer registers;
// FP64 Q5 33^3 43.7 / 40.0, Q7 40^3 193 / 169, but Q3 80^3 177 / 191, Q4 64^3 196 / 204, Q8 2^3 9.0 / 10.4).
constexpr bool dg_phases(int p, bool fp64) { return fp64 && p >= 5 && p <= 7; }
template <int P, typename Real>
__device__ __forceinline__ void phase_end() {
  if constexpr (dg_phases(P, sizeof(Real) == 8)) __builtin_amdgcn_sched_barrier(0);
}

// What bounds it: LDS (95 accesses per lane at degree 4), vector arithmetic and the L1's line accesses at
// similar shares, so the waves in flight decide.  Every global line (dg_early: of the row segment's ends
// too) is asked for before the first barrier and reduced to the end value and derivative that are needed
// of it as it arrives.  The last contraction is along z, where a lane's stores are contiguous across
// lanes.  Line after line per direction and the last contraction along x -> this: FP64 Q4 64^3 231 -> 196 us,
// Q5 16^3 9.6 -> 10.2, Q6 14^3 11.3 -> 12.6 and 46^3 273 -> 234, Q7 40^3 246 -> 169, Q8 36^3 322 -> 224; FP32 Q3 80^3
// 93 -> 81, Q8 36^3 124 -> 110.  EPI is an instance of its own: as a branch it cost the plain operator 5 % (Q5
// to Q8).
template <int P, typename Real, bool EPI>
__global__ __launch_bounds__(DgCell<P>::THREADS) void dg_kron_kernel(const Real* __restrict__ src, int n, int slab_planes, Real h,
                                                                     Real sigma, DgKron<P, Real> kt, DgEpilogue<Real> ep) {
  using C = DgCell<P>;
  constexpr int N1 = C::N1, T = C::T, NQ = C::NQ, CPW = C::CPW;
  constexpr int R = N1 | 1;  // row stride in LDS
  __shared__ Real lds[2 * CPW * R * T];
  const int tid = threadIdx.x;
  const int lc = tid / T, e = tid - lc * T;
  const int e0 = e % N1, e1 = e / N1;
  // A workgroup takes CPW consecutive cells of one x-row of cells.  Its place in the launch order
  // (XCD-contiguous: block b runs on XCD b % 8 and takes the (b / 8)-th item of that XCD's
  // contiguous share) walks slabs of slab_planes z-planes (n/8 rounded up: about one slab per
  // XCD): within a slab z fastest, then the row segments along x, then y.  The z- and
  // x-neighbours' lines are then read a few workgroups after they were fetched, the
  // y-neighbours' one slab-row later, from the XCD's L2; only the lines across a slab boundary
  // come from HBM again.
  const int64_t G = gridDim.x, q8 = G / 8, r8 = G % 8;
  const int64_t x8 = blockIdx.x % 8, i8 = blockIdx.x / 8;
  const int64_t blk = (x8 < r8 ? x8 * (q8 + 1) : r8 * (q8 + 1) + (x8 - r8) * q8) + i8;
  const int nxb = (n + CPW - 1) / CPW;                 // row segments per x-row
  const int64_t slab = (int64_t)slab_planes * n * nxb;  // workgroups per full slab
  const int kb = (int)(blk / slab);
  const int64_t rs = blk - kb * slab;
  const int tz = min(slab_planes, n - kb * slab_planes);  // planes of this slab (the last may be thinner)
  const int jrow = (int)(rs / ((int64_t)nxb * tz));
  const int r2 = (int)(rs - (int64_t)jrow * nxb * tz);
  const int xb = r2 / tz;
  const int kz = kb * slab_planes + (r2 - xb * tz);
  const int i0 = xb * CPW;
  const int cnt = min(CPW, n - i0);                    // cells of this row segment
  const int64_t nn = (int64_t)n * n;
  const int64_t cell0 = i0 + (int64_t)n * jrow + nn * kz;
  const bool live = lc < cnt;
  const int64_t K = live ? cell0 + lc : cell0;
  const int64_t base = K * NQ;
  const Real ih = (Real)1 / h, h2 = h * h;
  // two arrays of this cell, node (a, b, c) at a + R b + R N1 c (R odd: line starts spread over the banks)
  Real* W0 = lds + lc * (R * T);
  Real* W1 = W0 + CPW * (R * T);
  const int ox = R * e, oy = e0 + R * N1 * e1, oz = e0 + R * e1;  // this lane's lines along x, y and z
  constexpr int SY = R, SZ = R * N1;
  // Every line that comes from global memory is asked for before the first barrier: the own z-line and
  // the z-neighbours' (contiguous across lanes), the y-neighbours', and the x-neighbours' at the row
  // segment's ends.  The own cells' x- and y-lines are read back from LDS.
  constexpr int B = (int)sizeof(Real);
  const bool hasLo[3] = {i0 + lc > 0, jrow > 0, kz > 0}, hasHi[3] = {i0 + lc < n - 1, jrow < n - 1, kz < n - 1};
  const int64_t first = cell0 * NQ, ny = (int64_t)n * NQ, nz = nn * NQ;
  const int vz = live ? (lc * NQ + e) * B : kNoAccess, vy = live ? (lc * NQ + e0 + T * e1) * B : kNoAccess;
  auto end = [&](auto upper, int64_t shift, bool there, int v, int stride) {
    const auto buf = node_buffer(src + (there ? first + shift : first), there ? kBufferRange : 0);
    return dg_end<N1, decltype(upper)::value, Real>(kt, [&](int a) {
      Real x;
      node_load(buf, v + stride * a, 0, x);
      return x;
    });
  };
  Real u[N1];
  const auto own = node_buffer(src + first);
#pragma unroll
  for (int c = 0; c < N1; ++c) node_load(own, vz + T * B * c, 0, u[c]);
  const auto zLo = end(std::false_type{}, -nz, hasLo[2], vz, T * B), zHi = end(std::true_type{}, nz, hasHi[2], vz, T * B);
  const auto yLo = end(std::false_type{}, -ny, hasLo[1], vy, N1 * B), yHi = end(std::true_type{}, ny, hasHi[1], vy, N1 * B);
  constexpr bool EARLY = dg_early(P, sizeof(Real) == 8);
  DgEnd<Real> xLo, xHi;
  if constexpr (EARLY) {
    const int vx = live ? (lc * NQ + N1 * e) * B : kNoAccess;
    xLo = end(std::false_type{}, -(int64_t)NQ, i0 > 0, lc == 0 ? vx : kNoAccess, B);
    xHi = end(std::true_type{}, NQ, i0 + cnt < n, lc == cnt - 1 ? vx : kNoAccess, B);
  }
#pragma unroll
  for (int c = 0; c < N1; ++c) W1[oz + SZ * c] = u[c];
  Real wz[N1];
  dg_line_terms<N1>(u, zLo, zHi, hasLo[2], hasHi[2], h, ih, h2, sigma, kt, wz);
  __syncthreads();
  const int64_t gx = base + N1 * e;
  const bool inLo = lc > 0, inHi = lc + 1 < cnt;  // the x-neighbour is in the row segment
  const auto segLo = dg_end<N1, false, Real>(kt, [&](int a) {
    if constexpr (EARLY) return W1[inLo ? ox + a - R * T : ox];
    return inLo ? W1[ox + a - R * T] : live && hasLo[0] ? src[gx - NQ + a] : (Real)0;
  });
  const auto segHi = dg_end<N1, true, Real>(kt, [&](int a) {
    if constexpr (EARLY) return W1[inHi ? ox + a + R * T : ox];
    return inHi ? W1[ox + a + R * T] : live && hasHi[0] ? src[gx + NQ + a] : (Real)0;
  });
  if (!EARLY || inLo) xLo = segLo;
  if (!EARLY || inHi) xHi = segHi;
  phase_end<P, Real>();
  {
    Real w[N1];
#pragma unroll
    for (int a = 0; a < N1; ++a) u[a] = W1[ox + a];
    dg_line_terms<N1>(u, xLo, xHi, hasLo[0], hasHi[0], h, ih, h2, sigma, kt, w);
#pragma unroll
    for (int a = 0; a < N1; ++a) W0[ox + a] = w[a];
  }
  phase_end<P, Real>();
  Real wy[N1];
#pragma unroll
  for (int b = 0; b < N1; ++b) u[b] = W1[oy + SY * b];
  dg_line_terms<N1>(u, yLo, yHi, hasLo[1], hasHi[1], h, ih, h2, sigma, kt, wy);
  __syncthreads();
  // A u = M_z (M_y w_x + M_x w_y) + M_x M_y w_z: w_y replaces the copy of the source, then w_z replaces w_y
#pragma unroll
  for (int b = 0; b < N1; ++b) W1[oy + SY * b] = wy[b];
  {  // y-lines: W0 <- M_y w_x
    Real r[N1];
#pragma unroll
    for (int b = 0; b < N1; ++b) u[b] = W0[oy + SY * b];
    eo_apply<N1, 1, false>(kt.M, u, r);
#pragma unroll
    for (int b = 0; b < N1; ++b) W0[oy + SY * b] = r[b];
  }
  __syncthreads();
  {  // x-lines: W0 <- W0 + M_x w_y
    Real r[N1];
#pragma unroll
    for (int a = 0; a < N1; ++a) u[a] = W1[ox + a];
    eo_apply<N1, 1, false>(kt.M, u, r);
#pragma unroll
    for (int a = 0; a < N1; ++a) W0[ox + a] += r[a];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < N1; ++c) W1[oz + SZ * c] = wz[c];
  Real y[N1];  // z-line of the result: M_z W0 first
  {
#pragma unroll
    for (int c = 0; c < N1; ++c) u[c] = W0[oz + SZ * c];
    eo_apply<N1, 1, false>(kt.M, u, y);
  }
  __syncthreads();
  {  // x-lines: W1 <- M_x w_z
    Real r[N1];
#pragma unroll
    for (int a = 0; a < N1; ++a) u[a] = W1[ox + a];
    eo_apply<N1, 1, false>(kt.M, u, r);
#pragma unroll
    for (int a = 0; a < N1; ++a) W1[ox + a] = r[a];
  }
  __syncthreads();
  {  // y-lines: W1 <- M_y W1
    Real r[N1];
#pragma unroll
    for (int b = 0; b < N1; ++b) u[b] = W1[oy + SY * b];
    eo_apply<N1, 1, false>(kt.M, u, r);
#pragma unroll
    for (int b = 0; b < N1; ++b) W1[oy + SY * b] = r[b];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < N1; ++c) y[c] += W1[oz + SZ * c];
  if constexpr (!EPI) {
    if (!live) return;
#pragma unroll
    for (int c = 0; c < N1; ++c) ep.dst[base + e + T * c] = y[c];
    return;
  }
  // through LDS in node order, so the accesses are contiguous over the workgroup's cells
#pragma unroll
  for (int c = 0; c < N1; ++c) W1[oz + SZ * c] = y[c];
  __syncthreads();
  const Real* v = lds + CPW * R * T;
  const int limit = cnt * NQ;
  for (int i = tid; i < limit; i += C::THREADS) {
    const Real yi = v[R == N1 ? i : i / N1 * R + i % N1];
    const int64_t gi = first + i;
    if (ep.mode == kChebStep) {
      const Real rv = ep.r[gi] - yi;
      const Real dv = ep.c1 * src[gi] + ep.c2 * ep.dinv[gi] * rv;
      ep.r[gi] = rv;
      ep.dnew[gi] = dv;
      ep.x[gi] += dv;
    } else {
      ep.r[gi] = ep.b[gi] - yi;
    }
  }
}

struct DgApplyArgs {
  int mode;
  void* dst;
  const void* b;
  const void* dinv;
  void* x;
  void* r;
  void* dnew;
  double c1, c2;
};

template <int P, typename Real>
hipError_t dg_apply_pr(int n, const Real* src, const DgEpilogue<Real>& ep, hipStream_t st) {
  using C = DgCell<P>;
  static const DgKron<P, Real> kt = make_dg_kron<P, Real>();
  const Real h = (Real)(1.0 / n);
  const Real sigma = (Real)(2.0 * (P + 1) * (P + 1) * n);
  const int64_t g = (int64_t)((n + C::CPW - 1) / C::CPW) * n * n;  // row segments of CPW cells
  if (g > 0x7fffffff) return hipErrorInvalidValue;
  const int slab_planes = (n + 7) / 8;
  if (ep.mode == kStore)
    dg_kron_kernel<P, Real, false><<<(unsigned)g, C::THREADS, 0, st>>>(src, n, slab_planes, h, sigma, kt, ep);
  else
    dg_kron_kernel<P, Real, true><<<(unsigned)g, C::THREADS, 0, st>>>(src, n, slab_planes, h, sigma, kt, ep);
  return hipGetLastError();
}

template <int P>
hipError_t dg_apply_p(int n, int precision, const void* src, const DgApplyArgs& a, hipStream_t st) {
  if (precision == MFQ_FP64) {
    const DgEpilogue<double> ep{a.mode, (double*)a.dst, (const double*)a.b, (const double*)a.dinv, (double*)a.x,
                                (double*)a.r, (double*)a.dnew, a.c1, a.c2};
    return dg_apply_pr<P, double>(n, (const double*)src, ep, st);
  }
  const DgEpilogue<float> ep{a.mode, (float*)a.dst, (const float*)a.b, (const float*)a.dinv, (float*)a.x,
                             (float*)a.r, (float*)a.dnew, (float)a.c1, (float)a.c2};
  return dg_apply_pr<P, float>(n, (const float*)src, ep, st);
}

hipError_t dg_apply(int p, int n, int precision, const void* src, const DgApplyArgs& a, hipStream_t st) {
  switch (p) {
    case 1: return dg_apply_p<1>(n, precision, src, a, st);
    case 2: return dg_apply_p<2>(n, precision, src, a, st);
    case 3: return dg_apply_p<3>(n, precision, src, a, st);
    case 4: return dg_apply_p<4>(n, precision, src, a, st);
    case 5: return dg_apply_p<5>(n, precision, src, a, st);
    case 6: return dg_apply_p<6>(n, precision, src, a, st);
    case 7: return dg_apply_p<7>(n, precision, src, a, st);
    case 8: return dg_apply_p<8>(n, precision, src, a, st);
    default: return hipErrorInvalidValue;
  }
}

// Jacobi diagonal of the DG-SIPG matrix in closed form.  With m_a = sum_q w_q S_qa^2 and
// k_a = sum_q w_q D_qa^2 (1D Gauss sums), the cell part of DoF (a,b,c) is
// h (k_a m_b m_c + m_a k_b m_c + m_a m_b k_c); a face of normal d adds, at the cell's face-layer
// nodes only (the trace of every other basis function vanishes on the GLL end points),
// h^2 m_a1 m_a2 (sigma + c l'_end(end) / h) with c = -1 for the upper face and +1 for the lower one
// of an interior face (the mean halves the two cross terms), doubled on boundary faces.
struct DgDiag1D {
  double m[kMaxDegree + 1];
  double k[kMaxDegree + 1];
  double dp1;  // l_p'(1)
  double d00;  // l_0'(0)
};

template <typename Real>
__global__ __launch_bounds__(256) void dg_diag_kernel(Real* __restrict__ diag, int p, int n, DgDiag1D t) {
  const int N1 = p + 1;
  const int64_t nloc = (int64_t)N1 * N1 * N1;
  const int64_t N = (int64_t)n * n * n * nloc;
  const double h = 1.0 / n, sigma = 2.0 * N1 * N1 * n;
  for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < N; g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t K = g / nloc;
    const int i = (int)(g - K * nloc);
    const int ai[3] = {i % N1, (i / N1) % N1, i / (N1 * N1)};
    const int64_t ck[3] = {K % n, (K / n) % n, K / ((int64_t)n * n)};
    double v = h * (t.k[ai[0]] * t.m[ai[1]] * t.m[ai[2]] + t.m[ai[0]] * t.k[ai[1]] * t.m[ai[2]] +
                    t.m[ai[0]] * t.m[ai[1]] * t.k[ai[2]]);
    for (int d = 0; d < 3; ++d) {
      const int t1 = d == 0 ? 1 : 0, t2 = d == 2 ? 1 : 2;
      const double mm = h * h * t.m[ai[t1]] * t.m[ai[t2]];
      if (ai[d] == 0) v += mm * (sigma + (ck[d] == 0 ? 2.0 : 1.0) * t.d00 / h);
      if (ai[d] == p) v += mm * (sigma - (ck[d] == n - 1 ? 2.0 : 1.0) * t.dp1 / h);
    }
    diag[g] = (Real)v;
  }
}

// Continuous Q_p (lattice of (pn+1)^3 nodes, Dirichlet nodes zero) <-> DG on the same mesh and
// nodes.  Prolongation copies each lattice node into every cell that holds it; restriction (its
// transpose) sums, per free lattice node, the entries of the cells that hold it in a fixed order.
// The switch kernels are HBM bound once their index arithmetic is: degree known at compile time and 32-bit
// indices (a DG space has less than 2^31 entries; 64-bit divisions by run-time sizes took as long as the
// accesses).  ADD: dg += E cg.
// Q4 80^3 FP32: E 265 us and the addition after it 76, now 196 together; E^T 230 -> 208.
template <int P, typename Real, bool ADD>
__global__ __launch_bounds__(256) void dg_from_cg_kernel(const Real* __restrict__ cg, Real* __restrict__ dg, int n) {
  constexpr unsigned N1 = P + 1, NL = N1 * N1 * N1;
  const unsigned nc = (unsigned)n, L1 = P * nc + 1, N = nc * nc * nc * NL, step = gridDim.x * 256;
  for (unsigned g = blockIdx.x * 256 + threadIdx.x; g < N; g += step) {
    const unsigned K = g / NL, row = K / nc, plane = row / nc;
    const unsigned i = g - K * NL;
    const unsigned I = P * (K - row * nc) + i % N1, J = P * (row - plane * nc) + i / N1 % N1, L = P * plane + i / (N1 * N1);
    const Real v = cg[I + L1 * (J + L1 * L)];
    dg[g] = ADD ? dg[g] + v : v;
  }
}

// per node the sum of its cell copies, lower cell first in every direction; zero on the boundary
template <int P, typename Real>
__global__ __launch_bounds__(256) void cg_from_dg_kernel(const Real* __restrict__ dg, Real* __restrict__ cg, int n) {
  constexpr unsigned N1 = P + 1, NL = N1 * N1 * N1;
  const unsigned nc = (unsigned)n, pn = P * nc, L1 = pn + 1, M = L1 * L1 * L1, step = gridDim.x * 256;
  for (unsigned g = blockIdx.x * 256 + threadIdx.x; g < M; g += step) {
    const unsigned row = g / L1, plane = row / L1;
    const unsigned X[3] = {g - row * L1, row - plane * L1, plane};
    if (X[0] == 0 || X[0] == pn || X[1] == 0 || X[1] == pn || X[2] == 0 || X[2] == pn) {
      cg[g] = (Real)0;
      continue;
    }
    // per direction the first cell that holds the node, the node's place there, and whether the next
    // cell holds it too (a cell vertex)
    unsigned c[3], a[3], two[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      c[d] = X[d] / P;
      a[d] = X[d] - P * c[d];
      two[d] = a[d] == 0;
      if (two[d]) {
        c[d] -= 1;
        a[d] = P;
      }
    }
    Real s = 0;
    for (unsigned kz = 0; kz <= two[2]; ++kz)
      for (unsigned ky = 0; ky <= two[1]; ++ky)
        for (unsigned kx = 0; kx <= two[0]; ++kx) {
          const unsigned K = c[0] + kx + nc * (c[1] + ky + nc * (c[2] + kz));
          s += dg[K * NL + (kx ? 0 : a[0]) + N1 * ((ky ? 0 : a[1]) + N1 * (kz ? 0 : a[2]))];
        }
    cg[g] = s;
  }
}

int dg_grid(int64_t work) {
  int64_t g = (work + 255) / 256;
  return (int)(g > 65536 ? 65536 : g < 1 ? 1 : g);
}

}  // namespace

hipError_t launch_dg_vmult(int p, int n, int precision, const void* src, void* dst, hipStream_t st) {
  DgApplyArgs a{};
  a.mode = kStore;
  a.dst = dst;
  return dg_apply(p, n, precision, src, a, st);
}

hipError_t launch_dg_cheb_step(int p, int n, int precision, const void* d, const void* dinv, void* x, void* r,
                               void* dnew, double c1, double c2, hipStream_t st) {
  DgApplyArgs a{};
  a.mode = kChebStep;
  a.dinv = dinv;
  a.x = x;
  a.r = r;
  a.dnew = dnew;
  a.c1 = c1;
  a.c2 = c2;
  return dg_apply(p, n, precision, d, a, st);
}

hipError_t launch_dg_residual(int p, int n, int precision, const void* b, const void* x, void* r, hipStream_t st) {
  DgApplyArgs a{};
  a.mode = kResidual;
  a.b = b;
  a.r = r;
  return dg_apply(p, n, precision, x, a, st);
}

hipError_t launch_dg_diagonal(int p, int n, int precision, void* diag, hipStream_t st) {
  const Tables1D& tb = tables(p);
  DgDiag1D t{};
  for (int a = 0; a <= p; ++a) {
    double m = 0, k = 0;
    for (int q = 0; q <= p; ++q) {
      m += tb.omega[q] * tb.S[q * (p + 1) + a] * tb.S[q * (p + 1) + a];
      k += tb.omega[q] * tb.D[q * (p + 1) + a] * tb.D[q * (p + 1) + a];
    }
    t.m[a] = m;
    t.k[a] = k;
  }
  t.dp1 = lagrange_derivative(tb.xi, p, 1.0);
  t.d00 = lagrange_derivative(tb.xi, 0, 0.0);
  const int64_t N = (int64_t)n * n * n * (p + 1) * (p + 1) * (p + 1);
  if (precision == MFQ_FP64)
    dg_diag_kernel<double><<<dg_grid(N), 256, 0, st>>>((double*)diag, p, n, t);
  else
    dg_diag_kernel<float><<<dg_grid(N), 256, 0, st>>>((float*)diag, p, n, t);
  return hipGetLastError();
}

namespace {
template <int P, typename Real>
void dg_transfer_pr(int n, DgSwitch op, const void* in, void* out, hipStream_t st) {
  const int64_t N = (int64_t)n * n * n * (P + 1) * (P + 1) * (P + 1), L1 = (int64_t)P * n + 1;
  if (op == kDgFromCg)
    dg_from_cg_kernel<P, Real, false><<<dg_grid(N), 256, 0, st>>>((const Real*)in, (Real*)out, n);
  else if (op == kDgAddFromCg)
    dg_from_cg_kernel<P, Real, true><<<dg_grid(N), 256, 0, st>>>((const Real*)in, (Real*)out, n);
  else
    cg_from_dg_kernel<P, Real><<<dg_grid(L1 * L1 * L1), 256, 0, st>>>((const Real*)in, (Real*)out, n);
}
template <int P>
hipError_t dg_transfer_p(int n, int precision, DgSwitch op, const void* in, void* out, hipStream_t st) {
  if (precision == MFQ_FP64)
    dg_transfer_pr<P, double>(n, op, in, out, st);
  else
    dg_transfer_pr<P, float>(n, op, in, out, st);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_dg_transfer(int p, int n, int precision, DgSwitch op, const void* in, void* out, hipStream_t st) {
  switch (p) {
    case 1: return dg_transfer_p<1>(n, precision, op, in, out, st);
    case 2: return dg_transfer_p<2>(n, precision, op, in, out, st);
    case 3: return dg_transfer_p<3>(n, precision, op, in, out, st);
    case 4: return dg_transfer_p<4>(n, precision, op, in, out, st);
    case 5: return dg_transfer_p<5>(n, precision, op, in, out, st);
    case 6: return dg_transfer_p<6>(n, precision, op, in, out, st);
    case 7: return dg_transfer_p<7>(n, precision, op, in, out, st);
    case 8: return dg_transfer_p<8>(n, precision, op, in, out, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mfq
