// Level transfer of the geometric multigrid (Sec. 3.5): interpolation between nested Q_p spaces.
//
// Isotropic refinement (Sec. 3.1) makes each coarse cell the union of 2^3 fine cells, and the
// hierarchy may also switch to a lower degree on the same mesh (as the paper's Sec. 6.1
// hierarchy switches spaces).  Prolongation evaluates the coarse function at the fine nodes inside
// each coarse cell: a tensor product of one 1D matrix P1 [nf1 x (pc+1)] applied in x, y and z; its
// first and last rows are exactly the identity (a face's fine nodes see the face's coarse nodes
// only).  Restriction is the transpose, so along a line a coarse vertex collects the two cells around
// it and the other coarse nodes one cell.
//
// What bounds them: the fine vector's traffic and, above degree 4, the LDS passes.  Time per call on
// MI355X, per-cell kernels (the restriction in eight coloured launches after a clearing one) -> this:
// Q4 32^3 -> 64^3 FP32 restriction 160 -> 44 us, prolongation 59 -> 25 (77 MB: 3.1 TB/s); Q3 32^3 81 -> 24 /
// 35 -> 15; Q8 12^3 90 -> 46 / 29 -> 16; meshes below 10^3 cells 45 -> 8 / 9 -> 8 (the host's time per call).
//
// Both stream columns of fine nodes along z through registers, coalesced along x, and do the x and y
// passes in LDS on a tile of coarse cells.  A workgroup writes every node it owns once (its cells'
// lower faces and interiors; the mesh's last cells also the upper faces): no atomics, no clearing, one
// launch, a fixed summation order that does not depend on the tiling.  The restriction of the highest degrees
// goes cell by cell where that is faster (Tile::by_cells).
#include "batch.hpp"
#include "kernels_common.hpp"

namespace mfq {

namespace {

// Tile of coarse cells of a workgroup (x, y).  A row of about 40 fine nodes keeps the columns' loads
// and stores coalesced; above degree 2 one cell in y (two for the restriction's halo) fills the
// workgroup.
template <int PC, int NF1>
struct Tile {
  static constexpr int S = NF1 - 1;  // fine nodes per coarse cell and direction
  static constexpr int OX = S <= 2 ? 16 : S <= 4 ? 8 : S <= 6 ? 6 : S <= 8 ? 4 : S <= 10 ? 3 : S <= 14 ? 2 : 1;
  static constexpr int OY = S <= 2 ? 4 : S <= 4 ? 2 : 1;
  static constexpr int BLOCK = S >= 12 ? 512 : 256;
  // The restriction's arrays leave one workgroup per CU in FP64 from degree 7 on, so it takes more lanes: a
  // column of fine nodes each at degree 8 (16^3 -> 32^3 189 -> 155 us), two at degree 7 (14^3 96 -> 79).
  template <typename Real>
  static constexpr int rblock = sizeof(Real) == 8 && S >= 14 ? (S == 14 ? 640 : 1024) : BLOCK;
  // Where the restriction goes cell by cell instead (restrict_cells), FP64 from degree 7 on: a single cell,
  // where a tile's halo is most of the work (degree 7 12.4 -> 9.7 us, degree 8 14.2 -> 11.2), and large
  // meshes, whose tiles read each fine node three to four times (degree 7 18^3 136 -> 127, 29^3 509 -> 408;
  // degree 8 16^3 155 -> 155, 25^3 568 -> 539; below, degree 7 14^3 79 -> 89, 9^3 31 -> 67).  Batched transfers
  // are FP32 and go by tiles.
  template <typename Real>
  static bool by_cells(int nc) {
    return sizeof(Real) == 8 && S >= 14 && (nc == 1 || nc >= 17);
  }
  static int tiles(int nc) { return ((nc + OX - 1) / OX) * ((nc + OY - 1) / OY); }
  // coarse layers that a workgroup of the restriction walks along z (the layer below its first one
  // is read once more): as many as leave a thousand workgroups
  static int layers(int nc) {
    const int64_t z = (int64_t)tiles(nc) * nc / 1024;
    return z < 1 ? 1 : z > 8 ? 8 : (int)z;
  }
  static int64_t blocks(int nc, bool prolongate) {
    return (int64_t)tiles(nc) * (prolongate ? nc : (nc + layers(nc) - 1) / layers(nc));
  }
};

template <int PC, int NF1, typename Real>
struct TransferTable {
  Real P[NF1 * (PC + 1)];  // P[i*(PC+1)+a]
};

// prolongation: block b of the grid (tile fastest, then layer); ADD: added to the fine vector (the
// multigrid correction) instead of stored
template <int PC, int NF1, typename Real, bool ADD>
__device__ __forceinline__ void prolongate_block(const Real* __restrict__ coarse, Real* __restrict__ fine, int nc, int bc,
                                                 const TransferTable<PC, NF1, Real>& tr, int b) {
  using T = Tile<PC, NF1>;
  constexpr int M = PC + 1, S = T::S, BLOCK = T::BLOCK;
  constexpr int CX = T::OX * PC + 1, CY = T::OY * PC + 1, FX = T::OX * S + 1, FY = T::OY * S + 1;
  __shared__ Real u[M * CY * CX];
  __shared__ Real t1[M * CY * FX];
  __shared__ Real Ps[NF1 * M];
  const int tx = (nc + T::OX - 1) / T::OX, ty = (nc + T::OY - 1) / T::OY;
  const int ic = (b % tx) * T::OX, jc = (b / tx % ty) * T::OY, kc = b / (tx * ty);
  const int E = PC * nc, Ef = S * nc;
  const int64_t N1c = E + 1, N1f = Ef + 1;
  for (int k = threadIdx.x; k < NF1 * M; k += BLOCK) Ps[k] = tr.P[k];
  for (int k = threadIdx.x; k < M * CY * CX; k += BLOCK) {
    const int I = PC * ic + k % CX, J = PC * jc + (k / CX) % CY, K = PC * kc + k / (CX * CY);
    const bool zero = I > E || J > E || (bc && (I == 0 || J == 0 || K == 0 || I == E || J == E || K == E));
    const Real v = coarse[zero ? 0 : I + N1c * (J + N1c * K)];
    u[k] = zero ? (Real)0 : v;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < M * CY * FX; k += BLOCK) {  // x
    const int x = k % FX, row = k / FX;
    const int cell = min(x / S, T::OX - 1), i = x - cell * S;
    const Real* up = u + row * CX + cell * PC;
    Real s = 0;
#pragma unroll
    for (int a = 0; a < M; ++a) s = fmad(Ps[i * M + a], up[a], s);
    t1[k] = s;
  }
  __syncthreads();
  // y and z per column of fine nodes
  for (int k = threadIdx.x; k < FX * FY; k += BLOCK) {
    const int x = k % FX, y = k / FX;
    const int I = S * ic + x, J = S * jc + y;
    // the tile's upper faces belong to the next tile, or to this one at the mesh's end
    if (I > Ef || J > Ef || (x == FX - 1 && I != Ef) || (y == FY - 1 && J != Ef)) continue;
    const int cell = min(y / S, T::OY - 1), j = y - cell * S;
    Real v[M];
#pragma unroll
    for (int c = 0; c < M; ++c) v[c] = 0;
#pragma unroll
    for (int bb = 0; bb < M; ++bb) {
      const Real p = Ps[j * M + bb];
#pragma unroll
      for (int c = 0; c < M; ++c) v[c] = fmad(p, t1[x + FX * (cell * PC + bb + CY * c)], v[c]);
    }
    const bool bxy = bc && (I == 0 || J == 0 || I == Ef || J == Ef);
    Real* out = fine + I + N1f * (J + N1f * (int64_t)(S * kc));
    const int64_t plane = N1f * N1f;
    Real x0[ADD ? S : 1];
    if constexpr (ADD) {
#pragma unroll
      for (int l = 0; l < S; ++l) x0[l] = out[l * plane];
    }
#pragma unroll
    for (int l = 0; l <= S; ++l) {
      if (l == S && kc < nc - 1) break;
      Real s = 0;
#pragma unroll
      for (int c = 0; c < M; ++c) s = fmad(tr.P[l * M + c], v[c], s);
      const bool bnd = bxy || (bc && ((l == 0 && kc == 0) || l == S));
      if constexpr (ADD) {
        if (!bnd) out[l * plane] = (l < S ? x0[l < S ? l : 0] : out[l * plane]) + s;
      } else {
        out[l * plane] = bnd ? (Real)0 : s;
      }
    }
  }
}

template <int PC, int NF1, typename Real, bool ADD>
__global__ __launch_bounds__((Tile<PC, NF1>::BLOCK)) void prolongate_kernel(const Real* __restrict__ coarse, Real* __restrict__ fine, int nc,
                                                         int bc, TransferTable<PC, NF1, Real> tr) {
  prolongate_block<PC, NF1, Real, ADD>(coarse, fine, nc, bc, tr, (int)blockIdx.x);
}

// Coarse node o of a line (counted from the first owned one, a vertex) from the fine values f with
// stride `st`, f[0] the first fine node inside the cell below: node o = PC cell + a, its vertex at
// f[S (cell + 1) - 1].  The vertex that ends the tile's `cells` owned cells is written only at the
// mesh's end, where there is no cell above it.  P in LDS.
template <int PC, int NF1, typename Real>
__device__ __forceinline__ Real restrict_node(const Real* f, int st, int o, int cells, const Real* Ps) {
  constexpr int M = PC + 1, S = NF1 - 1;
  const int cell = o / PC, a = o - cell * PC;
  const Real* v = f + (S * (cell + 1) - 1) * st;
  Real lo = 0, hi = 0;
  if (a == 0) {
#pragma unroll
    for (int i = 1; i < S; ++i) lo = fmad(Ps[i * M + PC], v[(i - S) * st], lo);
  }
  if (cell < cells) {
#pragma unroll
    for (int i = S - 1; i > 0; --i) hi = fmad(Ps[i * M + a], v[i * st], hi);
  }
  return a == 0 ? lo + hi + v[0] : hi;  // each cell's terms towards the vertex, its own (the largest) last
}

// restriction of `fine`, or with SUB of fine - minus (the multigrid residual b - A x, which is then
// never stored): block b of the grid (tile fastest, then group of layers).  The next layer's columns
// are loaded before the y and x passes of the current one where the registers allow it.
template <int PC, int NF1, typename Real, bool SUB>
__device__ __forceinline__ void restrict_block(const Real* __restrict__ fine, const Real* __restrict__ minus,
                                               Real* __restrict__ coarse, int nc, int bc,
                                               int layers, const TransferTable<PC, NF1, Real>& tr, int b) {
  using T = Tile<PC, NF1>;
  constexpr int M = PC + 1, S = T::S, BLOCK = T::template rblock<Real>;
  // fine nodes inside the cell below, the owned cells and, for the mesh's last vertex, their end
  constexpr int FX = (T::OX + 1) * S, FY = (T::OY + 1) * S;
  constexpr int WX = T::OX * PC + 1, WY = T::OY * PC + 1;
  constexpr int COLS = (FX * FY + BLOCK - 1) / BLOCK;
  __shared__ Real t1[PC * FY * FX];  // after z: [a][y][x]
  constexpr int R2 = FX | 1;         // odd: lanes of several rows read the same place of each
  __shared__ Real t2[PC * WY * R2];  // after y
  __shared__ Real Ps[NF1 * M];
  const int tx = (nc + T::OX - 1) / T::OX, ty = (nc + T::OY - 1) / T::OY;
  const int ic = (b % tx) * T::OX, jc = (b / tx % ty) * T::OY, k0 = b / (tx * ty) * layers;
  const int k1 = min(k0 + layers, nc);
  const int E = PC * nc, Ef = S * nc;
  const int64_t N1c = E + 1, N1f = Ef + 1, plane = N1f * N1f;
  const int tid = threadIdx.x;
  for (int k = tid; k < NF1 * M; k += BLOCK) Ps[k] = tr.P[k];
  auto value = [&](int64_t g) -> Real {
    if constexpr (SUB) return fine[g] - minus[g];
    return fine[g];
  };
  // the 1D matrix of the z pass: scalars, or from LDS at degree 7 in FP64, where it would be spilled lane by lane
  // and that costs more (FP64: 202 spilled scalars, 14^3 96 -> 84 us; not at degree 8, and FP32 29^3 274 -> 290)
  constexpr bool ZL = S == 14 && sizeof(Real) == 8;
  if (ZL) __syncthreads();
  auto z = [&](int k) -> Real { return ZL ? Ps[k] : tr.P[k]; };
  // this thread's columns; fine nodes outside the mesh or in Dirichlet faces count as zero
  int64_t col[COLS];
  bool on[COLS];
  Real carry[COLS];
#pragma unroll
  for (int q = 0; q < COLS; ++q) {
    const int k = tid + q * BLOCK, x = k % FX, y = k / FX;
    const int I = S * (ic - 1) + 1 + x, J = S * (jc - 1) + 1 + y;
    on[q] = k < FX * FY && I >= 0 && J >= 0 && I <= Ef && J <= Ef && !(bc && (I == 0 || J == 0 || I == Ef || J == Ef));
    col[q] = on[q] ? I + N1f * J : 0;
    carry[q] = 0;
    if (k0 > 0) {
#pragma unroll
      for (int i = 1; i < S; ++i) {
        const Real v = value(col[q] + plane * (S * (k0 - 1) + i));
        carry[q] = fmad(z(i * M + PC), on[q] ? v : (Real)0, carry[q]);
      }
    }
  }
  constexpr bool AHEAD = sizeof(Real) == 4 && COLS <= 3;
  Real f[AHEAD ? COLS : 1][S];
  // fine planes S kc .. S kc + S - 1 of column q (past the mesh's last layer its end plane alone)
  auto load = [&](int kc, int q, Real (&v)[S]) {
    const int64_t g = col[q] + plane * (int64_t)(S * kc);
#pragma unroll
    for (int i = 0; i < S; ++i)
      if (i == 0 || kc < nc) v[i] = value(g + i * plane);
  };
  auto load_all = [&](int kc) {
    if constexpr (AHEAD) {
#pragma unroll
      for (int q = 0; q < COLS; ++q) load(kc, q, f[q]);
    }
  };
  // a layer's planes a = 0..PC-1, and after the mesh's last layer its last vertex plane
  const int kend = k1 == nc ? nc + 1 : k1;
  load_all(k0);
  for (int kc = k0; kc < kend; ++kc) {
    const bool last = kc == nc;
    const int planes = last ? 1 : PC;
    __syncthreads();  // the passes of the layer before have read t1 and t2
#pragma unroll
    for (int q = 0; q < COLS; ++q) {
      const int k = tid + q * BLOCK;
      const bool bz = bc && (kc == 0 || last);
      Real(&fq)[S] = f[AHEAD ? q : 0];
      if constexpr (!AHEAD) load(kc, q, fq);
      Real out[PC];
      // (rounding: FP32 as restrict_node, but for the order of the terms where the matrix's scalars are
      // spilled and a second walk through them costs a tenth; FP64 frees registers first)
      constexpr bool DOWN = sizeof(Real) == 4 && S < 14;
      const Real end = on[q] && !bz ? fq[0] : (Real)0;
      const Real below = carry[q];
      out[0] = sizeof(Real) == 8 ? below + end : (Real)0;
      if (!last) {
#pragma unroll
        for (int a = 1; a < PC; ++a) out[a] = 0;
        carry[q] = 0;
#pragma unroll
        for (int i = 1; i < S; ++i) {
          const Real v = on[q] ? fq[i] : (Real)0;
#pragma unroll
          for (int a = DOWN; a < PC; ++a) out[a] = fmad(z(i * M + a), v, out[a]);
          carry[q] = fmad(z(i * M + PC), v, carry[q]);
        }
        if (DOWN) {
#pragma unroll
          for (int i = S - 1; i > 0; --i) out[0] = fmad(z(i * M), on[q] ? fq[i] : (Real)0, out[0]);
        }
      }
      if (sizeof(Real) == 4) out[0] = below + out[0] + end;
      if (k < FX * FY) {
        const int x = k % FX, y = k / FX;
        if (last)
          t1[x + FX * y] = out[0];
        else
#pragma unroll
          for (int a = 0; a < PC; ++a) t1[x + FX * (y + FY * a)] = out[a];
      }
    }
    if (kc + 1 < kend) load_all(kc + 1);
    __syncthreads();
    for (int k = tid; k < planes * WY * FX; k += BLOCK) {  // y
      const int x = k % FX, o = (k / FX) % WY, a = k / (FX * WY);
      t2[x + R2 * (o + WY * a)] = restrict_node<PC, NF1>(t1 + x + FX * FY * a, FX, o, T::OY, Ps);
    }
    __syncthreads();
    for (int k = tid; k < planes * WY * WX; k += BLOCK) {  // x
      const int ox = k % WX, oy = (k / WX) % WY, a = k / (WX * WY);
      const int I = PC * ic + ox, J = PC * jc + oy, K = PC * kc + a;
      if (I > E || J > E || (ox == WX - 1 && I != E) || (oy == WY - 1 && J != E)) continue;
      const bool bnd = bc && (I == 0 || J == 0 || K == 0 || I == E || J == E || K == E);
      const Real s = restrict_node<PC, NF1>(t2 + R2 * (oy + WY * a), 1, ox, T::OX, Ps);
      coarse[I + N1c * (J + N1c * K)] = bnd ? (Real)0 : s;
    }
  }
}

template <int PC, int NF1, typename Real, bool SUB>
__global__ __launch_bounds__((Tile<PC, NF1>::template rblock<Real>)) void restrict_kernel(const Real* __restrict__ fine,
                                                                        const Real* __restrict__ minus,
                                                                        Real* __restrict__ coarse, int nc, int bc, int layers, TransferTable<PC, NF1, Real> tr) {
  restrict_block<PC, NF1, Real, SUB>(fine, minus, coarse, nc, bc, layers, tr, (int)blockIdx.x);
}

// Restriction cell by cell: coarse cell b of colour `colour` by the workgroup.  Fine values are weighted by 1 /
// (number of coarse cells that hold the node), so the cells' transposes sum to P^T; cells of one colour
// (parities of the coordinates) share no coarse node and add with plain stores, colours in order, into the
// cleared coarse vector.
constexpr int kCellBlock = 512;
template <int PC, int NF1, typename Real, bool SUB>
__global__ __launch_bounds__(kCellBlock) void restrict_cells_kernel(const Real* __restrict__ fine, const Real* __restrict__ minus,
                                                                   Real* __restrict__ coarse, int nc, int bc, int colour,
                                                                   TransferTable<PC, NF1, Real> tr) {
  constexpr int M = PC + 1, S = NF1 - 1;
  __shared__ Real f[NF1 * NF1 * NF1];  // the cell's fine nodes, zero on Dirichlet nodes
  __shared__ Real t1[M * NF1 * NF1];   // after x: [l][j][a]
  __shared__ Real t2[M * M * NF1];     // after y: [l][b][a]
  __shared__ Real Ps[NF1 * M];
  const int px = colour & 1, py = (colour >> 1) & 1, pz = colour >> 2;
  const int cxn = (nc + 1 - px) / 2, cyn = (nc + 1 - py) / 2, b = (int)blockIdx.x;
  const int ic = 2 * (b % cxn) + px, jc = 2 * (b / cxn % cyn) + py, kc = 2 * (b / (cxn * cyn)) + pz;
  const int E = PC * nc, Ef = S * nc;
  const int64_t N1c = E + 1, N1f = Ef + 1;
  auto share = [&](int i, int cell) -> Real { return (i == 0 && cell > 0) || (i == S && cell < nc - 1) ? (Real)0.5 : (Real)1; };
  for (int k = threadIdx.x; k < NF1 * M; k += kCellBlock) Ps[k] = tr.P[k];
  for (int k = threadIdx.x; k < NF1 * NF1 * NF1; k += kCellBlock) {
    const int I = S * ic + k % NF1, J = S * jc + k / NF1 % NF1, K = S * kc + k / (NF1 * NF1);
    const bool zero = bc && (I == 0 || J == 0 || K == 0 || I == Ef || J == Ef || K == Ef);
    const int64_t g = I + N1f * (J + N1f * K);
    Real v = fine[g];
    if constexpr (SUB) v -= minus[g];
    f[k] = zero ? (Real)0 : v;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < M * NF1 * NF1; k += kCellBlock) {
    const int a = k % M, j = k / M % NF1, l = k / (M * NF1);
    Real s = 0;
#pragma unroll
    for (int i = 0; i < NF1; ++i) s = fmad(Ps[i * M + a] * share(i, ic), f[i + NF1 * (j + NF1 * l)], s);
    t1[k] = s * (share(j, jc) * share(l, kc));
  }
  __syncthreads();
  for (int k = threadIdx.x; k < M * M * NF1; k += kCellBlock) {
    const int a = k % M, bb = k / M % M, l = k / (M * M);
    Real s = 0;
#pragma unroll
    for (int j = 0; j < NF1; ++j) s = fmad(Ps[j * M + bb], t1[a + M * (j + NF1 * l)], s);
    t2[k] = s;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < M * M * M; k += kCellBlock) {
    const int a = k % M, bb = k / M % M, c = k / (M * M);
    Real s = 0;
#pragma unroll
    for (int l = 0; l < NF1; ++l) s = fmad(Ps[l * M + c], t2[a + M * (bb + M * l)], s);
    const int I = PC * ic + a, J = PC * jc + bb, K = PC * kc + c;
    const bool bnd = bc && (I == 0 || J == 0 || K == 0 || I == E || J == E || K == E);
    if (!bnd) coarse[I + N1c * (J + N1c * K)] += s;
  }
}

template <int PC, int NF1, typename Real, bool SUB>
hipError_t restrict_cells(const Real* fine, const Real* minus, Real* coarse, int64_t n_coarse, int nc, int bc,
                          const TransferTable<PC, NF1, Real>& tr, hipStream_t st) {
  hipError_t e = launch_fill(sizeof(Real) == 8 ? MFQ_FP64 : MFQ_FP32, coarse, n_coarse, 0.0, st);
  if (e != hipSuccess) return e;
  for (int c = 0; c < kColours; ++c) {
    const int64_t cells = (int64_t)((nc + 1 - (c & 1)) / 2) * ((nc + 1 - ((c >> 1) & 1)) / 2) * ((nc + 1 - (c >> 2)) / 2);
    if (cells == 0) continue;
    restrict_cells_kernel<PC, NF1, Real, SUB><<<(unsigned)cells, kCellBlock, 0, st>>>(fine, minus, coarse, nc, bc, c, tr);
  }
  return hipGetLastError();
}

// Batched forms (serving): workgroup b belongs to the item whose range [first, next first) holds it and
// does that item's block b - first, as the single-transfer launch does (results bitwise equal).
__device__ __forceinline__ int transfer_item(const TransferItem* __restrict__ it, int count, int64_t b) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (it[mid].first <= b) lo = mid; else hi = mid - 1;
  }
  return lo;
}

template <int PC, int NF1>
__global__ __launch_bounds__((Tile<PC, NF1>::BLOCK)) void batch_prolongate_kernel(const TransferItem* __restrict__ items, int count,
                                                               TransferTable<PC, NF1, float> tr) {
  const TransferItem& it = items[transfer_item(items, count, blockIdx.x)];
  prolongate_block<PC, NF1, float, true>((const float*)it.in, (float*)it.out, it.nc, it.bc, tr, (int)(blockIdx.x - it.first));
}

template <int PC, int NF1, bool SUB>
__global__ __launch_bounds__((Tile<PC, NF1>::BLOCK)) void batch_restrict_kernel(const TransferItem* __restrict__ items, int count,
                                                             TransferTable<PC, NF1, float> tr) {
  const TransferItem& it = items[transfer_item(items, count, blockIdx.x)];
  restrict_block<PC, NF1, float, SUB>((const float*)it.in, (const float*)it.minus, (float*)it.out, it.nc, it.bc, it.layers, tr,
                                 (int)(blockIdx.x - it.first));
}

template <int PC, int NF1, typename Real>
TransferTable<PC, NF1, Real> transfer_table(const std::vector<double>& P1) {
  TransferTable<PC, NF1, Real> tr;
  for (int k = 0; k < NF1 * (PC + 1); ++k) tr.P[k] = (Real)P1[k];
  return tr;
}

template <int PC, int NF1>
hipError_t batch_transfer_pn(bool h_transfer, bool prolongate, bool sub, const TransferItem* items, int count, int64_t blocks,
                             hipStream_t st) {
  int nf1 = 0;
  const std::vector<double> P1 = transfer_matrix_1d(PC, h_transfer ? PC : NF1 - 1, h_transfer, &nf1);
  if (nf1 != NF1) return hipErrorInvalidValue;
  const auto tr = transfer_table<PC, NF1, float>(P1);
  if (prolongate)
    batch_prolongate_kernel<PC, NF1><<<(unsigned)blocks, Tile<PC, NF1>::BLOCK, 0, st>>>(items, count, tr);
  else if (sub)
    batch_restrict_kernel<PC, NF1, true><<<(unsigned)blocks, Tile<PC, NF1>::BLOCK, 0, st>>>(items, count, tr);
  else
    batch_restrict_kernel<PC, NF1, false><<<(unsigned)blocks, Tile<PC, NF1>::BLOCK, 0, st>>>(items, count, tr);
  return hipGetLastError();
}

template <int PC, int NF1, typename Real>
hipError_t transfer_pnr(const mfq_transfer* t, TransferOp op, const Real* in, const Real* minus, Real* out,
                        hipStream_t st) {
  const auto tr = transfer_table<PC, NF1, Real>(t->P1);
  const int nc = t->coarse->mesh->n, bc = t->coarse->bc;
  using T = Tile<PC, NF1>;
  const bool up = op == kProlongate || op == kProlongateAdd;
  const unsigned grid = (unsigned)T::blocks(nc, up);
  if (op == kProlongate)
    prolongate_kernel<PC, NF1, Real, false><<<grid, T::BLOCK, 0, st>>>(in, out, nc, bc, tr);
  else if (op == kProlongateAdd)
    prolongate_kernel<PC, NF1, Real, true><<<grid, T::BLOCK, 0, st>>>(in, out, nc, bc, tr);
  else {
    constexpr int RB = T::template rblock<Real>;
    if constexpr (sizeof(Real) == 8 && T::S >= 14)
      if (T::template by_cells<Real>(nc)) {
        const int64_t n = t->coarse->n_dofs;
        return op == kRestrict ? restrict_cells<PC, NF1, Real, false>(in, nullptr, out, n, nc, bc, tr, st)
                               : restrict_cells<PC, NF1, Real, true>(in, minus, out, n, nc, bc, tr, st);
      }
    if (op == kRestrict)
      restrict_kernel<PC, NF1, Real, false><<<grid, RB, 0, st>>>(in, nullptr, out, nc, bc, T::layers(nc), tr);
    else
      restrict_kernel<PC, NF1, Real, true><<<grid, RB, 0, st>>>(in, minus, out, nc, bc, T::layers(nc), tr);
  }
  return hipGetLastError();
}

template <int PC, int NF1>
hipError_t transfer_pn(const mfq_transfer* t, int precision, TransferOp op, const void* in, const void* minus, void* out,
                       hipStream_t st) {
  if (precision == MFQ_FP64)
    return transfer_pnr<PC, NF1, double>(t, op, (const double*)in, (const double*)minus, (double*)out, st);
  return transfer_pnr<PC, NF1, float>(t, op, (const float*)in, (const float*)minus, (float*)out, st);
}

template <int PC, int NF1>
int64_t transfer_blocks_pn(int nc, bool prolongate, int* layers) {
  *layers = Tile<PC, NF1>::layers(nc);
  return Tile<PC, NF1>::blocks(nc, prolongate);
}

}  // namespace

hipError_t launch_transfer(const mfq_transfer* t, int precision, TransferOp op, const void* in, const void* minus,
                           void* out, hipStream_t st) {
  const int pc = t->coarse->p;
  if (t->h_transfer) {
    switch (pc) {
      case 1: return transfer_pn<1, 3>(t, precision, op, in, minus, out, st);
      case 2: return transfer_pn<2, 5>(t, precision, op, in, minus, out, st);
      case 3: return transfer_pn<3, 7>(t, precision, op, in, minus, out, st);
      case 4: return transfer_pn<4, 9>(t, precision, op, in, minus, out, st);
      case 5: return transfer_pn<5, 11>(t, precision, op, in, minus, out, st);
      case 6: return transfer_pn<6, 13>(t, precision, op, in, minus, out, st);
      case 7: return transfer_pn<7, 15>(t, precision, op, in, minus, out, st);
      case 8: return transfer_pn<8, 17>(t, precision, op, in, minus, out, st);
      default: return hipErrorInvalidValue;
    }
  }
  const int pf = t->fine->p;
  // degree switches of the hierarchy rule: p -> ceil(p/2)
#define MFQ_PT(a, b) \
  if (pc == a && pf == b) return transfer_pn<a, b + 1>(t, precision, op, in, minus, out, st);
  MFQ_PT(1, 2) MFQ_PT(2, 3) MFQ_PT(2, 4) MFQ_PT(3, 5) MFQ_PT(3, 6) MFQ_PT(4, 7) MFQ_PT(4, 8)
#undef MFQ_PT
  return hipErrorInvalidValue;
}

hipError_t launch_batch_transfer(int pc, int pf, bool h_transfer, bool prolongate, bool sub, const TransferItem* items, int count,
                                 int64_t blocks, hipStream_t st) {
  if (count <= 0 || blocks <= 0) return hipSuccess;
  if (h_transfer) {
    switch (pc) {
      case 1: return batch_transfer_pn<1, 3>(true, prolongate, sub, items, count, blocks, st);
      case 2: return batch_transfer_pn<2, 5>(true, prolongate, sub, items, count, blocks, st);
      case 3: return batch_transfer_pn<3, 7>(true, prolongate, sub, items, count, blocks, st);
      case 4: return batch_transfer_pn<4, 9>(true, prolongate, sub, items, count, blocks, st);
      case 5: return batch_transfer_pn<5, 11>(true, prolongate, sub, items, count, blocks, st);
      case 6: return batch_transfer_pn<6, 13>(true, prolongate, sub, items, count, blocks, st);
      case 7: return batch_transfer_pn<7, 15>(true, prolongate, sub, items, count, blocks, st);
      case 8: return batch_transfer_pn<8, 17>(true, prolongate, sub, items, count, blocks, st);
      default: return hipErrorInvalidValue;
    }
  }
#define MFQ_PT(a, b) \
  if (pc == a && pf == b) return batch_transfer_pn<a, b + 1>(false, prolongate, sub, items, count, blocks, st);
  MFQ_PT(1, 2) MFQ_PT(2, 3) MFQ_PT(2, 4) MFQ_PT(3, 5) MFQ_PT(3, 6) MFQ_PT(4, 7) MFQ_PT(4, 8)
#undef MFQ_PT
  return hipErrorInvalidValue;
}

int64_t transfer_blocks(int pc, int pf, bool h_transfer, int nc, bool prolongate, int* layers) {
  if (h_transfer) {
    switch (pc) {
      case 1: return transfer_blocks_pn<1, 3>(nc, prolongate, layers);
      case 2: return transfer_blocks_pn<2, 5>(nc, prolongate, layers);
      case 3: return transfer_blocks_pn<3, 7>(nc, prolongate, layers);
      case 4: return transfer_blocks_pn<4, 9>(nc, prolongate, layers);
      case 5: return transfer_blocks_pn<5, 11>(nc, prolongate, layers);
      case 6: return transfer_blocks_pn<6, 13>(nc, prolongate, layers);
      case 7: return transfer_blocks_pn<7, 15>(nc, prolongate, layers);
      default: return transfer_blocks_pn<8, 17>(nc, prolongate, layers);
    }
  }
#define MFQ_PT(a, b) \
  if (pc == a && pf == b) return transfer_blocks_pn<a, b + 1>(nc, prolongate, layers);
  MFQ_PT(1, 2) MFQ_PT(2, 3) MFQ_PT(2, 4) MFQ_PT(3, 5) MFQ_PT(3, 6) MFQ_PT(4, 7) MFQ_PT(4, 8)
#undef MFQ_PT
  return 0;
}

}  // namespace mfq
