// Occupied-virtual rotation of an SCC basis (systems of 33 to 256 AOs).
//
// The density of a gapped closed-shell system depends on the span of its
// occupied orbitals only.  Once an eigensolve has left the basis C nearly
// canonical, an SCC iteration need not diagonalise C^T F C again: the
// couplings A_vo = C_v^T F C_o between virtual and occupied orbitals give the
// rotation X = -A_vo / (eps_v - eps_o) to first order, the couplings inside
// each class change no density, and the next iteration's A_vo carries what
// this one left.  The fixed point, A_vo = 0, is exact whatever the
// denominators.  The rotation K = [[0, -X^T], [X, 0]] is applied as
//     U = 1 + K + K^2/2 + K^3/8 - K^5/128,
// whose even part 1 + K^2/2 fixes the odd part by U^T U = 1 (the square root
// of K^2 + K^4/4, as a series); it is cut where |K| makes the next term
// vanish in FP64, so C stays S-orthonormal to rounding without a
// normalisation.
//
// An iteration by this route is three contractions on the FP64 matrix cores
// (C_o F, C_v (C_o F)^T and the rows' rotation, about 40 MFLOP for a pentacene
// dimer of 232 AOs) in place of the congruence product, the Jacobi sweeps and
// the rotation of the eigenvector rows (150 MFLOP, most of it on the vector
// units).
#include <hip/hip_runtime.h>

#include "fx_device.hpp"
#include "fx_kernels.hpp"

namespace fx {

typedef double v4d __attribute__((ext_vector_type(4)));

namespace {
// position of row r of a 16-row chunk in LDS when a lane's four consecutive
// k values feed four successive matrix instructions: instruction m then reads
// the four consecutive positions 4 m .. 4 m + 3
__device__ inline int perm16(int r) { return (r & ~15) | ((r & 3) << 2) | ((r >> 2) & 3); }
}  // namespace

// X = -A_vo / (eps_v - eps_o) of the listed systems in rotation mode, into
// Xpool (mat offsets; nvp x nop row-major, both dimensions rounded up to 16
// and zero there).  A work-group of eight waves takes 32 occupied orbitals:
// T = (C_o F)^T first (wave = 16 AO columns; F from L2, the orbitals staged in
// LDS), T then takes the orbitals' place in LDS and A_vo = C_v T follows (16
// virtual x 16 occupied blocks dealt to the waves), so the intermediate never
// leaves the CU.  Both loops are bound by the FP64 matrix instructions (64
// cycles each for 512 operand bytes).  The squared norm of the work-group's
// part of X goes to xpart[16 system + tile].
__global__ void __launch_bounds__(64 * OV_WAVES)
    k_ov_grad(DevBatch bt, const int* list, int nl, int tiles_per_sys, double* __restrict__ Xpool, double* xpart) {
  extern __shared__ double ov_lds[];
  int sl, tile;
  xcd_slot_tile(blockIdx.x, tiles_per_sys, sl, tile);
  if (sl >= nl) return;
  const int si = list[sl];
  if (bt.status[si] != 0 || bt.mode[si] != 1) return;
  const SysDesc d = bt.desc[si];
  const int n = d.nao, no = bt.ov_no[si], nv = n - no;
  const int o0 = tile * OV_ROWS;
  if (o0 >= no) return;
  const int np = (n + 15) & ~15, nop = (no + 15) & ~15, nvp = (nv + 15) & ~15;
  const int nrb = min(OV_ROWS, nop - o0) >> 4;  // 16-orbital blocks of this tile: 1 or 2
  const double* __restrict__ Ct = bt.Ct + d.mat_off;
  const double* __restrict__ F = bt.F + d.mat_off;
  const double* eps = bt.eps + d.ao_off;
  const int* ox = bt.ov_idx + d.ao_off;
  const int* vx = ox + no;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, g = lane >> 4;
  double* B0 = ov_lds;            // [np][16], first 16 orbitals
  double* B1 = ov_lds + np * 16;  // second 16
  // the orbitals, transposed: [k][orbital], zero past n and past no
  for (int u = wave; u < nrb * (np >> 4); u += OV_WAVES) {
    const int rb = u >= (np >> 4) ? 1 : 0, c = u - rb * (np >> 4);
    const int o = o0 + 16 * rb + i, k = 16 * c + 4 * g;
    const double* row = Ct + (long long)(o < no ? ox[o] : 0) * n;
    double* dst = (rb ? B1 : B0) + k * 16 + i;
#pragma unroll
    for (int m = 0; m < 4; ++m) dst[16 * m] = (o < no && k + m < n) ? row[k + m] : 0.0;
  }
  __syncthreads();
  // T[mu][o] = sum_k F[k][mu] C_o[k]; F is symmetric, rows past n are read
  // clamped (their factors in LDS are zero)
  constexpr int RND = OV_MAXN / 16 / OV_WAVES;
  v4d acc[RND][2];
#pragma unroll
  for (int r = 0; r < RND; ++r) {
    acc[r][0] = (v4d){0.0, 0.0, 0.0, 0.0};
    acc[r][1] = (v4d){0.0, 0.0, 0.0, 0.0};
    const int mu0 = 16 * (wave + OV_WAVES * r);
    if (mu0 >= n) continue;
    const double* Fc = F + min(mu0 + i, n - 1);
    double a[4], an[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) a[m] = Fc[(long long)min(4 * m + g, n - 1) * n];
    for (int k0 = 0; k0 < np; k0 += 16) {
      if (k0 + 16 < np)
#pragma unroll
        for (int m = 0; m < 4; ++m) an[m] = Fc[(long long)min(k0 + 16 + 4 * m + g, n - 1) * n];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int row = (k0 + 4 * m + g) * 16 + i;
        acc[r][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m], B0[row], acc[r][0], 0, 0, 0);
        if (nrb > 1) acc[r][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m], B1[row], acc[r][1], 0, 0, 0);
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) a[m] = an[m];
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RND; ++r) {
    const int mu0 = 16 * (wave + OV_WAVES * r);
    if (mu0 >= n) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      // element (row g + 4 q, column i), in the permuted row order
      const bool in = mu0 + g + 4 * q < n;
      const int at = (mu0 + perm16(g + 4 * q)) * 16 + i;
      B0[at] = in ? acc[r][0][q] : 0.0;
      if (nrb > 1) B1[at] = in ? acc[r][1][q] : 0.0;
    }
  }
  __syncthreads();
  double* X = Xpool + d.mat_off;
  double xs = 0.0;
  const int nunit = (nvp >> 4) * nrb;
  for (int u = wave; u < nunit; u += OV_WAVES) {
    const int vb = nrb > 1 ? u >> 1 : u, rb = nrb > 1 ? u & 1 : 0;
    const double* Bt = rb ? B1 : B0;
    const int v = 16 * vb + i;
    const double* row = Ct + (long long)vx[min(v, nv - 1)] * n;
    v4d c = (v4d){0.0, 0.0, 0.0, 0.0};
    double a[8], an[8];
    auto fetch = [&](double* t, int k0) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int m = 0; m < 4; ++m) t[4 * h + m] = row[min(k0 + 16 * h + 4 * g + m, n - 1)];
    };
    fetch(a, 0);
    for (int k0 = 0; k0 < np; k0 += 32) {
      if (k0 + 32 < np) fetch(an, k0 + 32);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (k0 + 16 * h < np)
#pragma unroll
          for (int m = 0; m < 4; ++m)
            c = __builtin_amdgcn_mfma_f64_16x16x4f64(a[4 * h + m], Bt[(k0 + 16 * h + 4 * m + g) * 16 + i], c, 0, 0, 0);
      }
#pragma unroll
      for (int m = 0; m < 8; ++m) a[m] = an[m];
    }
    const int o = o0 + 16 * rb + i;
    const double eo = o < no ? eps[ox[o]] : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int vr = 16 * vb + g + 4 * q;
      double x = 0.0;
      if (vr < nv && o < no) x = -c[q] / (eps[vx[vr]] - eo);
      X[vr * nop + o] = x;
      xs = fma(x, x, xs);
    }
  }
  xs = wave_sum_f64(xs);
  __syncthreads();  // the last reads of T
  if (lane == 0) ov_lds[wave] = xs;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < OV_WAVES; ++w) s += ov_lds[w];
    xpart[16 * si + tile] = s;
  }
}

// Rows of C^T (in place) times U for the listed systems in rotation mode.  A
// work-group of eight waves takes 16 CB columns: the rows live in LDS by class
// (occupied first, then virtual, each padded to 16 with zeros) and the wave's
// own 16-row blocks in registers; each product with K is two blocks of
// X Z_o and X^T Z_v per wave with X from L2 (shared by the system's tiles on
// one XCD), so the series costs no pass over HBM beyond C^T once in and out.
// CB is the launch's choice (2 where the batch fills the chip, else 1: more
// work-groups per system); the sums are the same.
template <int CB>
__global__ void __launch_bounds__(64 * OV_WAVES)
    k_ov_apply(DevBatch bt, const int* list, int nl, int tiles_per_sys, const double* __restrict__ Xpool,
               const double* xpart) {
  extern __shared__ double ov_lds[];
  int sl, tile;
  xcd_slot_tile(blockIdx.x, tiles_per_sys, sl, tile);
  if (sl >= nl) return;
  const int si = list[sl];
  if (bt.status[si] != 0 || bt.mode[si] != 1) return;
  const SysDesc d = bt.desc[si];
  const int n = d.nao, no = bt.ov_no[si], nv = n - no;
  const int c0 = tile * 16 * CB;
  if (c0 >= n) return;
  const int nop = (no + 15) & ~15, nvp = (nv + 15) & ~15, R = nop + nvp;
  const int nvb = nvp >> 4, nbk = R >> 4;
  double* Ct = bt.Ct + d.mat_off;
  const int* ox = bt.ov_idx + d.ao_off;
  const int* vx = ox + no;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, g = lane >> 4;
  const double* __restrict__ X = Xpool + d.mat_off;
  // |X| and, where it exceeds OV_XMAX (the couplings are too large for this
  // route; the mixer sends the system back to the eigensolver), a shorter step
  double x2 = 0.0;
  for (int t = 0; t * OV_ROWS < no; ++t) x2 += xpart[16 * si + t];
  const double xn = sqrt(x2);
  const double sc = xn > OV_XMAX ? OV_XMAX / xn : 1.0;
  const double xk = xn * sc;
  if (tile == 0 && threadIdx.x == 0) bt.xn[si] = xn;
  // terms of U kept: the first one left out is below 1e-15 (5: |K|^8 / 512,
  // 3: |K|^6 / 64, 2: |K|^4 / 4, 1: |K|^2)
  const int order = xk < 1e-8 ? 1 : xk < 2e-4 ? 2 : xk < 6e-3 ? 3 : 5;
  // block b of the wave: virtual blocks first, then occupied ones
  constexpr int U = OV_BLK;
  v4d c[U][CB], z[U][CB];
#pragma unroll
  for (int t = 0; t < U; ++t) {
    const int b = wave + OV_WAVES * t;
    if (b >= nbk) continue;
    const bool vir = b < nvb;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = g + 4 * q;
      const int k = 16 * (vir ? b : b - nvb) + r;
      const bool in = k < (vir ? nv : no);
      const double* row = Ct + (long long)(in ? (vir ? vx[k] : ox[k]) : 0) * n;
      const int at = vir ? nop + k : perm16(k);
#pragma unroll
      for (int w = 0; w < CB; ++w) {
        const int col = c0 + 16 * w + i;
        const double e = in && col < n ? row[col] : 0.0;
        c[t][w][q] = e;
        ov_lds[(w * R + at) * 16 + i] = e;
      }
    }
  }
  __syncthreads();
  for (int p = order; p >= 1; --p) {
    // Z <- C + f K Z (order 5 starts with -K/16 C alone)
    const double f = sc * (p >= 4 ? (p == 5 ? -1.0 / 16.0 : 1.0) : p == 3 ? 0.25 : p == 2 ? 0.5 : 1.0);
    const double keep = p == 5 ? 0.0 : 1.0;
#pragma unroll
    for (int t = 0; t < U; ++t) {
      const int b = wave + OV_WAVES * t;
#pragma unroll
      for (int w = 0; w < CB; ++w) z[t][w] = (v4d){0.0, 0.0, 0.0, 0.0};
      if (b >= nbk) continue;
      if (b < nvb) {
        // - X Z_o: four consecutive occupied columns of X per lane and chunk
        const double* xr = X + (long long)(16 * b + i) * nop + 4 * g;
        double a[4], an[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) a[m] = xr[m];
        for (int k0 = 0; k0 < nop; k0 += 16) {
          if (k0 + 16 < nop)
#pragma unroll
            for (int m = 0; m < 4; ++m) an[m] = xr[k0 + 16 + m];
#pragma unroll
          for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int w = 0; w < CB; ++w)
              z[t][w] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[m], ov_lds[(w * R + k0 + 4 * m + g) * 16 + i], z[t][w],
                                                             0, 0, 0);
#pragma unroll
          for (int m = 0; m < 4; ++m) a[m] = an[m];
        }
#pragma unroll
        for (int w = 0; w < CB; ++w) z[t][w] = keep * c[t][w] - f * z[t][w];
      } else {
        // X^T Z_v
        const double* xr = X + (long long)g * nop + 16 * (b - nvb) + i;
        double a[4], an[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) a[m] = xr[4 * m * nop];
        for (int k0 = 0; k0 < nvp; k0 += 16) {
          if (k0 + 16 < nvp)
#pragma unroll
            for (int m = 0; m < 4; ++m) an[m] = xr[(k0 + 16 + 4 * m) * nop];
#pragma unroll
          for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int w = 0; w < CB; ++w)
              z[t][w] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                  a[m], ov_lds[(w * R + nop + k0 + 4 * m + g) * 16 + i], z[t][w], 0, 0, 0);
#pragma unroll
          for (int m = 0; m < 4; ++m) a[m] = an[m];
        }
#pragma unroll
        for (int w = 0; w < CB; ++w) z[t][w] = keep * c[t][w] + f * z[t][w];
      }
    }
    if (p > 1) __syncthreads();  // Z has been read
#pragma unroll
    for (int t = 0; t < U; ++t) {
      const int b = wave + OV_WAVES * t;
      if (b >= nbk) continue;
      const bool vir = b < nvb;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 16 * (vir ? b : b - nvb) + g + 4 * q;
        if (p > 1) {
          const int at = vir ? nop + k : perm16(k);
#pragma unroll
          for (int w = 0; w < CB; ++w) ov_lds[(w * R + at) * 16 + i] = z[t][w][q];
        } else if (k < (vir ? nv : no)) {
          double* row = Ct + (long long)(vir ? vx[k] : ox[k]) * n;
#pragma unroll
          for (int w = 0; w < CB; ++w)
            if (c0 + 16 * w + i < n) row[c0 + 16 * w + i] = z[t][w][q];
        }
      }
    }
    if (p > 1) __syncthreads();
  }
}

template __global__ void k_ov_apply<1>(DevBatch, const int*, int, int, const double*, const double*);
template __global__ void k_ov_apply<2>(DevBatch, const int*, int, int, const double*, const double*);

// After a solve: the gap of the systems that converged in a rotation from the
// expectation values C_i^T F C_i of the orbitals whose last eigenvalue lies
// within 0.05 Eh of the gap's edges.  Where it no longer keeps the
// occupations at 0 and 2 to 1e-10, the system leaves the rotation route for
// good (mode 2) and becomes active again; *reopened counts them.
__global__ void __launch_bounds__(256) k_ov_gap(DevBatch bt, const int* list, double kT, int* reopened) {
  const int si = list[blockIdx.x];
  if (bt.status[si] != 1 || !(bt.xn[si] >= 0.0)) return;
  const SysDesc d = bt.desc[si];
  const int n = d.nao, no = bt.ov_no[si];
  const double* eps = bt.eps + d.ao_off;
  const int* ox = bt.ov_idx + d.ao_off;
  const double* F = bt.F + d.mat_off;
  const double* Ct = bt.Ct + d.mat_off;
  __shared__ double red[4];
  __shared__ double crow[MAXN];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double homo = -1e300, lumo = 1e300;
  for (int k = 0; k < n; ++k) {
    if (k < no) homo = fmax(homo, eps[ox[k]]);
    else lumo = fmin(lumo, eps[ox[k]]);
  }
  double ho = -1e300, lu = 1e300;
  for (int k = 0; k < n; ++k) {
    const int o = ox[k];
    const double e = eps[o];
    if (k < no ? e < homo - 0.05 : e > lumo + 0.05) continue;
    for (int j = threadIdx.x; j < n; j += 256) crow[j] = Ct[(long long)o * n + j];
    __syncthreads();
    double v = 0.0;
    for (int r = wave; r < n; r += 4) {
      double t = 0.0;
      for (int j = lane; j < n; j += 64) t = fma(F[(long long)r * n + j], crow[j], t);
      v = fma(crow[r], t, v);
    }
    v = wave_sum_f64(v);
    if (lane == 0) red[wave] = v;
    __syncthreads();
    v = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    if (k < no) ho = fmax(ho, v);
    else lu = fmin(lu, v);
  }
  if (threadIdx.x == 0 && !(exp(-0.5 * (lu - ho) / kT) <= 1e-10)) {
    bt.mode[si] = 2;
    bt.status[si] = 0;
    atomicAdd(reopened, 1);
  }
}

}  // namespace fx
