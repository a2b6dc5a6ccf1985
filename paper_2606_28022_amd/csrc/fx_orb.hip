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
//     U = 1 + K + K^2/2 + K^3/8 - K^5/128 + K^7/1024,
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

#include <type_traits>

namespace fx {

typedef double v4d __attribute__((ext_vector_type(4)));

namespace {
// position of row r of a 16-row chunk in LDS when a lane's four consecutive
// k values feed four successive matrix instructions: instruction m then reads
// the four consecutive positions 4 m .. 4 m + 3
__device__ inline int perm16(int r) { return (r & ~15) | ((r & 3) << 2) | ((r >> 2) & 3); }

// the chunks 0 .. nch - 1 of a contraction: load(t, c) fetches a chunk's four
// operand values, mul(t, c) multiplies it.  Loads run D chunks ahead and, but
// for the last ones, without a condition, so that each multiplication waits
// for its own chunk only: the operands come from HBM for a system's first
// work-group, and one chunk of matrix instructions does not cover that.
template <int D, typename Load, typename Mul>
__device__ inline void chunk_pipeline(int nch, Load load, Mul mul) {
  double t[D + 1][4];
#pragma unroll
  for (int j = 0; j < D; ++j) load(t[j], min(j, nch - 1));
  int c = 0;
  for (; c + D + 1 <= nch; c += D + 1)
#pragma unroll
    for (int j = 0; j <= D; ++j) {
      load(t[(j + D) % (D + 1)], min(c + j + D, nch - 1));
      __builtin_amdgcn_sched_barrier(0);  // (the scheduler would sink the loads)
      mul(t[j], c + j);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
  for (int j = 0; j < D; ++j)
    if (c + j < nch) mul(t[j], c + j);
}
}  // namespace

// X = -A_vo / (eps_v - eps_o) of the listed systems in rotation mode, both
// dimensions rounded up to 16 with zeros, as 16 x 16 blocks [virtual][occupied]
// (mat offsets), each stored by occupied columns: element (v, o) of a block at
// 16 o + v, which is the order of the matrix instructions' operands, so that a
// block is 2 KB read in one piece by X Z_o and by X^T Z_v alike.  A work-group of eight waves takes 32 occupied orbitals:
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
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = lane & 15, g = lane >> 4;
  double* B0 = ov_lds;            // [np][16], first 16 orbitals
  double* B1 = ov_lds + np * 16;  // second 16
  // the class lists and their eigenvalues, staged once (their use in each
  // block would be two dependent memory accesses)
  __shared__ int ox[OV_MAXN];
  __shared__ double eps[OV_MAXN];
  if ((int)threadIdx.x < n) {
    const int o = bt.ov_idx[d.ao_off + threadIdx.x];
    ox[threadIdx.x] = o;
    eps[threadIdx.x] = bt.eps[d.ao_off + o];
  }
  __syncthreads();
  const int* vx = ox + no;
  // the orbitals, transposed: [k][orbital], zero past n and past no.  All of a
  // wave's loads are issued before the first is used (clamped addresses, no
  // branch): the chain of HBM accesses would otherwise be the longest part.
  {
    constexpr int UN = 2 * (OV_MAXN / 16) / OV_WAVES;
    const int nc = np >> 4, nu = nrb * nc;
    double v[UN][4];
#pragma unroll
    for (int j = 0; j < UN; ++j) {
      const int u = min(wave + OV_WAVES * j, nu - 1), rb = u >= nc ? 1 : 0;
      const int o = min(o0 + 16 * rb + i, no - 1), k = 16 * (u - rb * nc) + 4 * g;
      const double* row = Ct + ox[o] * n;
#pragma unroll
      for (int m = 0; m < 4; ++m) v[j][m] = row[min(k + m, n - 1)];
    }
#pragma unroll
    for (int j = 0; j < UN; ++j) {
      const int u = wave + OV_WAVES * j, rb = u >= nc ? 1 : 0;
      if (u >= nu) continue;
      const int k = 16 * (u - rb * nc) + 4 * g;
      double* dst = (rb ? B1 : B0) + k * 16 + i;
#pragma unroll
      for (int m = 0; m < 4; ++m) dst[16 * m] = (o0 + 16 * rb + i < no && k + m < n) ? v[j][m] : 0.0;
    }
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
    // (32-bit byte offsets from the matrix)
    const char* Fb = reinterpret_cast<const char*>(F);
    const unsigned colb = 8u * (unsigned)min(mu0 + i, n - 1), rowb = 8u * (unsigned)n;
    auto load = [&](double* t, int c) {
#pragma unroll
      for (int m = 0; m < 4; ++m)
        t[m] = *reinterpret_cast<const double*>(Fb + (colb + (unsigned)min(16 * c + 4 * m + g, n - 1) * rowb));
    };
    // (one or two orbital blocks: two code paths, so that no branch separates
    // a chunk's LDS reads from its matrix instructions)
    auto run = [&](auto two) {
      constexpr bool TWO = decltype(two)::value;
      chunk_pipeline<3>(np >> 4, load, [&](const double* t, int c) {
        const int row = (16 * c + g) * 16 + i;
        double x[4], y[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          x[m] = B0[row + 64 * m];
          y[m] = TWO ? B1[row + 64 * m] : 0.0;
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          acc[r][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[m], x[m], acc[r][0], 0, 0, 0);
          if (TWO) acc[r][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[m], y[m], acc[r][1], 0, 0, 0);
        }
      });
    };
    if (nrb > 1) run(std::true_type{});
    else run(std::false_type{});
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
  // A_vo^T: 16 occupied rows x 16 virtual columns per block
  double* X = Xpool + d.mat_off;
  double xs = 0.0;
  const int nvb = nvp >> 4, nob = nop >> 4;
  const int nunit = nvb * nrb;
  for (int u = wave; u < nunit; u += OV_WAVES) {
    const int vb = nrb > 1 ? u >> 1 : u, rb = nrb > 1 ? u & 1 : 0;
    const double* Bt = rb ? B1 : B0;
    const int v = 16 * vb + i, ov = vx[min(v, nv - 1)];
    const double ev = eps[no + min(v, nv - 1)];
    const char* Cb = reinterpret_cast<const char*>(Ct);
    const unsigned rowb = 8u * (unsigned)(ov * n);
    v4d c = (v4d){0.0, 0.0, 0.0, 0.0};
    auto load = [&](double* t, int ch) {
      // four consecutive elements of the lane's row (the last chunk clamped)
      const int k = 16 * ch + 4 * g;
      if (16 * ch + 16 <= n) {
        __builtin_memcpy(t, Cb + (rowb + 8u * (unsigned)k), 32);
      } else {
#pragma unroll
        for (int m = 0; m < 4; ++m)
          t[m] = *reinterpret_cast<const double*>(Cb + (rowb + 8u * (unsigned)min(k + m, n - 1)));
      }
    };
    auto mul = [&](const double* t, int ch) {
#pragma unroll
      for (int m = 0; m < 4; ++m)
        c = __builtin_amdgcn_mfma_f64_16x16x4f64(Bt[(16 * ch + 4 * m + g) * 16 + i], t[m], c, 0, 0, 0);
    };
    chunk_pipeline<3>(np >> 4, load, mul);
    const int ob = (o0 >> 4) + rb;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int o = 16 * ob + g + 4 * q;
      double x = 0.0;
      if (v < nv && o < no) x = -c[q] / (ev - eps[o]);
      X[((vb * nob + ob) * 4 + q) * 64 + lane] = x;
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
// (occupied first, then virtual, each padded to 16 with zeros); each product
// with K is BLK 16-row blocks of X Z_o or X^T Z_v per wave with X from L2
// (shared by the system's tiles on one XCD), so the series costs no pass over
// HBM beyond C^T once in and out.
// CB is the launch's choice (2 where the batch fills the chip, else 1: more
// work-groups per system); the sums are the same.
// BLK 16-row blocks per wave: 2 serve up to 256 padded rows.
template <int CB, int BLK>
__global__ void __launch_bounds__(64 * OV_WAVES) __attribute__((amdgpu_waves_per_eu(4)))
    k_ov_apply(DevBatch bt, const int* list, int nl, int tiles_per_sys, const double* __restrict__ Xpool,
               const double* xpart, double xmax) {
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
  const double* X = Xpool + d.mat_off;
  const int nob = nop >> 4;
  // |X| and, where it exceeds xmax (the couplings are too large for this
  // route; the mixer sends the system back to the eigensolver), a shorter step
  double x2 = 0.0;
  for (int t = 0; t * OV_ROWS < no; ++t) x2 += xpart[16 * si + t];
  const double xn = sqrt(x2);
  const double sc = xn > xmax ? xmax / xn : 1.0;
  const double xk = xn * sc;
  if (tile == 0 && threadIdx.x == 0) bt.xn[si] = xn;
  // products with K: the first term of U^T U left out stays below 1e-15 (7:
  // 3e-4 |K|^10 at the two-norm, a fraction of the Frobenius norm at hand; 5:
  // |K|^8 / 512; 3: |K|^6 / 64; 2: |K|^4 / 4; 1: |K|^2)
  const int order = xk < 1e-8 ? 1 : xk < 2e-4 ? 2 : xk < 6e-3 ? 3 : xk < 0.03 ? 5 : 7;
  // element q of the lane in block t of the wave (virtual blocks first, then
  // occupied ones): offset of its row of C^T (-1: padding), position in LDS.
  // All loads are issued before the first is used (clamped, no branch).
  int ro[BLK][4];
  v4d c[BLK][CB];
  auto lds_row = [&](int t, int q) {
    const int b = wave + OV_WAVES * t;
    return b < nvb ? nop + perm16(16 * b + g + 4 * q) : 16 * (b - nvb) + g + 4 * q;
  };
#pragma unroll
  for (int t = 0; t < BLK; ++t) {
    const int b = min(wave + OV_WAVES * t, nbk - 1);
    const bool vir = b < nvb;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = 16 * (vir ? b : b - nvb) + g + 4 * q, last = (vir ? nv : no) - 1;
      const int idx = (vir ? vx : ox)[min(k, last)];
      ro[t][q] = k <= last ? idx * n : -1;
    }
  }
#pragma unroll
  for (int t = 0; t < BLK; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int w = 0; w < CB; ++w) c[t][w][q] = Ct[max(ro[t][q], 0) + min(c0 + 16 * w + i, n - 1)];
#pragma unroll
  for (int t = 0; t < BLK; ++t) {
    if (wave + OV_WAVES * t >= nbk) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int w = 0; w < CB; ++w) {
        if (ro[t][q] < 0 || c0 + 16 * w + i >= n) c[t][w][q] = 0.0;
        ov_lds[(w * R + lds_row(t, q)) * 16 + i] = c[t][w][q];
      }
  }
  __syncthreads();
  for (int p = order; p >= 1; --p) {
    // Z <- keep C + f K Z, by Horner's rule from the highest term
    const double f = sc * (p == 1 || p == 4 || p == 6 ? 1.0 : p == 2 ? 0.5 : p == 3 ? 0.25 : p == 5 ? -1.0 / 16.0 : -0.125);
    const bool keep = p != 5 && p != 7;
    v4d z[BLK][CB];
#pragma unroll
    for (int t = 0; t < BLK; ++t) {
      const int b = wave + OV_WAVES * t;
#pragma unroll
      for (int w = 0; w < CB; ++w) z[t][w] = (v4d){0.0, 0.0, 0.0, 0.0};
      if (b >= nbk) continue;
      // virtual rows: X Z_o, instruction m takes columns 4 m + g of the chunk's
      // block; occupied rows: X^T Z_v, it takes rows 4 g + m (Z_v's rows are
      // permuted to match), a lane's four being consecutive
      const bool vir = b < nvb;
      const int nch = vir ? nob : nvb;
      const double* xb = X + (vir ? 256 * (b * nob) + lane : 256 * (b - nvb) + 16 * i + 4 * g);
      const int es = vir ? 64 : 1, cs = vir ? 256 : 256 * nob;
      const double* zl = ov_lds + (vir ? 0 : nop * 16) + lane;
      auto load = [&](double* x, int c) {
#pragma unroll
        for (int m = 0; m < 4; ++m) x[m] = xb[cs * c + es * m];
      };
      auto mul = [&](const double* x, int c) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
          for (int w = 0; w < CB; ++w)
            z[t][w] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[m], zl[w * R * 16 + 256 * c + 64 * m], z[t][w], 0, 0, 0);
      };
      chunk_pipeline<1>(nch, load, mul);
    }
    if (p > 1) __syncthreads();  // Z has been read
#pragma unroll
    for (int t = 0; t < BLK; ++t) {
      const int b = wave + OV_WAVES * t;
      if (b >= nbk) continue;
      const double fb = b < nvb ? -f : f;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int w = 0; w < CB; ++w) {
          const double v = fma(fb, z[t][w][q], keep ? c[t][w][q] : 0.0);
          if (p > 1) ov_lds[(w * R + lds_row(t, q)) * 16 + i] = v;
          else if (ro[t][q] >= 0 && c0 + 16 * w + i < n) Ct[ro[t][q] + c0 + 16 * w + i] = v;
        }
    }
    if (p > 1) __syncthreads();
  }
}

template __global__ void k_ov_apply<1, 2>(DevBatch, const int*, int, int, const double*, const double*, double);
template __global__ void k_ov_apply<1, 3>(DevBatch, const int*, int, int, const double*, const double*, double);
template __global__ void k_ov_apply<2, 2>(DevBatch, const int*, int, int, const double*, const double*, double);

// After a solve: the gap of the systems that converged in a rotation.  The
// couplings A_kj inside the classes, which the rotations leave, move the levels
// to second order, about as much as the expectation values A_kk have moved (1e-3
// Eh in pentacene pairs), so a level is taken as A_kk and, towards the gap, the
// sum of min(|A_kj|, A_kj^2 / |eps_k - eps_j|) over its class, for the orbitals
// whose last eigenvalue eps lies within 0.05 Eh of the gap's edges.  Where the
// gap no longer keeps the occupations at 0 and 2 to 2 occ, the system leaves the
// rotation route for good (mode 2) and becomes active again; *reopened counts
// them.
// (The true gap is met to 2e-4 Eh in pentacene pairs and to 1e-3 in pairs of six
// waters; the expectation values alone missed it by 1e-3 and 4e-3.)
// Bound by the chain of orbitals, a product with F and one with the class
// each: sixteen waves, 0.12 ms for 13 pentacene pairs and 2.05 ms for 3425 (without
// the couplings 0.085 and 1.2; four waves without them 0.16 and 1.5).
__global__ void __launch_bounds__(1024) k_ov_gap(DevBatch bt, const int* list, double kT, double occ, int* reopened) {
  const int si = list[blockIdx.x];
  if (bt.status[si] != 1 || !(bt.xn[si] >= 0.0)) return;
  const SysDesc d = bt.desc[si];
  const int n = d.nao, no = bt.ov_no[si];
  const double* eps = bt.eps + d.ao_off;
  const int* ov = bt.ov_idx + d.ao_off;
  const double* F = bt.F + d.mat_off;
  const double* Ct = bt.Ct + d.mat_off;
  __shared__ double diag, shift[16], crow[OV_MAXN], u[OV_MAXN], es[OV_MAXN];
  __shared__ int ox[OV_MAXN];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    ox[k] = ov[k];
    es[k] = eps[ox[k]];
  }
  __syncthreads();
  double homo = -1e300, lumo = 1e300;
  for (int k = 0; k < n; ++k) {
    if (k < no) homo = fmax(homo, es[k]);
    else lumo = fmin(lumo, es[k]);
  }
  double ho = -1e300, lu = 1e300;
  for (int k = 0; k < n; ++k) {
    const double e = es[k];
    if (k < no ? e < homo - 0.05 : e > lumo + 0.05) continue;
    for (int j = threadIdx.x; j < n; j += blockDim.x) crow[j] = Ct[ox[k] * n + j];
    __syncthreads();
    for (int r = wave; r < n; r += nw) {
      double t = 0.0;
      for (int j = lane; j < n; j += 64) t = fma(F[r * n + j], crow[j], t);
      t = wave_sum_f64(t);
      if (lane == 0) u[r] = t;
    }
    __syncthreads();
    double sh = 0.0;
    for (int c = (k < no ? 0 : no) + wave; c < (k < no ? no : n); c += nw) {
      double t = 0.0;
      for (int j = lane; j < n; j += 64) t = fma(Ct[ox[c] * n + j], u[j], t);
      t = fabs(wave_sum_f64(t));
      if (c != k) sh += fmin(t, t * t / fabs(e - es[c]));
    }
    if (lane == 0) shift[wave] = sh;
    if (wave == 0) {
      double t = 0.0;
      for (int j = lane; j < n; j += 64) t = fma(crow[j], u[j], t);
      t = wave_sum_f64(t);
      if (lane == 0) diag = t;
    }
    __syncthreads();
    sh = 0.0;
    for (int w = 0; w < nw; ++w) sh += shift[w];
    if (k < no) ho = fmax(ho, diag + sh);
    else lu = fmin(lu, diag - sh);
    __syncthreads();  // (diag, shift, crow and u have been read)
  }
  if (threadIdx.x == 0 && !(exp(-0.5 * (lu - ho) / kT) <= occ)) {
    bt.mode[si] = 2;
    bt.status[si] = 0;
    atomicAdd(reopened, 1);
  }
}

}  // namespace fx
