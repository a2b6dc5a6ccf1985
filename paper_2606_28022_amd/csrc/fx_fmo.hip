// FMO bookkeeping kernels: moving shell charges between the supersystem and
// the fragment batches, the dimer/trimer terms of the many-body energy, and
// the fixed-order energy sum.
//
// Cluster terms (section "Fragment molecular orbital method"): the charge
// transfer ddq = dq^X - (dq^I + dq^J (+ dq^K)) of eq. ddq_calc / ctijk, the
// embedding correction Delta E^V = ddq . phi^X of eqs.
// dimer_embedding_correction and trimer_embedding, and the interaction
// energy Delta E_X = E_X - sum E_I + Delta E^V of eqs.
// fmo2-energy-components and trimer_interaction_energy.
#include <hip/hip_runtime.h>

#include "fx_device.hpp"
#include "fx_kernels.hpp"

namespace fx {

__global__ void k_gather_shell(DevBatch bt, const double* src_global, double* dst_local) {
  int si = blockIdx.x;
  const SysDesc d = bt.desc[si];
  for (int s = threadIdx.x; s < d.nsh; s += blockDim.x)
    dst_local[d.sh_off + s] = src_global[bt.sys_sh_global[d.sh_off + s]];
}

__global__ void k_scatter_shell(DevBatch bt, const double* src_local, double* dst_global) {
  int si = blockIdx.x;
  const SysDesc d = bt.desc[si];
  for (int s = threadIdx.x; s < d.nsh; s += blockDim.x)
    dst_global[bt.sys_sh_global[d.sh_off + s]] = src_local[d.sh_off + s];
}

// max |a - b| in two stages: one partial per work-group (grid-stride), then
// one work-group over the partials (the maximum does not depend on the order)
__global__ void k_absdiff_part(const double* a, const double* b, int n, double* part) {
  __shared__ double red[256];
  double m = 0.0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) m = fmax(m, fabs(a[i] - b[i]));
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void k_max_reduce(const double* part, int np, double* out) {
  __shared__ double red[256];
  double m = 0.0;
  for (int i = threadIdx.x; i < np; i += blockDim.x) m = fmax(m, part[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0];
}

// per cluster system: ddq (written per local shell), Delta E^V and Delta E_X
__global__ void k_cluster_terms(DevBatch bt, const double* qmono, const double* e_mono, double* ddq, double* dEV,
                                double* dE) {
  int si = blockIdx.x;
  const SysDesc d = bt.desc[si];
  __shared__ double red[256];
  double loc = 0.0;
  for (int s = threadIdx.x; s < d.nsh; s += blockDim.x) {
    double v = bt.q_out[d.sh_off + s] - qmono[bt.sys_sh_global[d.sh_off + s]];
    ddq[d.sh_off + s] = v;
    loc += v * bt.phi[d.sh_off + s];
  }
  red[threadIdx.x] = loc;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double ev = red[0];
    double e = bt.e_int[si];
    for (int k = 0; k < d.nfrag; ++k) e -= e_mono[d.frag[k]];
    dEV[si] = ev;
    dE[si] = e + ev;
  }
}

// Neumaier-compensated sum of several arrays in a fixed order, in two stages:
// a work-group takes a contiguous slice of the concatenated sequence (its
// threads consecutive entries, so the reads are coalesced), combines its
// threads' (sum, compensation) pairs by a tree and writes one pair; one
// work-group combines the pairs.  Deterministic for a given input.  (One
// work-group with a contiguous slice per thread and a serial sum of the 256
// partial pairs took 940 us for the 530,000 terms of 1,024 waters and 35 us
// for the fewest; the two stages take 10 and 8 us.)
__device__ inline void neu_add(double& s, double& c, double v) {
  double t = s + v;
  if (fabs(s) >= fabs(v)) c += (s - t) + v;
  else c += (v - t) + s;
  s = t;
}

// pairs of the work-group's 256 threads into thread 0's
__device__ inline void neu_block(double& s, double& c) {
  __shared__ double ps[256], pc[256];
  ps[threadIdx.x] = s;
  pc[threadIdx.x] = c;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      double S = ps[threadIdx.x], C = pc[threadIdx.x];
      neu_add(S, C, ps[threadIdx.x + w]);
      ps[threadIdx.x] = S;
      pc[threadIdx.x] = C + pc[threadIdx.x + w];
    }
    __syncthreads();
  }
  s = ps[0];
  c = pc[0];
}

__global__ void __launch_bounds__(256) k_sum_neumaier(SumArrays a, double* part) {
  long long total = 0;
  for (int k = 0; k < a.n; ++k) total += a.len[k];
  const long long per = (total + gridDim.x - 1) / gridDim.x;
  const long long b = per * blockIdx.x, e = b + per < total ? b + per : total;
  double s = 0.0, c = 0.0;
  long long base = 0;
  for (int k = 0; k < a.n; ++k) {
    const long long lo = b > base ? b : base;
    const long long hi = e < base + a.len[k] ? e : base + a.len[k];
    for (long long i = lo + threadIdx.x; i < hi; i += 256) neu_add(s, c, a.p[k][i - base]);
    base += a.len[k];
  }
  neu_block(s, c);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = s;
    part[2 * blockIdx.x + 1] = c;
  }
}

__global__ void __launch_bounds__(256) k_sum_neumaier_final(const double* part, int nparts, double* out) {
  double s = 0.0, c = 0.0;
  for (int k = threadIdx.x; k < nparts; k += 256) {
    neu_add(s, c, part[2 * k]);
    c += part[2 * k + 1];
  }
  neu_block(s, c);
  if (threadIdx.x == 0) *out = s + c;
}

// ---------------------------------------------------------------------------
// Anderson (Pulay) mixing of a long vector (the monomer charges of the
// self-consistent embedding).  History slots are passed oldest first.
// B_ij = r_i . r_j, one work-group per (i, j), fixed-order tree reduction
// Gram matrix of the history residuals in one pass over them: each
// work-group accumulates all m (m + 1) / 2 products of its slice (grid-stride)
// and writes them to part[block][HIST_TRI]; k_hist_solve adds the partials in
// block order (deterministic).
constexpr int HIST_TRI = HIST * (HIST + 1) / 2;
__global__ void __launch_bounds__(256) k_hist_gram_part(const double* R, long long n, Slots sl, double* part) {
  const int m = sl.m;
  double acc[HIST_TRI];
#pragma unroll
  for (int t = 0; t < HIST_TRI; ++t) acc[t] = 0.0;
  for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long long)gridDim.x * blockDim.x) {
    double r[HIST];
#pragma unroll
    for (int i = 0; i < HIST; ++i) r[i] = i < m ? R[(long long)sl.id[i] * n + k] : 0.0;
    int t = 0;
#pragma unroll
    for (int i = 0; i < HIST; ++i)
#pragma unroll
      for (int j = i; j < HIST; ++j) acc[t++] += r[i] * r[j];
  }
  __shared__ double red[4][HIST_TRI];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int t = 0; t < HIST_TRI; ++t) {
    double v = acc[t];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane == 0) red[wave][t] = v;
  }
  __syncthreads();
  if (threadIdx.x < HIST_TRI)
    part[(long long)blockIdx.x * HIST_TRI + threadIdx.x] =
        red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
}

// B_ij from the partials (block order), then the mixing coefficients:
// minimise |sum c_k r_k| subject to sum c_k = 1 (bordered normal equations,
// Gaussian elimination with partial pivoting, in LDS by one thread)
__global__ void k_hist_solve(const double* part, int np, Slots sl, double* coef) {
  const int m = sl.m, M = m + 1;
  __shared__ double tri[HIST_TRI];
  __shared__ double A[(HIST + 1) * (HIST + 1)], rhs[HIST + 1];
  for (int t = threadIdx.x; t < HIST_TRI; t += blockDim.x) {
    double v = 0.0;
    for (int p = 0; p < np; ++p) v += part[(long long)p * HIST_TRI + t];
    tri[t] = v;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  auto Bij = [&](int i, int j) {
    const int a = i < j ? i : j, b = i < j ? j : i;
    return tri[a * HIST - a * (a - 1) / 2 + (b - a)];  // row a of the packed upper triangle
  };
  double tr = 0.0;
  for (int i = 0; i < m; ++i) tr += Bij(i, i);
  for (int i = 0; i < M; ++i) {
    rhs[i] = (i == m) ? 1.0 : 0.0;
    for (int j = 0; j < M; ++j) {
      double v;
      if (i < m && j < m) v = Bij(i, j) + (i == j ? 1e-14 * tr : 0.0);
      else if (i == m && j == m) v = 0.0;
      else v = 1.0;
      A[i * M + j] = v;
    }
  }
  for (int c = 0; c < M; ++c) {
    int piv = c;
    for (int r = c + 1; r < M; ++r)
      if (fabs(A[r * M + c]) > fabs(A[piv * M + c])) piv = r;
    if (piv != c) {
      for (int k = 0; k < M; ++k) {
        double t = A[c * M + k];
        A[c * M + k] = A[piv * M + k];
        A[piv * M + k] = t;
      }
      double t = rhs[c];
      rhs[c] = rhs[piv];
      rhs[piv] = t;
    }
    double dv = A[c * M + c];
    if (fabs(dv) < 1e-300) dv = 1e-300;
    for (int r = c + 1; r < M; ++r) {
      double f = A[r * M + c] / dv;
      for (int k = c; k < M; ++k) A[r * M + k] -= f * A[c * M + k];
      rhs[r] -= f * rhs[c];
    }
  }
  for (int c = M - 1; c >= 0; --c) {
    double v = rhs[c];
    for (int k = c + 1; k < M; ++k) v -= A[c * M + k] * rhs[k];
    double dv = A[c * M + c];
    rhs[c] = v / (fabs(dv) < 1e-300 ? 1e-300 : dv);
  }
  for (int i = 0; i < m; ++i) coef[i] = rhs[i];
}

// q = sum_k c_k (x_k + beta r_k)
__global__ void k_hist_mix(const double* X, const double* R, long long n, Slots sl, const double* coef, double beta,
                           double* q) {
  long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  double v = 0.0;
  for (int i = 0; i < sl.m; ++i) {
    long long o = (long long)sl.id[i] * n + k;
    v += coef[i] * (X[o] + beta * R[o]);
  }
  q[k] = v;
}

// store x and r = y - x into history slot `slot`, and max |r| into *dmax
__global__ void k_hist_store(const double* x, const double* y, long long n, int slot, double* X, double* R) {
  long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  X[(long long)slot * n + k] = x[k];
  R[(long long)slot * n + k] = y[k] - x[k];
}

// ---------------------------------------------------------------------------
// The iterations over the whole charge vector (fused monomer steps, adjoint
// response) as few launches: on small systems a step is launch latency, and a
// step of separate gather, reset, scatter, difference, maximum, history and
// Gram launches took 18 of them besides its field pass and its SCC iteration.

// start of a fused monomer step, per monomer: charges and field of its shells,
// iteration state cleared (as k_reset_state with the residual kept); refresh:
// the eigensolver takes it.  The step's maxima are cleared too.
__global__ void __launch_bounds__(64) k_mono_begin(DevBatch bt, const double* q, const double* phi, int refresh,
                                                   unsigned long long* maxima) {
  const int si = blockIdx.x;
  const SysDesc d = bt.desc[si];
  for (int s = threadIdx.x; s < d.nsh; s += 64) {
    const int g = bt.sys_sh_global[d.sh_off + s];
    bt.q_in[d.sh_off + s] = q[g];
    bt.phi[d.sh_off + s] = phi[g];
  }
  if (threadIdx.x == 0) {
    bt.status[si] = 0;
    bt.niter[si] = 0;
    bt.nhist[si] = 0;
    bt.e_prev[si] = 0.0;
    if (refresh) {
      bt.mode[si] = 0;
      bt.xn[si] = -1.0;
    }
    if (si == 0)
      for (int k = 0; k < STEP_MAXIMA; ++k) maxima[k] = 0ULL;
  }
}

// history row of the system's shells: x and r into the newest slot, and the
// products of r with the m residuals into part[HIST si + k] (k-th oldest)
__device__ inline void hist_row(const DevBatch& bt, const SysDesc& d, int si, double* X, double* R, long long n,
                                const Slots& sl, const double* x, const double* r, double* part) {
  const int m = sl.m;
  double acc[HIST];
#pragma unroll
  for (int k = 0; k < HIST; ++k) acc[k] = 0.0;
  for (int s = threadIdx.x; s < d.nsh; s += 64) {
    const int g = bt.sys_sh_global[d.sh_off + s];
    X[(long long)sl.id[m - 1] * n + g] = x[s];
    R[(long long)sl.id[m - 1] * n + g] = r[s];
#pragma unroll
    for (int k = 0; k < HIST; ++k)
      if (k < m) acc[k] = fma(r[s], k == m - 1 ? r[s] : R[(long long)sl.id[k] * n + g], acc[k]);
  }
#pragma unroll
  for (int k = 0; k < HIST; ++k) {
    const double v = wave_sum_f64(acc[k]);
    if (threadIdx.x == 0) part[HIST * si + k] = v;
  }
}

// maximum into a cleared slot: non-negative numbers order as their bits (a NaN
// above all, so that it never passes for convergence)
__device__ inline void max_into(unsigned long long* m, double v) {
  atomicMax(m, (unsigned long long)__double_as_longlong(fabs(v)));
}

// end of a fused monomer step, per monomer (one wave): its charges into q_new,
// max |q_out - q_in|, max |X| (DevBatch) and whether it rotates next, and the
// history row of the
// Newton step (1 + M G)^-1 (q_out - q_in) (bt.pre, stored transposed)
__global__ void __launch_bounds__(64) k_mono_end(DevBatch bt, double* q_new, double* X, double* R, long long n, Slots sl,
                                                 double* part, unsigned long long* maxima) {
  const int si = blockIdx.x;
  const SysDesc d = bt.desc[si];
  const int ns = d.nsh, lane = threadIdx.x;
  __shared__ double r[MAXN], v[MAXN];
  const double* qi = bt.q_in + d.sh_off;
  const double* qo = bt.q_out + d.sh_off;
  double dm = 0.0;
  bool nan = false;
  for (int s = lane; s < ns; s += 64) {
    const double t = qo[s] - qi[s];
    r[s] = t;
    nan = nan || t != t;
    dm = fmax(dm, fabs(t));
    q_new[bt.sys_sh_global[d.sh_off + s]] = qo[s];
  }
  dm = wave_max_f64(dm);
  nan = __ballot(nan) != 0;
  __syncthreads();
  const float* Pr = bt.pre + d.gam_off;
  for (int s = lane; s < ns; s += 64) {
    double t = 0.0;
#pragma unroll 8
    for (int u = 0; u < ns; ++u) t += (double)Pr[(long long)u * ns + s] * r[u];
    v[s] = t;
  }
  __syncthreads();
  hist_row(bt, d, si, X, R, n, sl, qi, v, part);
  if (lane == 0) {
    max_into(maxima, nan ? __longlong_as_double(0x7ff8000000000000LL) : dm);
    const double xn = bt.xn[si];
    max_into(maxima + 1, xn < 0.0 ? 0.0 : xn);  // (a NaN goes on as one)
    max_into(maxima + 2, bt.mode[si] == 1 ? 0.0 : 1.0);
  }
}

// one adjoint response sweep, per monomer: w = R y, u = -M w
__global__ void __launch_bounds__(64) k_resp_sweep(DevBatch bt, const double* R, const double* M, const double* y,
                                                   double* w, double* u, unsigned long long* maxima) {
  const int si = blockIdx.x;
  const SysDesc d = bt.desc[si];
  const int ns = d.nsh;
  __shared__ double ys[MAXN], ws[MAXN];
  for (int s = threadIdx.x; s < ns; s += 64) ys[s] = y[bt.sys_sh_global[d.sh_off + s]];
  __syncthreads();
  for (int s = threadIdx.x; s < ns; s += 64) {
    double v = 0.0;
#pragma unroll 8
    for (int t = 0; t < ns; ++t) v += R[d.gam_off + (long long)s * ns + t] * ys[t];
    ws[s] = v;
    w[d.sh_off + s] = v;
  }
  __syncthreads();
  for (int s = threadIdx.x; s < ns; s += 64) {
    double v = 0.0;
#pragma unroll 8
    for (int t = 0; t < ns; ++t) v += M[d.gam_off + (long long)t * ns + s] * ws[t];  // (M is symmetric)
    u[bt.sys_sh_global[d.sh_off + s]] = -v;
  }
  if (si == 0 && threadIdx.x < STEP_MAXIMA) maxima[threadIdx.x] = 0ULL;
}

// its end, per monomer: y_new = v + field of u, max |y_new - y|, history row
__global__ void __launch_bounds__(64) k_resp_end(DevBatch bt, const double* v, const double* fu, const double* y,
                                                 double* y_new, double* X, double* R, long long n, Slots sl,
                                                 double* part, unsigned long long* maxima) {
  const int si = blockIdx.x;
  const SysDesc d = bt.desc[si];
  __shared__ double x[MAXN], r[MAXN];
  double dm = 0.0;
  bool nan = false;
  for (int s = threadIdx.x; s < d.nsh; s += 64) {
    const int g = bt.sys_sh_global[d.sh_off + s];
    const double yn = v[g] + fu[g], yo = y[g], t = yn - yo;
    y_new[g] = yn;
    x[s] = yo;
    r[s] = t;
    nan = nan || t != t;
    dm = fmax(dm, fabs(t));
  }
  dm = wave_max_f64(dm);
  nan = __ballot(nan) != 0;
  __syncthreads();
  hist_row(bt, d, si, X, R, n, sl, x, r, part);
  if (threadIdx.x == 0) max_into(maxima, nan ? __longlong_as_double(0x7ff8000000000000LL) : dm);
}

// Mixing of such a step: the newest residual's Gram row from the systems'
// parts (fixed order), the other entries from gram[slot][slot] (where
// work-group 0 also stores the new row), the coefficients by one wave of every
// work-group, and the work-group's slice of q = sum_k c_k (x_k + beta r_k).
__global__ void __launch_bounds__(256) k_hist_next(const double* X, const double* R, long long n, Slots sl,
                                                   const double* part, int nparts, double* gram, double beta,
                                                   double* q, const double* maxima, double* host_maxima) {
  const int m = sl.m, M = m + 1, W = M + 1, t = threadIdx.x;
  if (blockIdx.x == 0 && t < STEP_MAXIMA) host_maxima[t] = maxima[t];  // (pinned: the step's residual for the host)
  __shared__ double sum[32][HIST], row[HIST], B[(HIST + 1) * (HIST + 2)], f[HIST + 1], coef[HIST];
  {
    const int k = t & (HIST - 1);
    double v = 0.0;
    for (int p = t / HIST; p < nparts; p += 32) v += part[HIST * p + k];
    sum[t / HIST][k] = v;
  }
  __syncthreads();
  if (t < HIST) {
    double v = 0.0;
    for (int p = 0; p < 32; ++p) v += sum[p][t];
    row[t] = v;
    if (blockIdx.x == 0 && t < m) {
      gram[sl.id[m - 1] * HIST + sl.id[t]] = v;
      if (t != m - 1) gram[sl.id[t] * HIST + sl.id[m - 1]] = v;
    }
  }
  __syncthreads();
  if (t < 64) {
    auto entry = [&](int i, int j) {
      return i == m - 1 ? row[j] : j == m - 1 ? row[i] : gram[sl.id[i] * HIST + sl.id[j]];
    };
    double tr = 0.0;
    for (int i = 0; i < m; ++i) tr += entry(i, i);
    for (int e = t; e < M * W; e += 64) {
      const int i = e / W, j = e - i * W;
      double v = j == M ? (i == m ? 1.0 : 0.0) : i == j ? 0.0 : 1.0;
      if (i < m && j < m) v = entry(i, j) + (i == j ? 1e-14 * tr : 0.0);
      B[e] = v;
    }
    wave_sync();
    const double c = wave_solve(B, f, M);
    if (t < m) coef[t] = c;
  }
  __syncthreads();
  for (long long g = (long long)blockIdx.x * 256 + t; g < n; g += (long long)gridDim.x * 256) {
    double v = 0.0;
    for (int k = 0; k < m; ++k) v += coef[k] * (X[sl.id[k] * n + g] + beta * R[sl.id[k] * n + g]);
    q[g] = v;
  }
}

// Several host tables to their device buffers (or back) in one launch:
// blockIdx.y's piece lies at its offset of the pinned block `host`, which the
// kernel reads or writes over the bus.  A blocking copy each cost 25 to 35 us,
// about 60 of them per run; offsets are multiples of 16 bytes, device
// addresses those of whole buffers.
__global__ void __launch_bounds__(256) k_transfer(TransferList l, char* host, int to_host) {
  const TransferItem it = l.item[blockIdx.y];
  char* const h = host + it.off;
  char* const d = static_cast<char*>(it.dev);
  const char* const src = to_host ? d : h;
  char* const dst = to_host ? h : d;
  const long long tid = (long long)blockIdx.x * 256 + threadIdx.x, nth = (long long)gridDim.x * 256;
  const bool wide = (reinterpret_cast<unsigned long long>(d) & 15) == 0;
  const long long n16 = wide ? it.bytes / 16 : 0;
  for (long long k = tid; k < n16; k += nth)
    reinterpret_cast<float4*>(dst)[k] = reinterpret_cast<const float4*>(src)[k];
  for (long long k = 16 * n16 + tid; k < it.bytes; k += nth) dst[k] = src[k];
}

// Trimer corrections Delta E_IJK - Delta E_IJ - Delta E_IK - Delta E_JK
// (eq. fmo3_energy; an ES-DIM sub-pair enters with its ES-DIM value): sub
// holds, per trimer, the three sub-pairs as an index into dE_scc or nscc +
// an index into dE_esd.
__global__ void k_trimer_corr(long long ntri, const double* dEIJK, const double* dE_scc, long long nscc,
                              const double* dE_esd, const long long* sub, double* out) {
  const long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (k >= ntri) return;
  double v = dEIJK[k];
  for (int p = 0; p < 3; ++p) {
    const long long e = sub[3 * k + p];
    v -= e < nscc ? dE_scc[e] : dE_esd[e - nscc];
  }
  out[k] = v;
}

}  // namespace fx
