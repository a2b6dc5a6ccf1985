// Whole SCC solves of systems of up to 32 AOs (water monomers, pairs and
// triples), one wave per system.
//
// For such systems the batched kernels are launch latency: ten launches an
// iteration, 5 to 20 us each, for a few thousand operations.  Here a wave takes
// its system from Fock matrix to mixing, iteration after iteration, with the
// basis and the working matrices in LDS (7 KB for 16 AOs, 26 KB for 32), one
// work-group per wave so that no barrier is ever waited for; systems that are
// done leave the chip to the others.  The steps are those of the batched
// kernels: F = H0 + S (sigma + sigma') / 2, A = C^T F C on the FP64 matrix
// cores, cyclic Jacobi sweeps, Fermi occupations, the density's populations
// and energy, preconditioned Anderson mixing.
#include <hip/hip_runtime.h>

#include "fx_device.hpp"
#include "fx_kernels.hpp"

namespace fx {

typedef double v4d __attribute__((ext_vector_type(4)));

namespace {

// position of index slot k in round r of the round-robin tournament of m
__device__ inline int small_rr(int k, int r, int m) {
  if (k == 0) return 0;
  const int x = k - 1 + r;
  return 1 + (x >= m - 1 ? x - (m - 1) : x);
}

// D = op(A) B for NP x NP matrices in LDS (row stride LD): 16 x 16 blocks, the
// lane's element q of block (bi, bj) is row 16 bi + lane / 16 + 4 q, column
// 16 bj + lane % 16.  AT: A transposed, its rows weighted by w.  BT: B
// transposed.
template <int NP, int LD, bool AT, bool BT>
__device__ inline void small_gemm(const double* A, const double* B, const double* w, v4d (&d)[NP / 16][NP / 16]) {
  const int lane = threadIdx.x, i = lane & 15, g = lane >> 4;
#pragma unroll
  for (int a = 0; a < NP / 16; ++a)
#pragma unroll
    for (int b = 0; b < NP / 16; ++b) d[a][b] = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k0 = 0; k0 < NP; k0 += 4) {
    const int k = k0 + g;
    double x[NP / 16], y[NP / 16];
#pragma unroll
    for (int a = 0; a < NP / 16; ++a) {
      x[a] = AT ? A[k * LD + 16 * a + i] * w[k] : A[(16 * a + i) * LD + k];
      y[a] = BT ? B[(16 * a + i) * LD + k] : B[k * LD + 16 * a + i];
    }
#pragma unroll
    for (int a = 0; a < NP / 16; ++a)
#pragma unroll
      for (int b = 0; b < NP / 16; ++b)
        d[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[a], y[b], d[a][b], 0, 0, 0);
  }
}

template <int NP, int LD>
__device__ inline void small_put(double* D, const v4d (&d)[NP / 16][NP / 16]) {
  const int lane = threadIdx.x, i = lane & 15, g = lane >> 4;
#pragma unroll
  for (int a = 0; a < NP / 16; ++a)
#pragma unroll
    for (int b = 0; b < NP / 16; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) D[(16 * a + g + 4 * q) * LD + 16 * b + i] = d[a][b][q];
}

// value of a lane, as a wave-uniform number
__device__ inline double lane_f64(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Anderson coefficients from the Gram matrix G of the m residuals (indexed by
// slot): the bordered system in B.  Returns the lane's coefficient (lane k:
// the k-th oldest).
__device__ inline double small_anderson(const double (*G)[HIST], double* B, double* f, int nh, int m) {
  const int lane = threadIdx.x, M = m + 1, W = M + 1;
  for (int e = lane; e < M * W; e += 64) {
    const int r = e / W, c = e - r * W;
    double v = c == M ? (r == m ? 1.0 : 0.0) : r == c ? 0.0 : 1.0;
    if (r < m && c < m) {
      v = G[(nh - m + r) % HIST][(nh - m + c) % HIST];
      if (r == c) v *= 1.0 + 1e-12;  // (relative to itself: k_charges_mix)
    }
    B[e] = v;
  }
  wave_sync();
  return wave_solve(B, f, M);
}

}  // namespace

template <int NP>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NP == 16 ? 3 : 1)))
    k_scc_small(DevSystem sys, DevBatch bt, const int* list, SmallScc p) {
  constexpr int LD = NP + 1, NB = NP / 16;
  const int si = list[blockIdx.x];
  if (bt.status[si] != 0) return;
  const SysDesc d = bt.desc[si];
  const int n = d.nao, ns = d.nsh, lane = threadIdx.x;
  const double kT = sys.g.kT;
  __shared__ double C[NP * LD], F[NP * LD], T[NP * LD];
  __shared__ double pop[NP], eps[NP], occ[NP], sg[NP], cs_c[NP / 2], cs_s[NP / 2];
  __shared__ int cs_p[NP / 2], cs_q[NP / 2], ao_sh[NP];
  __shared__ double qv[NP], rv[NP], hX[HIST][NP], hR[HIST][NP], G[HIST][HIST];
  __shared__ double AB[(HIST + 1) * (HIST + 2)], Af[HIST + 1];
  const double* S = bt.S + d.mat_off;
  const double* H = bt.H0 + d.mat_off;
  const double* gam = bt.gam + d.gam_off;
  // this lane's AO and shell (ns <= n <= NP)
  for (int e = lane; e < NP * LD; e += 64) C[e] = T[e] = F[e] = 0.0;
  if (lane < NP) {
    ao_sh[lane] = lane < n ? bt.sys_ao_sh[d.ao_off + lane] : 0;
    occ[lane] = eps[lane] = sg[lane] = pop[lane] = qv[lane] = rv[lane] = 0.0;
  }
  __syncthreads();
  for (int e = lane; e < n * n; e += 64) {
    const int r = e / n;
    C[r * LD + e - r * n] = bt.Ct[d.mat_off + e];
  }
  const bool has = lane < ns;
  int mu0 = 0, nmu = 0, s0 = 0, s1 = 0;
  double q0 = 0.0, Gam = 0.0, phi = 0.0, qin = 0.0;
  if (has) {
    const int a = bt.sys_sh_atom[d.sh_off + lane];
    const DevElem& el = sys.elems[sys.elem[bt.sys_atoms[d.atom_off + a]]];
    s0 = bt.sys_atom_sh0[d.atom_off + a];
    s1 = a + 1 < d.nat ? bt.sys_atom_sh0[d.atom_off + a + 1] : ns;
    mu0 = bt.sys_atom_ao0[d.atom_off + a] + el.ao0[lane - s0];
    nmu = el.nao_sh[lane - s0];
    q0 = bt.sh_q0 ? bt.sh_q0[d.sh_off + lane] : el.q0[lane - s0];
    Gam = el.Gamma;
    phi = bt.phi[d.sh_off + lane];
    qin = bt.q_in[d.sh_off + lane];
  }
  // gamma times the vector in v (LDS), at this lane's shell
  auto gamma_times = [&](const double* v) {
    double t = 0.0;
    if (has)
      for (int u = 0; u < ns; ++u) t = fma(gam[u * ns + lane], v[u], t);
    return t;
  };
  auto atom_charge = [&](const double* v) {
    double t = 0.0;
    for (int u = s0; u < s1; ++u) t += v[u];
    return t;
  };
  double* hx = bt.hx + (long long)d.sh_off * HIST;
  double* hr = bt.hr + (long long)d.sh_off * HIST;
  int nh = max(0, bt.nhist[si]);
  for (int k = 0; k < HIST; ++k)
    if (lane < NP) {
      const bool in = has && k < nh;
      hX[k][lane] = in ? hx[k * ns + lane] : 0.0;
      hR[k][lane] = in ? hr[k * ns + lane] : 0.0;
    }
  __syncthreads();
  for (int a = 0; a < min(nh, HIST); ++a)
    for (int b = 0; b <= a; ++b) {
      const double v = wave_sum_f64(has ? hR[a][lane] * hR[b][lane] : 0.0);
      if (lane == 0) G[a][b] = G[b][a] = v;
    }
  double err = bt.err[si], e_prev = bt.e_prev[si], e_int = 0.0, mts = 0.0, qout = 0.0;
  int it = bt.niter[si], status = 0;
  const double erep = bt.erep[si];
  const int no = (int)(0.5 * d.nel + 0.5);
  const bool even = fabs(d.nel - 2.0 * no) < 1e-9 && no >= 1 && no < n;
  const int m = n + (n & 1);
  for (int pass = 0; pass < p.passes && status == 0; ++pass) {
    // ---- Fock matrix
    if (lane < NP) qv[lane] = qin;
    __syncthreads();
    {
      const double qa = atom_charge(qv);
      const double sig = gamma_times(qv) - Gam * qa * qa + phi;
      if (lane < NP) sg[lane] = sig;
      if (has) bt.sig[d.sh_off + lane] = sig;
    }
    __syncthreads();
    for (int e = lane; e < n * n; e += 64) {
      const int r = e / n, c = e - r * n;
      F[r * LD + c] = H[e] + 0.5 * S[e] * (sg[ao_sh[r]] + sg[ao_sh[c]]);
    }
    __syncthreads();
    // ---- A = (C^T F) C
    {
      v4d t[NB][NB];
      small_gemm<NP, LD, false, false>(C, F, nullptr, t);
      small_put<NP, LD>(T, t);
      __syncthreads();
      small_gemm<NP, LD, false, true>(T, C, nullptr, t);
      __syncthreads();
      small_put<NP, LD>(F, t);
      __syncthreads();
    }
    // ---- cyclic Jacobi on A (in F), rotating the rows of C
    {
      double f2 = 0.0;
      for (int e = lane; e < NP * LD; e += 64) f2 = fma(F[e], F[e], f2);
      const double fro = sqrt(wave_sum_f64(f2));
      const double thr = fmax(p.rel_tol * (fro > 0.0 ? fro : 1.0), p.thr_scale * err);
      const int msw = p.cold && pass == 0 ? p.max_sweeps : err > p.early_err || err <= p.cap_err ? 2 : 1;
      for (int sweep = 0; sweep < msw; ++sweep) {
        bool rot = false;
        for (int r = 0; r < m - 1; ++r) {
          bool mine = false;
          if (lane < m / 2) {
            const int x = small_rr(lane, r, m), y = small_rr(m - 1 - lane, r, m);
            const int pp = min(x, y), qq = max(x, y);
            double c = 1.0, s = 0.0;
            if (qq < n) {
              const double apq = F[pp * LD + qq];
              if (fabs(apq) > thr) {
                const double theta = (F[qq * LD + qq] - F[pp * LD + pp]) / (2.0 * apq);
                const double t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(fma(theta, theta, 1.0)));
                c = 1.0 / sqrt(fma(t, t, 1.0));
                s = t * c;
                mine = true;
              }
            }
            cs_c[lane] = c;
            cs_s[lane] = s;
            cs_p[lane] = pp;
            cs_q[lane] = min(qq, NP - 1);  // (a bye pairs with n < NP: a zero row, c = 1)
          }
          if (!__ballot(mine)) continue;
          rot = true;
          __syncthreads();
          // rows of A and C: lane = column, 64 / NP pairs at a time
          const int j = lane & (NP - 1);
          for (int k = lane / NP; k < m / 2; k += 64 / NP) {
            const double c = cs_c[k], s = cs_s[k];
            if (s != 0.0) {
              const int a = cs_p[k] * LD + j, b = cs_q[k] * LD + j;
              const double fa = F[a], fb = F[b], ca = C[a], cb = C[b];
              F[a] = c * fa - s * fb;
              F[b] = s * fa + c * fb;
              C[a] = c * ca - s * cb;
              C[b] = s * ca + c * cb;
            }
          }
          __syncthreads();
          // columns of A: lane = row
          for (int k = lane / NP; k < m / 2; k += 64 / NP) {
            const double c = cs_c[k], s = cs_s[k];
            if (s != 0.0) {
              const int a = j * LD + cs_p[k], b = j * LD + cs_q[k];
              const double fa = F[a], fb = F[b];
              F[a] = c * fa - s * fb;
              F[b] = s * fa + c * fb;
            }
          }
          __syncthreads();
        }
        if (!rot) break;
      }
    }
    // ---- Fermi occupations (k_fermi): Newton's method on the log ratio of
    // electrons above and holes below a gap, else bisection
    const double ev = lane < n ? F[lane * LD + lane] : 0.0;
    if (lane < NP) eps[lane] = ev;
    __syncthreads();
    double ef = 0.0;
    bool found = false;
    if (even) {
      int rank = 0;
      for (int j = 0; j < n; ++j) rank += eps[j] < ev || (eps[j] == ev && j < lane) ? 1 : 0;
      const bool oc = lane < n && rank < no, un = lane < n && rank >= no;
      const double homo = wave_max_f64(oc ? ev : -1e300), lumo = -wave_max_f64(un ? -ev : -1e300);
      const double gap = lumo - homo;
      if (gap > 8.0 * kT) {
        ef = 0.5 * (homo + lumo);
        found = gap > 1200.0 * kT;
        for (int k = 0; k < 20 && !found; ++k) {
          const double f = oc || un ? 1.0 / (1.0 + exp((oc ? ef - ev : ev - ef) / kT)) : 0.0, g = f * (1.0 - f);
          const double a0 = wave_sum_f64(un ? f : 0.0), a1 = wave_sum_f64(un ? g : 0.0);
          const double b0 = wave_sum_f64(oc ? f : 0.0), b1 = wave_sum_f64(oc ? g : 0.0);
          const double step = -kT * log(a0 / b0) / (a1 / a0 + b1 / b0);
          if (!(fabs(step) < gap)) break;
          ef += step;
          found = fabs(step) < 1e-9 * kT;
        }
      }
    }
    if (!found) {
      double lo = -wave_max_f64(lane < n ? -ev : -1e300) - 1.0, hi = wave_max_f64(lane < n ? ev : -1e300) + 1.0;
      for (int k = 0; k < 300; ++k) {
        const double mid = 0.5 * (lo + hi);
        const double tot = wave_sum_f64(lane < n ? 2.0 / (1.0 + exp((ev - mid) / kT)) : 0.0);
        if (tot > d.nel) hi = mid;
        else lo = mid;
        if (hi - lo < 1e-15) break;
      }
      ef = 0.5 * (lo + hi);
    }
    {
      double ts = 0.0;
      if (lane < n) {
        const double f = 1.0 / (1.0 + exp((ev - ef) / kT));
        occ[lane] = 2.0 * f;
        if (f > 0.0) ts += f * log(f);
        if (f < 1.0) ts += (1.0 - f) * log(1.0 - f);
      }
      mts = 2.0 * kT * wave_sum_f64(ts);
    }
    __syncthreads();
    // ---- density: populations (P S)_ii and Tr(P H0)
    double eh = 0.0;
    {
      v4d t[NB][NB];
      small_gemm<NP, LD, true, false>(C, C, occ, t);
      const int i = lane & 15, g = lane >> 4;
#pragma unroll
      for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = 16 * a + g + 4 * q;
          double v = 0.0;
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            const int c = 16 * b + i;
            if (r < n && c < n) {
              v = fma(t[a][b][q], S[r * n + c], v);
              eh = fma(t[a][b][q], H[r * n + c], eh);
            }
          }
#pragma unroll
          for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off);
          if (i == 0) pop[r] = v;
        }
      eh = wave_sum_f64(eh);
    }
    __syncthreads();
    // ---- charges, energy, residual
    if (has) {
      double v = 0.0;
      for (int u = mu0; u < mu0 + nmu; ++u) v += pop[u];
      qout = v - q0;
      qv[lane] = qout;
    }
    __syncthreads();
    {
      const double gq = gamma_times(qv), qa = atom_charge(qv);
      const double e2 = wave_sum_f64(has ? 0.5 * qout * gq : 0.0);
      const double e3 = wave_sum_f64(has && lane == s0 ? -Gam * qa * qa * qa / 3.0 : 0.0);
      e_int = eh + e2 + e3 + mts + erep;
    }
    err = wave_max_f64(has ? fabs(qout - qin) : 0.0);
    ++it;
    const bool conv = err < p.tol && fabs(e_int - e_prev) < p.etol && it > 1;
    e_prev = e_int;
    if (conv) status = 1;
    else if (it >= p.max_iter) status = 2;
    if (status != 0) break;
    // ---- mixing of the input charges (k_charges_mix)
    double r = qout - qin;
    if (bt.pre) {
      if (lane < NP) rv[lane] = r;
      __syncthreads();
      const float* pre = bt.pre + d.gam_off;
      double v = 0.0;
      if (has)
        for (int u = 0; u < ns; ++u) v = fma((double)pre[u * ns + lane], rv[u], v);
      r = v;
    }
    const int slot = nh % HIST;
    ++nh;
    const int hm = min(nh, HIST);
    if (has) {
      hX[slot][lane] = qin;
      hR[slot][lane] = r;
    }
    __syncthreads();
    for (int k = 0; k < hm; ++k) {
      const double v = wave_sum_f64(has ? hR[slot][lane] * hR[k][lane] : 0.0);
      if (lane == 0) G[slot][k] = G[k][slot] = v;
    }
    __syncthreads();
    if (hm == 1) {
      // (plain without a preconditioner)
      qin += p.beta * (bt.pre ? r : qout - qin);
    } else {
      const double x = small_anderson(G, AB, Af, nh, hm);
      double v = 0.0;
      for (int k = 0; k < hm; ++k) {
        const int sl = (nh - hm + k) % HIST;
        const double c = lane_f64(x, k);
        if (has) v = fma(c, fma(p.beta, hR[sl][lane], hX[sl][lane]), v);
      }
      qin = v;
    }
  }
  // ---- state
  __syncthreads();
  for (int e = lane; e < n * n; e += 64) {
    const int r = e / n;
    bt.Ct[d.mat_off + e] = C[r * LD + e - r * n];
  }
  if (lane < n) {
    bt.eps[d.ao_off + lane] = eps[lane];
    bt.occ[d.ao_off + lane] = occ[lane];
  }
  {
    const bool take = lane < n && occ[lane & (NP - 1)] > OCC_MIN;
    const unsigned long long b = __ballot(take);
    if (take) bt.occ_idx[d.ao_off + __popcll(b & ((1ULL << lane) - 1ULL))] = lane;
    if (lane == 0) bt.occ_cnt[si] = __popcll(b);
  }
  if (has) {
    bt.q_out[d.sh_off + lane] = qout;
    bt.q_in[d.sh_off + lane] = qin;
    if (status == 0)
      for (int k = 0; k < min(nh, HIST); ++k) {
        hx[k * ns + lane] = hX[k][lane];
        hr[k * ns + lane] = hR[k][lane];
      }
  }
  if (lane == 0) {
    bt.status[si] = status;
    bt.niter[si] = it;
    bt.nhist[si] = nh;
    bt.err[si] = err;
    bt.e_int[si] = e_int;
    bt.e_prev[si] = e_prev;
    bt.mts[si] = mts;
    bt.mode[si] = 0;
    bt.xn[si] = -1.0;
  }
}

template __global__ void k_scc_small<16>(DevSystem, DevBatch, const int*, SmallScc);
template __global__ void k_scc_small<32>(DevSystem, DevBatch, const int*, SmallScc);

}  // namespace fx
