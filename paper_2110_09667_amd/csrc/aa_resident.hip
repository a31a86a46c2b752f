// aa_resident.hip -- one iteration of Alg. 1 in one workgroup with every
// vector in registers.
//
// For n rows and a window of m columns with Q in the register file (n <= 512 R
// rows, m <= KM columns, R KM <= 40 doubles of Q per lane) an iteration is not
// bound by memory (400 KB at n = 4096, m = 5) but by its chain of dependent
// reductions.  The passes of aa_batch.hip walk Q once per reduction and run
// each dense tail from global memory: 46 us a step at n = 4096, m = 5 and
// 28 us at n = 576, m = 3, a dozen memory round trips.  Here every load is
// issued at the start, R and T sit in LDS, a reduction is one butterfly per
// wave and one barrier, every wave sums the eight waves' partials and runs the
// small triangular solves itself (so their results need no second barrier),
// and the columns of Q are written back once: 17.7 us at n = 4096, m = 5 (ICWY)
// and 7.3 us at n = 576, m = 3 (MGS).
//
// The quantities are those of aa_batch.hip, each the same sum over rows in
// another order; AA_FUSE_RHS and AA_FUSE_DELETE name passes to merge and have
// nothing to merge here.
#include <math.h>

#include <type_traits>

#include "aa_device.h"

namespace aa {
namespace res {

constexpr int kNT = 512, kNW = kNT / 64;

constexpr int pow2_at_least(int v) { return v <= 1 ? 1 : 2 * pow2_at_least((v + 1) / 2); }

// Reduction buffers: two, used in turn, so that one barrier per reduction is
// enough (a wave writes a buffer again only after the barrier of the reduction
// in between, which every wave reaches after its last read).
template <int KM>
struct Lds {
  static constexpr int NP = (KM - 2) * (KM - 3) / 2 > 0 ? (KM - 2) * (KM - 3) / 2 : 1;  // Gram pairs
  static constexpr int NG = (NP + 63) / 64 * 64;
  static constexpr int NV = pow2_at_least(2 * KM);  // dots, Gram row and ||f||^2
  double part[2][kNW][NV + NG];
  double R[KM * KM], T[KM * KM];  // column-major
  double gram[NG], row[KM];
  double c[KM], s[KM];
};

// v[0:N] summed over the wave into dst[0:N]
template <int N>
__device__ __forceinline__ void wave_part(double (&v)[N], double* dst) {
  const int lane = threadIdx.x & 63;
  const double r = multi_reduce<N>(v);
  if (lane < N) dst[lane] = r;
}

// value `at` summed over the waves
template <int S>
__device__ __forceinline__ double total(const double (&part)[kNW][S], int at) {
  double a[kNW];
#pragma unroll
  for (int w = 0; w < kNW; ++w) a[w] = part[w][at];
  return ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
}

template <int R, int KM, int VAR>
__global__ __launch_bounds__(kNT) void k_step(StepArgs a) {
  __shared__ Lds<KM> L;
  constexpr int NV = Lds<KM>::NV;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int n = (int)a.n, cap = a.sm.cap, k = a.k;
  const Small& sm = a.sm;
  int buf = 0;

  // every load of the iteration but the history's
  double x[R], g[R], f[R], v[R], dg[R], Q[KM][R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int p = t + r * kNT;
    const bool in = p < n;
    x[r] = in ? a.x[p] : 0.0;
    g[r] = in ? a.g[p] : 0.0;
    v[r] = in && !a.first ? a.f_prev[p] : 0.0;
    dg[r] = in && !a.first ? a.g_prev[p] : 0.0;
#pragma unroll
    for (int j = 0; j < KM; ++j) Q[j][r] = in && j < k ? a.Q[p + (int64_t)j * a.ld] : 0.0;
  }
  if (t < k * k) {
    L.R[t % k + t / k * KM] = sm.R[t % k + (t / k) * cap];
    if (VAR == AA_ICWY) L.T[t % k + t / k * KM] = sm.T[t % k + (t / k) * cap];
  }
  const bool ended = aa_stopped(sm);
  const int64_t cur = sm.stop->cur;
  const double res0 = sm.scal[S_RES0], step = sm.scal[S_STEP];
  auto put = [&](double* dst, const double (&src)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (t + r * kNT < n) dst[t + r * kNT] = src[r];
  };
  if (ended) {  // the iteration has ended: x_next = x
    if (a.xn != a.x) put(a.xn, x);
    return;
  }

  // history: f, Delta f (v), Delta g
#pragma unroll
  for (int r = 0; r < R; ++r) {
    f[r] = g[r] - x[r];
    v[r] = f[r] - v[r];
    dg[r] = g[r] - dg[r];
  }
  put(a.f_prev, f);
  put(a.g_prev, g);
  double ff = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) ff = fma(f[r], f[r], ff);
  auto reduce1 = [&](double s) {  // one value over the workgroup
    s = wave_sum(s);
    if (lane == 0) L.part[buf][w][0] = s;
    __syncthreads();
    const double r = total(L.part[buf], 0);
    buf ^= 1;
    return r;
  };
  if (a.first) {
    put(a.xn, g);
    const double r = reduce1(ff);
    if (t == 0) {
      sm.scal[S_RES] = sm.scal[S_RES0] = sm.scal[S_STEP] = r;
      sm.stop->cur = 1;
      a.state->m_i = 0;
    }
    return;
  }
  put(a.ring + (int64_t)a.slot * a.ld, dg);

  // QRDelete: Givens rotations from R by one wave (lane = column), applied to
  // this lane's rows
  const bool del = a.iter > a.m;
  const int kk = del ? k - 1 : k;
  __syncthreads();
  if (del && kk > 0) {
    if (w == 0) {
      const int col = lane < kk ? lane : 0;
      double top = L.R[(col + 1) * KM], nxt = L.R[1 + (col + 1) * KM];
      for (int j = 0; j < kk; ++j) {
        const double bot = nxt;
        if (j + 1 < kk) nxt = L.R[(j + 2) + (col + 1) * KM];
        const double p = lane_value(top, j), q = lane_value(bot, j);
        const double rho = hypot(p, q);
        const double c = rho > 0.0 ? p / rho : 1.0;
        const double s = rho > 0.0 ? q / rho : 0.0;
        const double keep = c * top + s * bot;
        top = -s * top + c * bot;
        // row j of the new R: column `lane`, whose old column lane + 1 has been
        // read to row j + 2 by every lane of this wave
        if (lane >= j && lane < kk) L.R[j + lane * KM] = keep;
        if (lane == 0) {
          L.c[j] = c;
          L.s[j] = s;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double top = Q[0][r];
#pragma unroll
      for (int j = 0; j < KM - 1; ++j)
        if (j < kk) {
          const double bot = Q[j + 1][r];
          Q[j][r] = L.c[j] * top + L.s[j] * bot;
          top = -L.s[j] * top + L.c[j] * bot;
        }
    }
  }
  // columns kk .. are no longer part of Q (their products are never used)

  // the first reduction: Q^T Delta f (MGS: q_0^T Delta f), the Gram row of
  // q_{kk-1} and, after a delete, the Gram of the columns before it (ICWY;
  // DCGS-2's row), ||f||^2; kk = 0: ||Delta f||^2
  const bool reorth = VAR == AA_DCGS2 && ((a.flags & AA_DCGS2_GUARD_GE3) ? kk >= 2 : kk > 2);
  double ql[R];
#pragma unroll
  for (int r = 0; r < R; ++r) ql[r] = 0.0;
  {
    double s[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) s[i] = 0.0;
#pragma unroll
    for (int j = 0; j < KM; ++j)
      if (j == kk - 1)
#pragma unroll
        for (int r = 0; r < R; ++r) ql[r] = Q[j][r];
#pragma unroll
    for (int j = 0; j < KM - 1; ++j)
      if (j < kk)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (VAR != AA_MGS || j == 0) s[j] = fma(Q[j][r], v[r], s[j]);
          if (VAR == AA_ICWY || VAR == AA_DCGS2) s[KM - 1 + j] = fma(Q[j][r], ql[r], s[KM - 1 + j]);
        }
    if (kk == 0)
#pragma unroll
      for (int r = 0; r < R; ++r) s[0] = fma(v[r], v[r], s[0]);
    s[NV - 1] = ff;
    wave_part<NV>(s, L.part[buf][w]);
  }
  if (VAR == AA_ICWY && del) {
    // pairs a (a - 1) / 2 + b, b < a < kk - 1, 64 at a time
    auto pairs = [&](auto C0) {
      constexpr int c0 = decltype(C0)::value;
      if constexpr (c0 < Lds<KM>::NP) {
        constexpr int NC = pow2_at_least(Lds<KM>::NP - c0 < 64 ? Lds<KM>::NP - c0 : 64);
        double s[NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) s[i] = 0.0;
#pragma unroll
        for (int i = 1; i < KM - 2; ++i)
#pragma unroll
          for (int j = 0; j < i; ++j) {
            const int p = i * (i - 1) / 2 + j - c0;
            if (p >= 0 && p < NC && i < kk - 1)
#pragma unroll
              for (int r = 0; r < R; ++r) s[p] = fma(Q[i][r], Q[j][r], s[p]);
          }
        wave_part<NC>(s, L.part[buf][w] + NV + c0);
      }
    };
    pairs(std::integral_constant<int, 0>{});
    pairs(std::integral_constant<int, 64>{});
    pairs(std::integral_constant<int, 128>{});
    static_assert(Lds<KM>::NP <= 192, "pair chunks");
  }
  __syncthreads();
  const auto& part = L.part[buf];
  buf ^= 1;
  const double res2 = total(part, NV - 1);
  const bool hit = a.stop_mode == kStopResidual ? sqrt(res2) <= a.stop_tol * sqrt(res0)
                                                : a.stop_mode == kStopStep && sqrt(step) < a.stop_tol;
  if (t == 0) {
    sm.scal[S_RES] = res2;
    if (hit) {
      sm.stop->iter = cur;
      sm.stop->k = k;
      sm.stop->m_i = a.m_prev;
      sm.stop->done = AA_STOPPED_TEST;
    } else {
      sm.stop->cur = cur + 1;
    }
  }
  if (hit) {  // the test held at the start of this iteration: x_next = x_i
    if (a.xn != a.x) put(a.xn, x);
    return;
  }

  // QRAdd.  cf: this lane's entry of column kk of R (lane j: R_{j,kk}).
  double cf = lane < kk ? total(part, lane) : 0.0, nrm2 = 0.0;
  // w = v - sum_{j < kc} Q_j c_j
  auto subtract = [&](double (&o)[R], double c, int kc) {
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0;
#pragma unroll
    for (int j = 0; j < KM - 1; ++j)
      if (j < kc) {
        const double cj = lane_value(c, j);
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = fma(Q[j][r], cj, acc[r]);
      }
#pragma unroll
    for (int r = 0; r < R; ++r) o[r] -= acc[r];
  };
  auto norm2 = [&] {
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) s = fma(v[r], v[r], s);
    return reduce1(s);
  };
  // Q^T y over kc columns, lane j: column j
  auto dots = [&](const double (&y)[R], int kc) {
    constexpr int ND = pow2_at_least(KM);
    double s[ND];
#pragma unroll
    for (int i = 0; i < ND; ++i) s[i] = 0.0;
#pragma unroll
    for (int j = 0; j < KM; ++j)
      if (j < kc)
#pragma unroll
        for (int r = 0; r < R; ++r) s[j] = fma(Q[j][r], y[r], s[j]);
    wave_part<ND>(s, L.part[buf][w]);
    __syncthreads();
    const double o = lane < kc ? total(L.part[buf], lane) : 0.0;
    buf ^= 1;
    return o;
  };
  if (kk == 0) {
    nrm2 = total(part, 0);
    cf = 0.0;
  } else if (VAR == AA_MGS) {
    double rj = total(part, 0);
    cf = lane == 0 ? rj : 0.0;
#pragma unroll
    for (int j = 0; j < KM - 1; ++j)
      if (j < kk) {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] -= Q[j][r] * rj;
        if (j + 1 < kk) {
          double s = 0.0;
#pragma unroll
          for (int r = 0; r < R; ++r) s = fma(Q[j + 1][r], v[r], s);
          rj = reduce1(s);
          if (lane == j + 1) cf = rj;
        }
      }
    nrm2 = norm2();
  } else if (VAR == AA_CGS2) {
    subtract(v, cf, kk);
    const double z = dots(v, kk);
    subtract(v, z, kk);
    cf += z;
    nrm2 = norm2();
  } else if (VAR == AA_ICWY) {
    // T: the last row from this reduction, the others from the Gram (delete)
    // or from memory.  Every wave writes the same values and reads its own.
    if (lane < kk - 1) L.row[lane] = total(part, KM - 1 + lane);
    if (del)
      for (int p = lane; p < (kk - 1) * (kk - 2) / 2; p += 64) L.gram[p] = total(part, NV + p);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double tr[KM];
#pragma unroll
    for (int b = 0; b < KM - 1; ++b) {
      tr[b] = 0.0;
      if (b < kk - 1 && lane > b && lane < kk)
        tr[b] = lane == kk - 1 ? L.row[b] : del ? L.gram[lane * (lane - 1) / 2 + b]
                                                : L.T[lane + b * KM];
    }
#pragma unroll
    for (int b = 0; b < KM - 1; ++b)
      if (b < kk - 1) {
        cf -= tr[b] * lane_value(cf, b);  // tr is zero in the lanes up to b
      }
    if (w == 0 && lane < kk)
#pragma unroll
      for (int b = 0; b < KM - 1; ++b)
        if (b < lane && (del || lane == kk - 1)) sm.T[lane + (size_t)b * cap] = tr[b];
    subtract(v, cf, kk);
    nrm2 = norm2();
  } else {  // DCGS-2: q_{p} -= Q s first (p = kk - 1), v - Q c with the new q_p
    const int p = kk - 1;
    if (reorth) {
      const double s = lane < p ? total(part, KM - 1 + lane) : 0.0;
      const double scale = (a.flags & AA_DCGS2_LITERAL) ? 1.0 : L.R[p + p * KM];
      subtract(ql, s, p);
      if (w == 0 && lane < p) L.R[lane + p * KM] += scale * s;
    }
    subtract(v, cf, p);
    const double cp = lane_value(cf, p);
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] -= ql[r] * cp;
#pragma unroll
    for (int j = 0; j < KM; ++j)
      if (j == p)
#pragma unroll
        for (int r = 0; r < R; ++r) Q[j][r] = ql[r];
    nrm2 = norm2();
  }
  const double nv = sqrt(nrm2);
  const double col = nv * nv + wave_sum(cf * cf);
  // breakdown: as run_tail's TAIL_NORM
  const bool bad = !(nv > kBreakdownRel * sqrt(col)) || !isfinite(nv);
  const int k1 = kk + 1;
#pragma unroll
  for (int j = 0; j < KM; ++j)
    if (j == kk)
#pragma unroll
      for (int r = 0; r < R; ++r) Q[j][r] = v[r] / nv;
  // column kk of R (every wave writes the same values); the other columns were
  // final before the last barrier
  if (lane < k1) L.R[lane + kk * KM] = lane == kk ? nv : cf;

  // R gamma = Q^T f
  double c = dots(f, k1);
#pragma unroll
  for (int j = 0; j < KM; ++j)
    if (j < k1 && (del || j == kk || (reorth && j == kk - 1)))
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (t + r * kNT < n) a.Q[t + r * kNT + (int64_t)j * a.ld] = Q[j][r];
  // the history's loads, under the back substitution
  double h[KM][R];
#pragma unroll
  for (int j = 0; j < KM - 1; ++j)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int p = t + r * kNT;
      int sl = a.slot0 + j;
      sl -= sl >= a.m ? a.m : 0;
      h[j][r] = j < a.m_i - 1 && p < n ? a.ring[p + (int64_t)sl * a.ld] : 0.0;
    }
  double rr[KM], gam = 0.0;
#pragma unroll
  for (int b = 0; b < KM; ++b) rr[b] = b < k1 && lane < k1 ? L.R[lane + b * KM] : 0.0;
  if (w == 0 && lane < k1) sm.coef1[lane] = c;
#pragma unroll
  for (int b = KM - 1; b >= 0; --b)
    if (b < k1) {
      const double gb = lane_value(c, b) / lane_value(rr[b], b);
      if (lane < b) c -= rr[b] * gb;
      if (lane == b) gam = gb;
    }
  if (t < k1 * k1) {
    const int i = t % k1, j = t / k1;
    sm.R[i + (size_t)j * cap] = i <= j ? L.R[i + j * KM] : 0.0;
  }
  if (w == 0 && lane < k1) sm.gamma[lane] = gam;
  if (t == 0) {
    a.state->m_i = a.m_i;
    if (bad) {  // x_{i+1} = G(x_i), and the iteration ends here
      *sm.status = AA_EBREAKDOWN;
      sm.stop->iter = cur;
      sm.stop->k = k1;
      sm.stop->m_i = a.m_i;
      sm.stop->done = AA_STOPPED_BREAKDOWN;
    }
  }
  if (bad) {
    put(a.xn, g);
    return;
  }
  // x_{i+1} = g - sum gamma_j Delta g_j (the newest Delta g still in registers)
  double d2 = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < KM - 1; ++j)
      if (j < a.m_i - 1) s = fma(h[j][r], lane_value(gam, j), s);
    s = fma(dg[r], lane_value(gam, a.m_i - 1), s);
    const double xn = g[r] - s, d = xn - x[r];
    d2 = fma(d, d, d2);
    x[r] = xn;
  }
  put(a.xn, x);
  const double sd = reduce1(d2);
  if (t == 0) sm.scal[S_STEP] = sd;
}

template <int R, int KM>
hipError_t launch_shape(const StepArgs& a, int variant, hipStream_t st) {
  const dim3 one(1), wg(kNT);
  switch (variant) {
    case AA_MGS: hipLaunchKernelGGL((k_step<R, KM, AA_MGS>), one, wg, 0, st, a); break;
    case AA_CGS2: hipLaunchKernelGGL((k_step<R, KM, AA_CGS2>), one, wg, 0, st, a); break;
    case AA_DCGS2: hipLaunchKernelGGL((k_step<R, KM, AA_DCGS2>), one, wg, 0, st, a); break;
    case AA_ICWY: hipLaunchKernelGGL((k_step<R, KM, AA_ICWY>), one, wg, 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace res

// Shapes: at most 40 doubles of Q per lane, which with the iteration's other
// vectors fills the 256 registers of a lane of eight resident waves.  (DCGS-2
// keeps one more vector, the column it reorthogonalizes: its widest instance, 8
// rows a lane and 5 columns, spills 104 registers and takes 29 us where the
// other variants take 20 to 21 in the same trace; the step with its vectors in
// memory took 46.  No other instance spills vector registers.)
bool resident_fits(int64_t n, int m) {
  return (n <= 1024 && m <= 20) || (n <= 2048 && m <= 10) || (n <= 4096 && m <= 5);
}

hipError_t launch_resident(const StepArgs& a, int variant, hipStream_t st) {
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  if (!resident_fits(a.n, a.m) || a.k > a.m) return hipErrorInvalidValue;
  if (a.n <= 512) return a.m <= 8 ? res::launch_shape<1, 8>(a, variant, st)
                                  : res::launch_shape<1, 20>(a, variant, st);
  if (a.n <= 1024) return a.m <= 8 ? res::launch_shape<2, 8>(a, variant, st)
                                   : res::launch_shape<2, 20>(a, variant, st);
  if (a.n <= 2048) return res::launch_shape<4, 10>(a, variant, st);
  return res::launch_shape<8, 5>(a, variant, st);
}

}  // namespace aa
