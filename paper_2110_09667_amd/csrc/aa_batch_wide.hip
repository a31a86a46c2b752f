// aa_batch_wide.hip -- batched iterations with many workgroups per instance.
//
// The persistent kernel of aa_batch.hip gives an instance one workgroup, which
// streams some 20 GB/s: a batch then takes as long as its largest instance
// (10 ms at n = 262144, m = 20) unless thousands share the chip.  Here every
// pass of the iteration is one launch over the chunks of all such ("wide")
// instances, each workgroup running the pass bodies of aa_passes.h on its
// chunk's tiles and publishing partial sums, and one finalize launch with a
// workgroup per instance sums them and runs the dense tail.  The kernel
// boundaries order the passes, whatever XCD a chunk ran on.  512 instances of
// side 32 to 512 (ICWY, both fusions): 7.2 -> 2.6 ms an iteration.
//
// Which passes an instance takes is read from its state on the device, so the
// launches of an iteration are the same every time and can be replayed as a
// graph; a pass an instance does not take costs its workgroups an early
// return.  BState.pending marks an iteration in progress between the launches:
// kRun, or kFirst for i = 0 (x_1 = G(x_0)); zero outside.
#include <math.h>

#include "aa_passes.h"

namespace aa {
namespace wide {

enum : int { kRun = 1, kFirst = 2 };

// Phases of an iteration, each a pass kernel and the finalize that follows it.
enum Phase : int { PH_HISTORY, PH_ROTATE, PH_DOTS, PH_CGS2B, PH_MGS, PH_UPDATE, PH_RHS, PH_X };

__device__ __forceinline__ Tail mk_tail(int op, int k) {
  Tail t{};
  t.op = op;
  t.k = k;
  return t;
}

// What an instance does in its current iteration (as wg_front of aa_batch.hip
// decides it).  k: columns on entry, kk: after QRDelete.
struct Plan {
  int m, m_i, k, kk;
  bool del, dfuse, folded;
  const double* fr;  // AA_FUSE_RHS: f_i joins the QRAdd passes
  double* slot;      // column kk
};

__device__ __forceinline__ Plan plan_of(const WideArgs& a, const BInst& I, const BState& st) {
  Plan p;
  p.m = I.m;
  p.m_i = (int)(st.iter < I.m ? st.iter : I.m);
  p.k = st.k;
  p.del = st.iter > I.m;
  p.kk = p.del ? p.k - 1 : p.k;
  p.fr = (a.flags & AA_FUSE_RHS) && a.variant != AA_MGS && I.m + 1 <= 64 ? I.f_prev : nullptr;
  p.folded = p.fr && p.kk >= 1;
  p.dfuse = p.del && (a.flags & AA_FUSE_DELETE) && a.variant != AA_MGS && p.k >= 2 &&
            p.k - 1 + (p.fr ? 2 : 1) <= a.kgram;
  p.slot = I.Q + (int64_t)p.kk * I.ld;
  return p;
}

// QRDelete's rotation pass (ICWY: with the Gram of T; fused: with the QRAdd's
// first products).  False if there is none.
__device__ __forceinline__ bool rotate_args(const WideArgs& a, const BInst& I, const Plan& p,
                                            RotArgs& r) {
  if (!p.del || p.k <= 1) return false;
  r = RotArgs{I.Q, I.ld, I.n, p.k, I.sm.givens, 0, nullptr, nullptr, 0, 0};
  if (p.dfuse) {
    r.gram = 1;
    r.v = I.W;
    r.f = p.fr;
    r.naug = p.fr ? 2 : 1;
  } else if (a.variant == AA_ICWY) {
    r.gram = 1;
    r.drop_last = 1;
  }
  return true;
}

__device__ __forceinline__ bool reorth_at(const WideArgs& a, int kk) {
  return (a.flags & AA_DCGS2_GUARD_GE3) ? kk >= 2 : kk > 2;
}

// The tail of the QRAdd's first reduction and where Q^T f sits in it.
__device__ __forceinline__ Tail first_tail(const WideArgs& a, const Plan& p) {
  Tail t = mk_tail(TAIL_ICWY, p.kk);
  t.rhs = p.folded ? 1 : 0;
  if (p.kk == 0) {
    t.op = TAIL_NORM;
    t.rhs = 0;
  } else if (a.variant == AA_MGS) {
    t.op = TAIL_MGS_R;
  } else if (a.variant == AA_CGS2) {
    t.op = TAIL_CGS2_S;
    t.zoff = p.kk;
  } else if (a.variant == AA_ICWY) {
    t.zoff = 2 * p.kk - 1;
  } else {
    t.op = TAIL_DCGS2;
    t.reorth = reorth_at(a, p.kk) ? 1 : 0;
    t.literal = (a.flags & AA_DCGS2_LITERAL) ? 1 : 0;
    t.zoff = p.kk + (t.reorth ? p.kk - 1 : 0);
  }
  return t;
}

// The QRAdd's first products (none where the rotation pass formed them).
__device__ __forceinline__ bool first_args(const WideArgs& a, const BInst& I, const Plan& p,
                                           DotsArgs& d) {
  if (p.dfuse) return false;
  d = DotsArgs{I.Q, I.ld, I.n, I.W, 0, nullptr, 0, 0, nullptr, 0, 0};
  if (p.kk == 0) {
    d.xx = 1;
    return true;
  }
  d.nx = a.variant == AA_MGS ? 1 : p.kk;
  if (a.variant == AA_ICWY || (a.variant == AA_DCGS2 && reorth_at(a, p.kk))) {
    d.y = I.Q + (int64_t)(p.kk - 1) * I.ld;
    d.ny = p.kk - 1;
  }
  if (p.folded) {
    d.z = p.fr;
    d.nz = p.kk;
  }
  return true;
}

// MGS step j (1 <= j < kk): subtract q_{j-1}, then q_j^T w.
__device__ __forceinline__ bool mgs_args(const BInst& I, const Plan& p, int j, UpdArgs& u) {
  if (j >= p.kk) return false;
  u = UpdArgs{};
  u.Q = I.Q; u.ldq = I.ld; u.n = I.n; u.Qw = I.Q; u.dcgs2_p = -1;
  u.v = I.W; u.out = I.W; u.j0 = j - 1; u.nc = 1;
  u.c1 = I.sm.R + (size_t)p.kk * I.sm.cap;
  u.dotcol = j;
  u.rev = j & 1;
  return true;
}

// The QRAdd's last pass: w into column kk, its norm (and w^T f).
__device__ __forceinline__ bool update_args(const WideArgs& a, const BInst& I, const Plan& p,
                                            UpdArgs& u) {
  if (p.kk == 0) return false;
  double* Rcol = I.sm.R + (size_t)p.kk * I.sm.cap;
  u = UpdArgs{};
  u.Q = I.Q; u.ldq = I.ld; u.n = I.n; u.Qw = I.Q; u.dotcol = -1; u.dcgs2_p = -1;
  u.v = I.W; u.out = p.slot; u.j0 = 0; u.nc = p.kk; u.c1 = I.sm.coef0; u.nrm = 1;
  u.rev = 1;
  if (p.folded) u.rhsv = p.fr;
  if (a.variant == AA_MGS) {
    u.j0 = p.kk - 1; u.nc = 1; u.c1 = Rcol; u.rev = p.kk & 1;
  } else if (a.variant == AA_CGS2) {
    u.c2 = I.sm.coef1; u.rev = 0;
  } else if (a.variant == AA_DCGS2) {
    u.c1 = Rcol;
    if (reorth_at(a, p.kk)) {
      u.dcgs2_p = p.kk - 1; u.reorth = 1; u.s = I.sm.coef1; u.nc = p.kk - 1;
    }
  }
  return true;
}

__device__ __forceinline__ bool rhs_args(const BInst& I, const Plan& p, DotsArgs& d) {
  if (p.folded) return false;
  d = DotsArgs{I.Q, I.ld, I.n, I.f_prev, p.kk + 1, nullptr, 0, 0, nullptr, 0, 0};
  return true;
}

// This workgroup's sums to the instance's partials ([value][chunk]).
__device__ __forceinline__ void publish(const BInst& I, const WideItem& w, int nred,
                                        const double* acc, int stride) {
  __syncthreads();
  for (int c = threadIdx.x; c < nred; c += kWG) {
    double s = acc[c];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) s += acc[v * stride + c];
    I.sm.partials[(size_t)c * w.chunks + w.chunk] = s;
  }
}

// G(x) (unless an accepted candidate left it in I.g) and the history in one
// pass: G is used in registers and kept as g_prev.  i = 0: f_0 and G(x_0) only
// (x_1 is written by the last pass: neighbours read x_0 here).
__global__ __launch_bounds__(kWG) void k_history(WideArgs a) {
  __shared__ double s_acc[kWaves];
  const WideItem w = a.items[blockIdx.x];
  const BInst& I = a.inst[w.j];
  const BState st = a.state[w.j];
  if (!st.active) return;
  const int lane = threadIdx.x & 63;
  const bool first = st.iter == 0, known = st.g_valid != 0;
  const int n = (int)I.n, s = (int)I.s, dim = I.dim, s2 = s * s;
  const double ih2 = 1.0 / (I.h * I.h), omega = I.omega, c = I.c;
  const double *u = I.x, *fm = I.f, *gk = I.g;
  double* dg = first ? nullptr : I.ring + (int64_t)((st.iter - 1) % I.m) * I.ld;
  auto g_at = [&](int p, int ix, int iy, int iz, double up, double fp) {
    double nb = 0.0;
    if (ix > 0) nb += u[p - 1];
    if (ix < s - 1) nb += u[p + 1];
    if (dim >= 2) {
      if (iy > 0) nb += u[p - s];
      if (iy < s - 1) nb += u[p + s];
    }
    if (dim >= 3) {
      if (iz > 0) nb += u[p - s2];
      if (iz < s - 1) nb += u[p + s2];
    }
    const double au = (2.0 * dim * up - nb) * ih2;
    return up - omega * (au + c * up * up * up - fp);
  };
  double sff = 0.0;
  for_tiles(I.n, w.chunk, w.chunks, [&](int64_t b2, auto full) {
    constexpr bool F = decltype(full)::value;
    double2 xv[kPairs], gv[kPairs], f[kPairs], fp[kPairs], gp[kPairs];
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {  // x is read again by neighbours: ordinary loads
      const int64_t row = b2 + (int64_t)i * 2 * kWG;
      if (F) {
        xv[i] = *reinterpret_cast<const double2*>(u + row);
      } else {
        xv[i].x = row < n ? u[row] : 0.0;
        xv[i].y = row + 1 < n ? u[row + 1] : 0.0;
      }
    }
    if (known) ld2<F>(gv, gk, b2, I.n);
    else ld2<F>(gv, fm, b2, I.n);
    if (!first) {
      ld2<F>(fp, I.f_prev, b2, I.n);
      ld2<F>(gp, I.g_prev, b2, I.n);
    }
    if (!known) {
#pragma unroll
      for (int i = 0; i < kPairs; ++i) {
        const int row = (int)b2 + i * 2 * kWG;
        const int q = row / s, ix = row - q * s, iz = dim >= 3 ? q / s : 0, iy = q - iz * s;
        gv[i].x = F || row < n ? g_at(row, ix, iy, iz, xv[i].x, gv[i].x) : 0.0;
        // the next point: same row of the grid, or the first of the next one
        const int x1 = ix + 1 < s ? ix + 1 : 0, y1 = x1 ? iy : (dim >= 3 && iy + 1 == s ? 0 : iy + 1);
        const int z1 = dim >= 3 && x1 == 0 && y1 == 0 ? iz + 1 : iz;
        gv[i].y = F || row + 1 < n ? g_at(row + 1, x1, y1, z1, xv[i].y, gv[i].y) : 0.0;
      }
    }
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
      f[i] = make_double2(gv[i].x - xv[i].x, gv[i].y - xv[i].y);
      if (!first) {
        fp[i] = make_double2(f[i].x - fp[i].x, f[i].y - fp[i].y);
        gp[i] = make_double2(gv[i].x - gp[i].x, gv[i].y - gp[i].y);
      }
    }
    if (!first) {
      st2<F>(fp, I.W, b2, I.n);
      st2<F>(gp, dg, b2, I.n);
    }
    st2<F>(f, I.f_prev, b2, I.n);
    st2<F>(gv, I.g_prev, b2, I.n);
    sff += dot2(f, f);
  });
  const double p = wave_sum(sff);
  if (lane == 0) s_acc[threadIdx.x >> 6] = p;
  publish(I, w, 1, s_acc, 1);
}

extern __shared__ double s_dyn[];  // Gram staging, then the waves' pair sums

// KB: window bucket of the batch (KG = max(16, KB) columns of the Gram).
template <int KB, bool GRAM>
__global__ __launch_bounds__(kWG) void k_rotate(WideArgs a) {
  constexpr int KG = KB < 16 ? 16 : KB;
  __shared__ double s_c[KG], s_s[KG];
  const WideItem w = a.items[blockIdx.x];
  const BInst& I = a.inst[w.j];
  const BState st = a.state[w.j];
  if (st.pending != kRun) return;
  const Plan p = plan_of(a, I, st);
  RotArgs r;
  if (!rotate_args(a, I, p, r)) return;
  givens_coefs(r, I.sm.cap, s_c, s_s, KG);
  __syncthreads();
  if constexpr (GRAM) {
    if (r.gram) {
      const int na = gram_cols(r), np = na * (na - 1) / 2;
      if (r.k - 1 + r.naug <= 8) {
        double acc[32];
        rotate_gram_small_body<8>(r, s_c, s_s, w.chunk, w.chunks, acc);
        const double v = multi_reduce<32>(acc);
        const int lane = threadIdx.x & 63;
        if (lane < np) s_dyn[(threadIdx.x >> 6) * np + lane] = v;
      } else {
        v4d acc[GramShape<KG>::NBP];
        rotate_gram_body<KG>(r, s_c, s_s, w.chunk, w.chunks, s_dyn, gram_stride(na), acc);
        __syncthreads();
        gram_store<KG>(acc, s_dyn + (threadIdx.x >> 6) * np, na);
      }
      publish(I, w, np, s_dyn, np);
      return;
    }
  }
  // (a tile of this body is 512 rows: twice the chunk's tiles)
  rotate_body(r, s_c, s_s, w.chunk, w.chunks);
}

template <int KB, int NR>
__global__ __launch_bounds__(kWG) void k_dots(WideArgs a, int rhs) {
  constexpr int STR = NR * KB + 2;
  __shared__ double s_acc[kWaves * STR];
  const WideItem w = a.items[blockIdx.x];
  const BInst& I = a.inst[w.j];
  const BState st = a.state[w.j];
  if (st.pending != kRun) return;
  const Plan p = plan_of(a, I, st);
  DotsArgs d;
  if (rhs ? !rhs_args(I, p, d) : !first_args(a, I, p, d)) return;
  lds_zero(s_acc, kWaves * STR);
  __syncthreads();
  // (beyond 96 running sums a lane the registers do not hold them)
  if constexpr (NR * KB <= 96)
    dots_reg_body<KB, NR>(d, w.chunk, w.chunks, s_acc + (threadIdx.x >> 6) * STR);
  else
    dots_body(d, w.chunk, w.chunks, s_acc + (threadIdx.x >> 6) * STR);
  publish(I, w, dots_nred(d), s_acc, STR);
}

template <int KB>
__global__ __launch_bounds__(kWG) void k_cgs2b(WideArgs a) {
  __shared__ double s_s[KB], s_acc[kWaves * KB];
  const WideItem w = a.items[blockIdx.x];
  const BInst& I = a.inst[w.j];
  const BState st = a.state[w.j];
  if (st.pending != kRun) return;
  const Plan p = plan_of(a, I, st);
  if (p.kk == 0) return;
  for (int j = threadIdx.x; j < KB; j += kWG) s_s[j] = j < p.kk ? I.sm.coef0[j] : 0.0;
  lds_zero(s_acc, kWaves * KB);
  __syncthreads();
  const Cgs2bArgs b{I.Q, I.ld, I.n, I.W, p.kk, I.sm.coef0, 1};
  if constexpr (KB <= 32)
    cgs2b_pair_body<KB, (KB <= 16 ? kPairs : 1)>(b, s_s, w.chunk, w.chunks,
                                                 s_acc + (threadIdx.x >> 6) * KB);
  else
    cgs2b_body<KB>(b, s_s, w.chunk, w.chunks, s_acc + (threadIdx.x >> 6) * KB);
  publish(I, w, p.kk, s_acc, KB);
}

// mgs >= 1: MGS step; 0: the last pass
__global__ __launch_bounds__(kWG) void k_update(WideArgs a, int mgs) {
  __shared__ double s_c1[kMaxCols], s_c2[kMaxCols], s_s[kMaxCols], s_acc[kWaves * 4];
  const WideItem w = a.items[blockIdx.x];
  const BInst& I = a.inst[w.j];
  const BState st = a.state[w.j];
  if (st.pending != kRun) return;
  const Plan p = plan_of(a, I, st);
  UpdArgs u;
  if (mgs ? !mgs_args(I, p, mgs, u) : !update_args(a, I, p, u)) return;
  update_coefs(u, s_c1, s_c2, s_s);
  lds_zero(s_acc, kWaves * 4);
  __syncthreads();
  update_body(u, s_c1, s_c2, s_s, w.chunk, w.chunks, s_acc + (threadIdx.x >> 6) * 4);
  publish(I, w, update_nred(u), s_acc, 4);
}

__global__ __launch_bounds__(kWG) void k_scale(WideArgs a) {
  const WideItem w = a.items[blockIdx.x];
  const BInst& I = a.inst[w.j];
  const BState st = a.state[w.j];
  if (st.pending != kRun) return;
  const Plan p = plan_of(a, I, st);
  scale_body(p.kk == 0 ? I.W : p.slot, p.slot, I.n, I.sm.R[p.kk + (size_t)p.kk * I.sm.cap], w.chunk,
             w.chunks);
}

// An instance of the split policy (a.split) that breaks down ends in this
// iteration with x_{i+1} = G(x_i); any other goes on and is ended by the next
// iteration's test.
__device__ __forceinline__ bool broken_now(const WideArgs& a, const BInst& I, int j) {
  return a.split[j] == kWideSplit && *I.sm.status != AA_OK;
}

__global__ __launch_bounds__(kWG) void k_xupdate(WideArgs a) {
  __shared__ double s_g[kMaxCols], s_acc[kWaves];
  __shared__ int s_slot[kMaxCols];
  const WideItem w = a.items[blockIdx.x];
  const BInst& I = a.inst[w.j];
  const BState st = a.state[w.j];
  if (st.pending == 0) return;
  if (st.pending == kFirst || broken_now(a, I, w.j)) {  // x_{i+1} = G(x_i)
    for_tiles(I.n, w.chunk, w.chunks, [&](int64_t b2, auto full) {
      constexpr bool F = decltype(full)::value;
      double2 v[kPairs];
      ld2<F>(v, I.g_prev, b2, I.n);
      st2<F>(v, I.x, b2, I.n);
    });
    return;
  }
  const Plan p = plan_of(a, I, st);
  const XupdArgs x{I.ring, I.ld, p.m, (int)((st.iter - p.m_i) % p.m), p.m_i, I.g_prev, I.x, I.x,
                   I.n, I.sm.gamma};
  xupdate_coefs(x, s_g, s_slot);
  lds_zero(s_acc, kWaves);
  __syncthreads();
  xupdate_body(x, s_g, s_slot, w.chunk, w.chunks, s_acc + (threadIdx.x >> 6));
  publish(I, w, 1, s_acc, 1);
}

// --------------------------------------------------------------------------
// finalize: one workgroup per instance
// --------------------------------------------------------------------------

// red[c] = sum over the chunks, in a fixed order: a thread per value while the
// chunks are few (eight loads in flight), a wave per value otherwise.
__device__ void sum_chunks(const BInst& I, int chunks, int nred, double* red) {
  if (chunks <= 64) {
    for (int c = threadIdx.x; c < nred; c += kWG) {
      const double* q = I.sm.partials + (size_t)c * chunks;
      double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
      int g = 0;
      for (; g + 8 <= chunks; g += 8)
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u] += q[g + u];
      for (int u = 0; g < chunks; ++g, ++u) s[u] += q[g];
      red[c] = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    }
  } else {
    const int lane = threadIdx.x & 63;
    for (int c0 = (threadIdx.x >> 6) * 4; c0 < nred; c0 += kWaves * 4) {
      double s[4] = {0.0, 0.0, 0.0, 0.0};
      for (int g = lane; g < chunks; g += 64)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (c0 + u < nred) s[u] += I.sm.partials[(size_t)(c0 + u) * chunks + g];
      const double r = multi_reduce<4>(s);
      if (lane < 4 && c0 + lane < nred) red[c0 + lane] = r;
    }
  }
  __syncthreads();
}

__global__ __launch_bounds__(kWG) void k_finalize(WideArgs a, int phase, int mgs) {
  __shared__ double red[kMaxRedAll], red2[kMaxRed];
  const WideItem w = a.list[blockIdx.x];
  const int j = w.j;
  const BInst& I = a.inst[j];
  const Small& sm = I.sm;
  BState st = a.state[j];
  if (phase == PH_HISTORY) {
    if (!st.active) return;
    sum_chunks(I, w.chunks, 1, red);
    const double res = sqrt(red[0]);
    if (!st.g_valid) st.g_evals += 1;
    st.g_valid = 0;
    st.res_norm = res;
    if (st.iter == 0) {
      st.res0_norm = res;
      st.pending = kFirst;
      if (threadIdx.x == 0) {
        sm.scal[S_RES] = sm.scal[S_RES0] = sm.scal[S_STEP] = red[0];
        a.state[j] = st;
      }
      return;
    }
    st.status = *sm.status;
    const bool end =
        res <= a.tol * st.res0_norm || st.iter >= a.max_iter || st.status != AA_OK;
    if (end) {
      st.active = 0;
      st.conv_iter = st.iter;
    } else {
      st.pending = kRun;
    }
    if (threadIdx.x == 0) {
      sm.scal[S_RES] = red[0];
      a.state[j] = st;
    }
    if (!end && st.iter > I.m && st.k > 1) givens_body(sm, st.k, s_dyn);
    return;
  }
  if (phase == PH_X) {
    if (st.pending == 0) return;
    if (st.pending == kFirst) {
      st.iter = 1;
      st.m_i = 0;
    } else {
      const Plan p = plan_of(a, I, st);
      st.k = p.kk + 1;
      st.m_i = p.m_i;
      st.status = *sm.status;
      if (broken_now(a, I, j)) {
        st.active = 0;
        st.conv_iter = st.iter;
      } else {
        sum_chunks(I, w.chunks, 1, red);
        if (threadIdx.x == 0) sm.scal[S_STEP] = red[0];
        st.iter += 1;
      }
    }
    st.pending = 0;
    if (threadIdx.x == 0) a.state[j] = st;
    return;
  }
  if (st.pending != kRun) return;
  const Plan p = plan_of(a, I, st);
  if (phase == PH_ROTATE) {
    RotArgs r;
    if (!rotate_args(a, I, p, r) || !r.gram) return;
    const int na = gram_cols(r);
    sum_chunks(I, w.chunks, na * (na - 1) / 2, red);
    if (a.variant == AA_ICWY) {
      run_tail(sm, mk_tail(TAIL_GRAM, p.dfuse ? p.kk : na), red);
      __syncthreads();
    }
    if (!p.dfuse) return;
    // the pairs laid out as the QRAdd's first pass would have reduced them
    const Tail t = first_tail(a, p);
    const int kk = p.kk;
    const bool row = t.op == TAIL_ICWY || (t.op == TAIL_DCGS2 && t.reorth);
    const int pv = kk * (kk - 1) / 2, pf = (kk + 1) * kk / 2, prow = (kk - 1) * (kk - 2) / 2;
    for (int b = threadIdx.x; b < kk; b += kWG) {
      red2[b] = red[pv + b];
      if (row && b < kk - 1) red2[kk + b] = red[prow + b];
      if (p.fr) red2[t.zoff + b] = red[pf + b];
    }
    __syncthreads();
    run_tail(sm, t, red2);
    return;
  }
  if (phase == PH_DOTS) {
    DotsArgs d;
    if (!first_args(a, I, p, d)) return;
    sum_chunks(I, w.chunks, dots_nred(d), red);
    run_tail(sm, first_tail(a, p), red);
  } else if (phase == PH_CGS2B) {
    if (p.kk == 0) return;
    sum_chunks(I, w.chunks, p.kk, red);
    run_tail(sm, mk_tail(TAIL_CGS2_Z, p.kk), red);
  } else if (phase == PH_MGS) {
    UpdArgs u;
    if (!mgs_args(I, p, mgs, u)) return;
    sum_chunks(I, w.chunks, 1, red);
    Tail t = mk_tail(TAIL_MGS_R, p.kk);
    t.row = mgs;
    run_tail(sm, t, red);
  } else if (phase == PH_UPDATE) {
    UpdArgs u;
    if (!update_args(a, I, p, u)) return;
    sum_chunks(I, w.chunks, update_nred(u), red);
    Tail t = mk_tail(TAIL_NORM, p.kk);
    t.rhs = p.folded ? 1 : 0;
    run_tail(sm, t, red);
  } else {  // PH_RHS
    DotsArgs d;
    if (!rhs_args(I, p, d)) return;
    sum_chunks(I, w.chunks, p.kk + 1, red);
    run_tail(sm, mk_tail(TAIL_RHS, p.kk + 1), red);
  }
}

template <int KB>
void passes(const WideArgs& a, int nitems, int ninst, int mmax, bool gram, int stage_cols,
            hipStream_t st) {
  const dim3 g(nitems), b(kWG), gi(ninst);
  const size_t h = sizeof(double) * (size_t)(mmax * mmax);  // Givens scratch
  auto fin = [&](int phase, int mgs = 0) {
    hipLaunchKernelGGL(k_finalize, gi, b, phase == PH_HISTORY ? h : 0, st, a, phase, mgs);
  };
  const bool rhs = (a.flags & AA_FUSE_RHS) && a.variant != AA_MGS;
  const int nr = rhs ? 3 : a.variant == AA_ICWY || a.variant == AA_DCGS2 ? 2 : 1;
  hipLaunchKernelGGL(k_history, g, b, 0, st, a);
  fin(PH_HISTORY);
  if (mmax > 1) {
    if (gram) {
      const size_t l = sizeof(double) * (size_t)gram_lds_doubles(stage_cols > 8 ? stage_cols : 8);
      hipLaunchKernelGGL((k_rotate<KB, true>), g, b, l, st, a);
      fin(PH_ROTATE);
    } else {
      hipLaunchKernelGGL((k_rotate<KB, false>), g, b, 0, st, a);
    }
  }
  if (nr == 1) hipLaunchKernelGGL((k_dots<KB, 1>), g, b, 0, st, a, 0);
  else if (nr == 2) hipLaunchKernelGGL((k_dots<KB, 2>), g, b, 0, st, a, 0);
  else hipLaunchKernelGGL((k_dots<KB, 3>), g, b, 0, st, a, 0);
  fin(PH_DOTS);
  if (a.variant == AA_CGS2) {
    hipLaunchKernelGGL(k_cgs2b<KB>, g, b, 0, st, a);
    fin(PH_CGS2B);
  }
  if (a.variant == AA_MGS)
    for (int j = 1; j < mmax - 1; ++j) {
      hipLaunchKernelGGL(k_update, g, b, 0, st, a, j);
      fin(PH_MGS, j);
    }
  hipLaunchKernelGGL(k_update, g, b, 0, st, a, 0);
  fin(PH_UPDATE);
  hipLaunchKernelGGL(k_scale, g, b, 0, st, a);
  hipLaunchKernelGGL((k_dots<KB, 1>), g, b, 0, st, a, 1);
  fin(PH_RHS);
  hipLaunchKernelGGL(k_xupdate, g, b, 0, st, a);
  fin(PH_X);
}

}  // namespace wide

hipError_t launch_wide(const WideArgs& a, int nitems, int ninst, int kbucket, int mmax, bool gram,
                       int stage_cols, hipStream_t st) {
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  switch (kbucket) {
    case 8: wide::passes<8>(a, nitems, ninst, mmax, gram, stage_cols, st); break;
    case 16: wide::passes<16>(a, nitems, ninst, mmax, gram, stage_cols, st); break;
    case 32: wide::passes<32>(a, nitems, ninst, mmax, gram, stage_cols, st); break;
    case 64: wide::passes<64>(a, nitems, ninst, mmax, gram, stage_cols, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace aa
