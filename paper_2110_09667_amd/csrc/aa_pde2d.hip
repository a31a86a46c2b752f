// aa_pde2d.hip -- fixed-point maps of the paper's 2D test problems: the
// steady heat equation with a nonlinear term (Sec. 5.1, both terms) and the
// Bratu problem (Sec. 5.2).  Each evaluation G(u) = A^{-1} rhs(u) solves a
// Poisson system, A = -L_h the 5-point Dirichlet Laplacian on an N x N
// interior grid (x fastest, h = 1 / (N + 1)), by the preconditioned conjugate
// gradient with one geometric-multigrid V(1,1) cycle as the preconditioner:
// red-black Gauss-Seidel (red then black before the coarse correction, black
// then red after it, so the cycle is symmetric), full weighting, bilinear
// interpolation, coarse point I at fine point 2 I + 1, and coarse operators
// whose last row and column keep the boundary at its true distance h (the
// 1D Galerkin products; diagonal 1 + 2^level in units of 1/H^2).
//
// Scaled right-hand sides.  Every level works on b = H^2 r, which makes each
// step free of the spacing: red e = b / d, black e = (b + sum of red e) / d
// (d the diagonal in units of 1 / H^2), and after those two half-sweeps the
// residual is zero at the black points and (sum of black e) / H^2 at the red
// ones, so full weighting gives the next level's b as a weighted sum of black
// values alone.  Nothing but b needs keeping for the way up: the corrected red
// value is b / d + P e_c again.
//
// Layout and launches.  Every level's vectors are N_l x N_l row-major arrays
// in the workspace.  Levels of more than 64 points per side take one launch
// down (k_down: pre-smoothing and restriction) and one up (k_up: correction
// and post-smoothing), each a tile per workgroup with its halo recomputed in
// LDS; the levels from 64 points down run in one kernel of one workgroup with
// every array in LDS, the last ones (at most 8 points per side) as one
// precomputed matrix.  Grids of at most 96 points per side are solved by one
// launch of one workgroup (k_solve_small).  On the fine grid k_down also takes the conjugate
// gradient's update of x and r, and k_up gives r.z.  A PCG iteration at N =
// 1024 is 10 launches (23 when each half-sweep, each restriction and each
// vector update was one); the whole working set (~60 MB) stays in the Infinity
// Cache, so the launches are latency bound.
//
// Reductions (r.z, p.q, r.r): each workgroup stores its partial sum, and
// every workgroup of the kernel that needs the value sums all partials itself
// in one fixed order (the same value everywhere, deterministic).  No device-
// scope fence (on gfx950 a release fence writes the whole L2 back: with one
// per workgroup the vector kernels took 28 us instead of ~10) and no
// finalize launch.  The stopping test runs on the device at the start of each
// iteration; once it holds, every later kernel returns at once, so the host
// may enqueue iterations ahead and read the state only now and then.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include "aa_device.h"

namespace aa {
namespace pde {

constexpr int kBX = 256;           // threads per workgroup of the grid-wide kernels
constexpr int kMaxWG = 1024;       // workgroups of a grid-wide kernel (partials)
constexpr int kCoarseN = 32;       // the hierarchy must reach this many points per side
constexpr int kLdsN = 64;          // levels of at most this many points per side in LDS
constexpr int kMatN = 8;           // levels of at most this many as one matrix
constexpr int kCoarseWG = 1024;    // threads of the coarse kernel
constexpr int kMaxLevels = 32;

// integer state words
enum : int { I_DONE = 0, I_ITERS = 1, I_CONV = 2, I_COUNT = 64 };
// scalar slots: r.r of the right-hand side, rho of the previous iteration
enum : int { S_RR0 = 0, S_RHO_PREV = 1, S_COUNT = 8 };

// Level operator, diagonal in units of 1 / H^2: 4 inside, 2 + dl on the last
// row or column, 2 dl in the last corner (dl = 1 + 2^level).
struct Lev {
  int N;
  double H2;      // spacing squared
  double i1, i2;  // 1 / (2 + dl), 1 / (2 dl)
  double* b;      // scaled right-hand side H^2 r (level 0: none, r is unscaled)
  double* z;      // post-smoothed correction (the cycle's output on the level)
};

struct Pcg {
  double* sc;        // S_RR0, S_RHO_PREV
  int* ist;          // I_DONE, I_ITERS, I_CONV
  double* p_rr;      // partials of r.r (k_init, k_down), kMaxWG each
  double* p_rho;     // partials of r.z (the cycle's last kernel on the fine grid)
  double* p_pq;      // partials of p.q (k_dir)
  int np_fine;       // partials of the fine-grid kernels (their workgroups)
  double tol2;
  int max_iter;
  int fixed;         // >= 0: exactly this many iterations
};

// reciprocal of the diagonal at (i, j)
__device__ __forceinline__ double inv_diag(int i, int j, int N, double i1, double i2) {
  const bool x = i == N - 1, y = j == N - 1;
  return x ? (y ? i2 : i1) : (y ? i1 : 0.25);
}

// --------------------------------------------------------------------------
// reductions: each workgroup stores its sum; the consumers add the partials
// in index order (per thread, then the fixed tree of block_sum)
// --------------------------------------------------------------------------

// the sum over the workgroup (NT threads, 4 or 16 waves), in every lane.  lds:
// 16 doubles that nobody reads any more.
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* lds) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) lds[w] = v;
  __syncthreads();
  v = lds[lane & (NT / 64 - 1)];
  if constexpr (NT == 1024) v = add_xor<4>(add_xor<8>(v));
  return add_xor<1>(add_xor<2>(v));
}

// this workgroup's sum of v, stored as its partial
__device__ void partial_store(double v, double* parts) {
  __shared__ double lds[16];
  const double s = block_sum<kBX>(v, lds);
  if (threadIdx.x == 0) parts[blockIdx.x] = s;
}

// The sum of np <= kMaxWG partials, in one fixed order (every workgroup gets the
// same): all of a thread's loads in flight at once, and before the kernel's
// other loads where their consumer comes last (one load and wait a turn, four
// turns a sum: 15.6 us in k_down at N = 1024, now 13.5).  A kernel's
// sums have a SLOT each.
template <int NT>
struct Parts {
  double v[kMaxWG / NT];
  __device__ __forceinline__ Parts(const double* parts, int np) {
#pragma unroll
    for (int q = 0; q < kMaxWG / NT; ++q) {
      const int e = threadIdx.x + q * NT;
      const double w = parts[e < np ? e : 0];
      v[q] = e < np ? w : 0.0;
    }
  }
  template <int SLOT>
  __device__ __forceinline__ double sum() const {
    __shared__ double lds[16];
    double acc = 0.0;
#pragma unroll
    for (int q = 0; q < kMaxWG / NT; ++q) acc += v[q];
    return block_sum<NT>(acc, lds);
  }
};

// The stopping test before iteration k (every workgroup decides alike; the
// first records it, and at k = 0 keeps r.r of the right-hand side).  Returns
// true when the solve has ended.  The first workgroup may record the end while
// others start, so one thread reads it for its whole workgroup: waves reading
// for themselves could part, some gone and the others with a sum that lacks
// theirs.
template <int NT>
__device__ __forceinline__ bool pcg_check(const Pcg& a, int k) {
  __shared__ int ended;
  const Parts<NT> parts(a.p_rr, a.np_fine);
  if (threadIdx.x == 0) ended = a.ist[I_DONE];
  const double rr = parts.template sum<0>();  // (its barrier also orders `ended`)
  if (ended) return true;
  const double rr0 = k == 0 ? rr : a.sc[S_RR0];
  if (k == 0 && blockIdx.x == 0 && threadIdx.x == 0) a.sc[S_RR0] = rr;
  bool stop;
  int conv;
  if (a.fixed >= 0) {
    stop = k >= a.fixed;
    conv = 1;
  } else {
    conv = rr <= a.tol2 * rr0;
    stop = conv || k >= a.max_iter;
  }
  if (stop && blockIdx.x == 0 && threadIdx.x == 0) {
    a.ist[I_DONE] = 1;
    a.ist[I_ITERS] = k;
    a.ist[I_CONV] = conv;
  }
  return stop;
}

// --------------------------------------------------------------------------
// grid-wide level kernels: one tile per workgroup and turn
// --------------------------------------------------------------------------

// Tiles of TX x TY fine points.  32 x 8 up to 512 points per side, where they
// are at most 1024, one turn of the workgroups the chip holds at once; 64 x 16
// above (at 512 and 448 points both take the same time, at 256 a solve of 10
// iterations takes 336 us with the small ones, 362 with the large; at 544 of 24
// iterations 1244 and 1065, at 640 of 11 655 and 565).
constexpr int kTileBig = 513;
__host__ __device__ constexpr int tiles_of(int N, int T) { return (N + T - 1) / T; }

// The PCG update that precedes a cycle on the fine grid: alpha = rho / p.q,
// x += alpha p, r_out = r_in - alpha q (r_out is another buffer: neighbouring
// tiles recompute r in their halos), r.r.
struct DownFine {
  const double* r_in;
  double* r_out;
  const double* p;
  const double* q;
  double* x;
};

// A thread's points are pairs of neighbours (2 i, 2 i + 1) in a row, one red and
// one black: 16-byte loads, half the indices, and the two colours lie in LDS
// arrays of their own that every lane reads at a stride of one.  (Levels that
// have a next one have an even number of points per side, and their arrays are
// aligned to 256 bytes; only x is the caller's and read 8 bytes at a time.)
// In row y of a tile the red point is the pair's second one when y is odd (a
// tile starts two rows above an even row).
//
// Pair of this thread in turn u of a tile W2 pairs wide and H rows high whose
// first point is (i, j).
template <int W2, int H>
struct Pair {
  int y, s, i, j;
  bool in;  // in the tile and in the grid
  __device__ __forceinline__ Pair(int u, int i0, int j0, int N) {
    const int e = threadIdx.x + u * kBX;
    y = e / W2;
    s = e - y * W2;
    i = i0 + 2 * s;
    j = j0 + y;
    in = e < W2 * H && i >= 0 && j >= 0 && i < N && j < N;
  }
  __device__ __forceinline__ int64_t at(int N) const { return in ? (int64_t)j * N + i : 0; }
};

__device__ __forceinline__ double2 ld_pair(const double* p) {
  return *reinterpret_cast<const double2*>(p);
}
__device__ __forceinline__ void st_pair(double* p, double x, double y) {
  *reinterpret_cast<double2*>(p) = make_double2(x, y);
}

enum : int { DOWN_LEVEL = 0, DOWN_FIRST = 1, DOWN_UPDATE = 2 };

// Pre-smoothing from zero (red, black) and restriction of one level: reads b
// (level 0: r), writes the next level's b.  Bound by latency and by the index
// arithmetic (16 cycles an instruction with a CU's 16 waves): one read of a tile
// with a halo of two points, every load issued before the first use, two LDS
// phases.  At N = 1024 the fine level with the update takes 13.5 us, the
// levels of 512 to 128 points 3.5 us each (one point a lane and turn, stride-two
// reads: 15.8 and 4.2; separate kernels for the update, the smoothing and the
// restriction: 13 + 8 + 9 and 9 to 14).
template <int TX, int TY, int MODE>
__global__ __launch_bounds__(kBX) void k_down(Lev L, Lev C, DownFine f, Pcg a, int k, int check) {
  constexpr int W2 = TX / 2 + 3, H = TY + 5;  // from (i0 - 2, j0 - 2)
  constexpr int U = (H * W2 + kBX - 1) / kBX;
  __shared__ double sr[H * W2], sk[H * W2];
  if (check ? pcg_check<kBX>(a, k) : a.ist[I_DONE] != 0) return;
  const int N = L.N, tx = tiles_of(N, TX), nt = tx * tiles_of(N, TY);
  const double* src = MODE == DOWN_LEVEL ? L.b : f.r_in;
  double acc = 0.0, alpha = 0.0;
  const Parts<kBX> prho(a.p_rho, MODE == DOWN_UPDATE ? a.np_fine : 0);
  const Parts<kBX> ppq(a.p_pq, MODE == DOWN_UPDATE ? a.np_fine : 0);
  for (int t = blockIdx.x; t < nt; t += gridDim.x) {
    const int i0 = t % tx * TX, j0 = t / tx * TY;
    auto pair = [&](int u) { return Pair<W2, H>(u, i0 - 2, j0 - 2, N); };
    auto inner = [&](const Pair<W2, H>& g) {
      return g.in && g.s >= 1 && g.s <= TX / 2 && g.y >= 2 && g.y < TY + 2;
    };
    // every load of the tile in flight at once, before the scalars they meet
    double2 b[U], qv[U], pv[U];
    double x0[U], x1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const auto g = pair(u);
      const int64_t p = g.at(N);
      b[u] = ld_pair(src + p);
      if (MODE == DOWN_UPDATE) {
        const int64_t o = inner(g) ? p : 0;
        qv[u] = ld_pair(f.q + p);
        pv[u] = ld_pair(f.p + o);
        x0[u] = f.x[o];
        x1[u] = f.x[o + 1];
      }
    }
    if (MODE == DOWN_UPDATE) {
      if (t == (int)blockIdx.x) {
        const double rho = prho.template sum<1>();
        alpha = rho / ppq.template sum<2>();
        // rho for the next iteration's beta (k_dir read the previous one already)
        if (blockIdx.x == 0 && threadIdx.x == 0) a.sc[S_RHO_PREV] = rho;
      }
    }
    double red[U], blk[U];  // the red e and the black b
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const auto g = pair(u);
      double2 v = b[u];
      if (MODE == DOWN_UPDATE) {
        v.x = fma(-alpha, qv[u].x, v.x);
        v.y = fma(-alpha, qv[u].y, v.y);
        if (inner(g)) {
          const int64_t p = g.at(N);
          f.x[p] = fma(alpha, pv[u].x, x0[u]);
          f.x[p + 1] = fma(alpha, pv[u].y, x1[u]);
          st_pair(f.r_out + p, v.x, v.y);
          acc = fma(v.x, v.x, acc);
          acc = fma(v.y, v.y, acc);
        }
      }
      if (MODE != DOWN_LEVEL) {
        v.x *= L.H2;
        v.y *= L.H2;
      }
      const int odd = g.y & 1;
      blk[u] = odd ? v.x : v.y;
      red[u] = g.in ? (odd ? v.y : v.x) * inv_diag(g.i + odd, g.j, N, L.i1, L.i2) : 0.0;
      const int e = threadIdx.x + u * kBX;
      if (e < H * W2) sr[e] = red[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const auto g = pair(u);
      const int e = threadIdx.x + u * kBX, odd = g.y & 1;
      // (the first and last row, and a neighbour past either end of a row, are
      // of no black point that the restriction reads)
      if (g.y >= 1 && g.y <= H - 2)
        sk[e] = g.in ? (blk[u] + (((red[u] + sr[odd ? e - 1 : e + 1]) + sr[e - W2]) + sr[e + W2])) *
                           inv_diag(g.i + 1 - odd, g.j, N, L.i1, L.i2)
                     : 0.0;
    }
    __syncthreads();
    // full weighting: a red point's residual is the sum of its four black
    // values; a coarse point takes its own and a quarter of its four corners'
    // (points outside the grid are zero, and their residuals have no part)
    if (threadIdx.x < TX / 2 * (TY / 2)) {
      const int Y = threadIdx.x / (TX / 2), X = threadIdx.x % (TX / 2);
      const int I = (i0 >> 1) + X, J = (j0 >> 1) + Y;
      if (I < C.N && J < C.N) {
        const double* m = sk + (2 * Y + 3) * W2 + X + 1;  // row 2 J + 1
        const double wx = I + 1 < C.N ? 1.5 : 1.25, wy = J + 1 < C.N ? 1.5 : 1.25;
        const double in = wx * (m[-W2] + m[W2]) + wy * (m[0] + m[1]);
        double out = (m[-W2 - 1] + m[W2 - 1]) + (m[-2 * W2] + m[-2 * W2 + 1]);
        out += m[-W2 + 1] + m[W2 + 1];
        if (J + 1 < C.N) out += m[2 * W2] + m[2 * W2 + 1];
        C.b[(int64_t)J * C.N + I] = in + 0.25 * out;
      }
    }
    __syncthreads();
  }
  if (MODE == DOWN_UPDATE) partial_store(acc, a.p_rr);
}

// Correction from the coarse level (ec, Nc per side) and post-smoothing (black,
// red) of one level; on the fine grid b = H^2 r and rho = r.z is formed.
// Three LDS phases on a tile with a halo of two points: 7.5 us on the fine grid
// at N = 1024, 3.3 us on the levels of 512 to 128 points (one point a lane and
// turn: 9.4 and 3.7; two half-sweep kernels: 8 + 12 and 9 to 13).
template <int TX, int TY, bool FINE>
__global__ __launch_bounds__(kBX) void k_up(Lev L, const double* r, const double* ec, int Nc,
                                            Pcg a, int dot) {
  constexpr int W2 = TX / 2 + 2, H = TY + 4;       // from (i0 - 2, j0 - 2)
  constexpr int WC = TX / 2 + 3, HC = TY / 2 + 3;  // coarse points i0 / 2 - 2 ..
  constexpr int U = (H * W2 + kBX - 1) / kBX, UC = (HC * WC + kBX - 1) / kBX;
  __shared__ double sr[H * W2], sk[H * W2], sc[HC * WC];
  if (a.ist[I_DONE]) return;
  const int N = L.N, tx = tiles_of(N, TX), nt = tx * tiles_of(N, TY);
  const double* src = FINE ? r : L.b;
  double acc = 0.0;
  for (int t = blockIdx.x; t < nt; t += gridDim.x) {
    const int i0 = t % tx * TX, j0 = t / tx * TY;
    auto pair = [&](int u) { return Pair<W2, H>(u, i0 - 2, j0 - 2, N); };
    double2 b[U];
    double cv[UC];
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const int e = threadIdx.x + u * kBX;
      const int I = i0 / 2 - 2 + e % WC, J = j0 / 2 - 2 + e / WC;
      const bool in = e < HC * WC && I >= 0 && J >= 0 && I < Nc && J < Nc;
      const double v = ec[in ? (int64_t)J * Nc + I : 0];
      cv[u] = in ? v : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) b[u] = ld_pair(src + pair(u).at(N));
#pragma unroll
    for (int u = 0; u < UC; ++u) {
      const int e = threadIdx.x + u * kBX;
      if (e < HC * WC) sc[e] = cv[u];
    }
    __syncthreads();
    double own[U], red[U], blk[U];  // the corrected red z, the red and the black b
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const auto g = pair(u);
      const int e = threadIdx.x + u * kBX, odd = g.y & 1;
      if (FINE) {
        b[u].x *= L.H2;
        b[u].y *= L.H2;
      }
      red[u] = odd ? b[u].y : b[u].x;
      blk[u] = odd ? b[u].x : b[u].y;
      own[u] = 0.0;
      if (g.in) {  // a coarse point itself, or the mean of four
        const double* q = sc + ((g.y >> 1) + 1) * WC + g.s + 1;
        const double corr = odd ? q[0] : 0.25 * ((q[-WC - 1] + q[-WC]) + (q[-1] + q[0]));
        own[u] = red[u] * inv_diag(g.i + odd, g.j, N, L.i1, L.i2) + corr;
      }
      if (e < H * W2) sr[e] = own[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const auto g = pair(u);
      const int e = threadIdx.x + u * kBX, odd = g.y & 1;
      if (g.y >= 1 && g.y <= H - 2) {
        own[u] = g.in ? (blk[u] + (((own[u] + sr[odd ? e - 1 : e + 1]) + sr[e - W2]) + sr[e + W2])) *
                            inv_diag(g.i + 1 - odd, g.j, N, L.i1, L.i2)
                      : 0.0;
        sk[e] = own[u];
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const auto g = pair(u);
      const int e = threadIdx.x + u * kBX, odd = g.y & 1;
      if (g.in && g.s >= 1 && g.s <= TX / 2 && g.y >= 2 && g.y < TY + 2) {
        const double z = (red[u] + (((own[u] + sk[odd ? e + 1 : e - 1]) + sk[e - W2]) + sk[e + W2])) *
                         inv_diag(g.i + odd, g.j, N, L.i1, L.i2);
        st_pair(L.z + g.at(N), odd ? own[u] : z, odd ? z : own[u]);
        if (FINE) acc = fma(red[u], z, fma(blk[u], own[u], acc));
      }
    }
    __syncthreads();
  }
  if (FINE && dot) partial_store(acc / L.H2, a.p_rho);
}

// --------------------------------------------------------------------------
// the levels from 64 points per side down: one workgroup, arrays in LDS
// --------------------------------------------------------------------------

// LDS levels 0 .. nlev-1 (each half the one before it; none in a solve whose
// second level is the matrix); with nmat > 0 the level after them (nmat points
// per side, at most 8) and everything below it is the matrix `mat` (nmat^2
// square, symmetric up to rounding) applied to its scaled right-hand side.
constexpr int kLdsLev = 4;  // 8, 4, 2, 1 in k_matrix; 64, 32, 16 otherwise

struct CoarseArgs {
  const double* in;    // right-hand side of the first LDS level (global)
  double scale;        // b = scale * in
  double* z_out;       // its post-smoothed correction (global)
  int N[kLdsLev];      // sizes of the LDS levels
  double inv[kLdsLev][3];    // 1 / diagonal inside, on the last row or column, in the corner
  int off[kLdsLev + 1];      // where a level's b and z start in LDS
  unsigned half[kLdsLev];    // div_small of (N + 1) / 2
  unsigned full[kLdsLev];    // div_small of N
  unsigned full_mat;         // div_small of nmat
  int nlev;
  int nmat;
  const double* mat;   // [out][in]
};

// e / d as (e m) >> 20 with m = div_small(d): exact while e d < 2^20 (here e <
// 2560 and d <= 64)
inline unsigned div_small(int d) { return (unsigned)(((1 << 20) + d - 1) / d); }
__device__ __forceinline__ int div_by(int e, unsigned m) {
  return (int)(((unsigned)e * m) >> 20);
}

// Bordered arrays: a border of zeros, rows of an even number of doubles.
__host__ __device__ constexpr int row_of(int N) { return N + 2 + (N & 1); }
__host__ __device__ constexpr int area_of(int N) { return row_of(N) * (N + 2); }
constexpr int kCoarseLds = 2 * (area_of(kLdsN) + area_of(kLdsN / 2) + area_of(kLdsN / 4));

// A slot is one red and one black point.  Even slots of a level take the rows
// 0, 2, ..., odd slots the rows 1, 3, ..., where the colour's columns have the
// other parity: 16 neighbouring lanes (128 bytes, what the LDS delivers in a
// cycle) read 16 different banks, where a row alone, every second double,
// conflicts two ways.  A point's word: offset | edges << 20 (edges: how many of
// "last column", "last row" it is in, the index into `inv`), -1 outside.
struct Slot {
  int red, blk;
  int cc;  // offset of the coarse point (I, J) = (i / 2, j / 2) of either
};

__device__ __forceinline__ Slot slot_of(int e, int N, unsigned half) {
  const int S = row_of(N), par = e & 1, h = e >> 1;
  const int J = div_by(h, half), s = h - J * ((N + 1) >> 1), j = 2 * J + par;
  auto word = [&](int i) {
    return i < N && j < N ? ((j + 1) * S + i + 1) | ((i == N - 1) + (j == N - 1)) << 20 : -1;
  };
  return Slot{word(2 * s + par), word(2 * s + 1 - par), (J + 1) * row_of(N >> 1) + s + 1};
}

// What is formed from v is formed anew from here on.  A solve in one workgroup
// forms the same offsets in every iteration: kept for all phases they would
// push its vectors out of the registers.
__device__ __forceinline__ void fresh(int& v) { asm volatile("" : "+v"(v)); }

__device__ __forceinline__ double four(const double* z, int S) {
  return ((z[-1] + z[1]) + z[-S]) + z[S];
}

// Sum of the interpolated corrections at the four red neighbours of a black
// point (N even), zc at its coarse point.  Two of the neighbours are coarse
// points, across the direction of the other two, which are means of four; the
// one after the point lies outside the grid on the last column or row (`edge`).
// par 0: j even, i odd, the means lie along x; par 1: along y.
__device__ __forceinline__ double interp_around(const double* zc, int Sc, int par, bool edge) {
  const int u = par ? Sc : 1, v = par ? 1 : Sc;
  const double here = zc[0] + zc[-v];
  const double before = zc[-u] + zc[-u - v], after = zc[u] + zc[u - v];
  return here + 0.25 * ((before + here) + (edge ? 0.0 : after + here));
}

// Scaled right-hand sides of the next level, n points per side, from the black
// values of one of N = 2 n: a coarse point's own residual (the sum of four black
// values) and a quarter of its four corners' (a corner outside the grid has
// none).  x and y are exchanged in every second row: lanes of both rows then
// read different banks.  put(J n + I, I, J, value)
template <class Put>
__device__ __forceinline__ void restrict_level(const double* z, int N, int n, unsigned full,
                                               Put&& put) {
  int t = threadIdx.x;
  fresh(t);
  const int S = row_of(N), par = t & 1;
  const int u = par ? S : 1, v = par ? 1 : S;
  const int points = 2 * n * ((n + 1) >> 1);
  for (int e = t; e < points; e += kCoarseWG) {
    const int h = e >> 1, Jp = div_by(h, full), I = h - Jp * n, J = 2 * Jp + par;
    if (J < n) {
      const bool xl = I == n - 1, yl = J == n - 1, ul = par ? yl : xl, vl = par ? xl : yl;
      const double* q = z + (2 * J + 2) * S + 2 * I + 2;
      const double in = (ul ? 1.25 : 1.5) * (q[-v] + q[v]) + (vl ? 1.25 : 1.5) * (q[-u] + q[u]);
      double out = (q[-v - 2 * u] + q[v - 2 * u]) + (q[-2 * v - u] + q[-2 * v + u]);
      if (!ul) out += q[-v + 2 * u] + q[v + 2 * u];
      if (!vl) out += q[2 * v - u] + q[2 * v + u];
      put(J * n + I, I, J, in + 0.25 * out);
    }
  }
}

struct MatLds {
  double in[kMatN * kMatN];
  double out[area_of(kMatN)];          // bordered
  double inv[kLdsLev * 3];             // CoarseArgs::inv
};

// This workgroup's slots, matrix share (row t / 16, columns t % 16, + 16, ...)
// and arrays.  LV levels at most, NS slots a thread on the first of them.
template <int LV, int NS>
struct Coarse {
  const CoarseArgs& c;
  double* buf;
  MatLds& m;
  Slot slot[LV][NS];
  double mat[4];

  __device__ double* b(int l) const { return buf + c.off[l]; }
  __device__ double* z(int l) const { return buf + (c.off[l] + c.off[l + 1]) / 2; }

  // (the caller clears buf, and a barrier comes before the first cycle)
  __device__ __forceinline__ Coarse(const CoarseArgs& c_, double* buf_, MatLds& m_)
      : c(c_), buf(buf_), m(m_) {
    const int t = threadIdx.x, n2 = c.nmat * c.nmat, row = t >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = (t & 15) + 16 * q;
      mat[q] = row < n2 && col < n2 ? c.mat[row * n2 + col] : 0.0;
    }
#pragma unroll
    for (int l = 0; l < LV; ++l) {
#pragma unroll
      for (int q = 0; q < (l ? 1 : NS); ++q)
        slot[l][q] = slot_of(t + q * kCoarseWG, c.N[l], c.half[l]);
      if (t < 3) m.inv[3 * l + t] = t == 0 ? c.inv[l][0] : t == 1 ? c.inv[l][1] : c.inv[l][2];
    }
    for (int e = t; e < area_of(kMatN); e += kCoarseWG) m.out[e] = 0.0;
  }

  // this thread's points of one colour of level l: body(offset, 1 / d, edges,
  // offset of the coarse point)
  template <class Body>
  __device__ __forceinline__ void colour(int l, int col, Body&& body) const {
#pragma unroll
    for (int q = 0; q < (l ? 1 : NS); ++q) {
      int w = col ? slot[l][q].blk : slot[l][q].red, cc = slot[l][q].cc;
      fresh(w);
      fresh(cc);
      if (w >= 0) body(w & 0xfffff, m.inv[3 * l + (w >> 20)], w >> 20, cc);
    }
  }

  // the right-hand sides of level l (the matrix: l = nlev) from the level above it
  __device__ __forceinline__ void restrict_to(int l, const double* zf, int N) const {
    const int n = N / 2;
    if (l >= LV || l == c.nlev) {
      restrict_level(zf, N, n, c.full_mat, [&](int p, int, int, double v) { m.in[p] = v; });
    } else {
      double *bl = b(l), *zl = z(l);
      restrict_level(zf, N, n, c.full[l], [&](int, int I, int J, double v) {
        const int o = (J + 1) * row_of(n) + I + 1;
        bl[o] = v;
        if (((I + J) & 1) == 0) zl[o] = v * m.inv[3 * l + (I == n - 1) + (J == n - 1)];
      });
    }
  }

  // The cycle on the LDS levels and the matrix; of level 0 the right-hand side
  // b and the red e = b / d are in place, its result is z(0).  The correction is
  // added to the red values only where the black sweep reads them: the red
  // sweep that follows needs none of their values.
  __device__ __forceinline__ void cycle() const {
#pragma unroll
    for (int l = 0; l < LV; ++l) {
      if (l < c.nlev) {
        const double* bl = b(l);
        double* zl = z(l);
        colour(l, 1, [&](int o, double inv, int, int) {
          zl[o] = (bl[o] + four(zl + o, row_of(c.N[l]))) * inv;
        });
        __syncthreads();
        const bool last = l + 1 == c.nlev;
        if (!last || c.nmat) {
          restrict_to(l + 1, zl, c.N[l]);
          __syncthreads();
        }
      }
    }
    if (c.nmat) {
      int t = threadIdx.x;
      fresh(t);
      const int n = c.nmat, row = t >> 4;
      double v = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int col = (t & 15) + 16 * q;
        if (col < n * n) v = fma(mat[q], m.in[col], v);
      }
      v = add_xor<1>(add_xor<2>(add_xor<4>(add_xor<8>(v))));
      const int J = div_by(row, c.full_mat);
      if (row < n * n && (t & 15) == 0) m.out[(J + 1) * row_of(n) + row - J * n + 1] = v;
      __syncthreads();
    }
#pragma unroll
    for (int l = LV - 1; l >= 0; --l) {
      if (l < c.nlev) {
        const double* bl = b(l);
        double* zl = z(l);
        const int S = row_of(c.N[l]), last = l + 1 == c.nlev;
        if (!last || c.nmat) {
          const double* zc = last ? m.out : z(l + 1 < LV ? l + 1 : l);
          const int Sc = row_of(c.N[l] / 2), par = threadIdx.x & 1;
          colour(l, 1, [&](int o, double inv, int edges, int cc) {
            zl[o] = (bl[o] + (four(zl + o, S) + interp_around(zc + cc, Sc, par, edges != 0))) *
                    inv;
          });
          __syncthreads();
        }
        colour(l, 0, [&](int o, double inv, int, int) {
          zl[o] = (bl[o] + four(zl + o, S)) * inv;
        });
        __syncthreads();
      }
    }
  }
};

// One workgroup: bound by its barrier phases (4 a level: 64, 32 and 16 points
// per side at N = 1024, then the matrix in 2) and the instructions and LDS
// reads between them: 9.3 us (14.4 with 5 a level, indices formed in each, and
// two-way bank conflicts).
__global__ __launch_bounds__(kCoarseWG) void k_coarse(CoarseArgs c, Pcg a, int k, int check) {
  __shared__ double buf[kCoarseLds];
  __shared__ MatLds m;
  const int t = threadIdx.x, N = c.N[0];
  const Coarse<3, 2> A(c, buf, m);
  // grid index of this thread's red points: every load in flight before the test
  int at[2];
  double br[2], bb[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const Slot& s = A.slot[0][q];
    const int e = t + q * kCoarseWG, par = e & 1, h = e >> 1;
    const int J = div_by(h, c.half[0]), i = h - J * ((N + 1) >> 1);
    at[q] = (2 * J + par) * N + 2 * i + par;
    br[q] = c.in[s.red >= 0 ? at[q] : 0];
    bb[q] = c.in[s.blk >= 0 ? at[q] + 1 - 2 * par : 0];
  }
  if (check ? pcg_check<kCoarseWG>(a, k) : a.ist[I_DONE] != 0) return;
  for (int e = t; e < c.off[c.nlev]; e += kCoarseWG) buf[e] = 0.0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const Slot& s = A.slot[0][q];
    if (s.red >= 0) {
      const double v = c.scale * br[q];
      A.b(0)[s.red & 0xfffff] = v;
      A.z(0)[s.red & 0xfffff] = v * m.inv[s.red >> 20];
    }
    if (s.blk >= 0) A.b(0)[s.blk & 0xfffff] = c.scale * bb[q];
  }
  __syncthreads();
  A.cycle();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const Slot& s = A.slot[0][q];
    if (s.red >= 0) c.z_out[at[q]] = A.z(0)[s.red & 0xfffff];
    if (s.blk >= 0) c.z_out[at[q] + 1 - 2 * (t & 1)] = A.z(0)[s.blk & 0xfffff];
  }
}

// The matrix of the last levels: workgroup e runs their cycle (c.nmat = 0) on
// the e-th unit vector and stores column e.
__global__ __launch_bounds__(kCoarseWG) void k_matrix(CoarseArgs c, double* mat) {
  __shared__ double buf[2 * (area_of(8) + area_of(4) + area_of(2) + area_of(1))];
  __shared__ MatLds m;
  const Coarse<4, 1> A(c, buf, m);
  const int N = c.N[0], S = row_of(N), n2 = N * N;
  for (int e = threadIdx.x; e < c.off[c.nlev]; e += kCoarseWG) buf[e] = 0.0;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int i = blockIdx.x % N, j = blockIdx.x / N, p = (j + 1) * S + i + 1;
    A.b(0)[p] = 1.0;
    if (((i + j) & 1) == 0) A.z(0)[p] = m.inv[(i == N - 1) + (j == N - 1)];
  }
  __syncthreads();
  A.cycle();
  for (int r = threadIdx.x; r < n2; r += kCoarseWG)
    mat[(size_t)r * n2 + blockIdx.x] = A.z(0)[(r / N + 1) * S + r % N + 1];
}

// --------------------------------------------------------------------------
// PCG vector kernels (level 0)
// --------------------------------------------------------------------------

__device__ __forceinline__ double c_term(int problem, double u) {
  if (problem == AA_PDE_HEAT_NL1) {
    const double eu = exp(u);
    const double d = u - eu;
    return u + u * eu + u * exp(-u) + d * d;
  }
  return 100.0 * (u - u * u);  // AA_PDE_HEAT_NL2
}

// r = rhs(u) at one point (heat: c(u) - b; Bratu: lambda e^u; plain solve: u)
__device__ __forceinline__ double rhs_at(int problem, double lambda, const double* b, double u,
                                         int64_t p) {
  if (problem == AA_PDE_BRATU) return lambda * exp(u);
  return problem == 0 ? u : c_term(problem, u) - b[p];
}

// r = rhs(u), x = 0, r.r; resets the solve state
__global__ __launch_bounds__(kBX) void k_init(int problem, double lambda, const double* b,
                                              const double* u, double* x, double* r, int N,
                                              Pcg a) {
  double acc = 0.0;
  const int64_t n = (int64_t)N * N;
  for (int64_t p = (int64_t)blockIdx.x * kBX + threadIdx.x; p < n; p += (int64_t)gridDim.x * kBX) {
    const double v = rhs_at(problem, lambda, b, u[p], p);
    r[p] = v;
    x[p] = 0.0;
    acc = fma(v, v, acc);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.ist[I_DONE] = 0;
    a.ist[I_ITERS] = 0;
    a.ist[I_CONV] = 0;
  }
  partial_store(acc, a.p_rr);
}

// p = z + beta p_prev (beta = rho_k / rho_{k-1}; p = z at k = 0), q = A p, p.q:
// 8.4 us at N = 1024 (9.5 with one point a lane and turn)
template <int TX, int TY>
__global__ __launch_bounds__(kBX) void k_dir(const double* z, const double* p_prev,
                                             double* p_cur, double* q, int N, double ih2, Pcg a,
                                             int k) {
  constexpr int W2 = TX / 2 + 2, H = TY + 2;  // from (i0 - 2, j0 - 1)
  constexpr int U = (H * W2 + kBX - 1) / kBX;
  __shared__ double2 sp[H * W2];
  if (a.ist[I_DONE]) return;
  const bool first = k == 0;
  const int tx = tiles_of(N, TX), nt = tx * tiles_of(N, TY);
  double acc = 0.0, beta = 0.0;
  const Parts<kBX> prho(a.p_rho, first ? 0 : a.np_fine);
  const double rho_prev = first ? 1.0 : a.sc[S_RHO_PREV];
  for (int t = blockIdx.x; t < nt; t += gridDim.x) {
    const int i0 = t % tx * TX, j0 = t / tx * TY;
    auto pair = [&](int u) { return Pair<W2, H>(u, i0 - 2, j0 - 1, N); };
    double2 zv[U], pv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t p = pair(u).at(N);
      zv[u] = ld_pair(z + p);
      pv[u] = first ? make_double2(0.0, 0.0) : ld_pair(p_prev + p);
    }
    if (t == (int)blockIdx.x && !first) beta = prho.template sum<1>() / rho_prev;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = threadIdx.x + u * kBX;
      const bool in = pair(u).in;
      pv[u].x = in ? fma(beta, pv[u].x, zv[u].x) : 0.0;
      pv[u].y = in ? fma(beta, pv[u].y, zv[u].y) : 0.0;
      if (e < H * W2) sp[e] = pv[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const auto g = pair(u);
      const int e = threadIdx.x + u * kBX;
      if (g.in && g.s >= 1 && g.s <= TX / 2 && g.y >= 1 && g.y <= TY) {
        const double2 c = pv[u], up = sp[e - W2], dn = sp[e + W2];
        const double l = sp[e - 1].y, r = sp[e + 1].x;
        const double q0 = (4.0 * c.x - (((l + c.y) + up.x) + dn.x)) * ih2;
        const double q1 = (4.0 * c.y - (((c.x + r) + up.y) + dn.y)) * ih2;
        const int64_t p = g.at(N);
        st_pair(p_cur + p, c.x, c.y);
        st_pair(q + p, q0, q1);
        acc = fma(c.x, q0, fma(c.y, q1, acc));
      }
    }
    __syncthreads();
  }
  partial_store(acc, a.p_pq);
}

// --------------------------------------------------------------------------
// whole solves of small grids: one workgroup
// --------------------------------------------------------------------------

constexpr int kSmallN = 96;  // its z and the levels below it fill the LDS (131 KB)

// The PCG solve of an N x N grid, N <= 96: r, p and A p of a thread's RP slots
// in registers, z (and p, for q = A p) of the fine grid and every coarser level
// in LDS, the last levels the matrix.  One launch instead of 4 an iteration (and
// none enqueued past the end).  Bound by its 20 to 30 barriers an iteration and
// by the instructions between them, 16 cycles each on the four SIMDs with all 16
// waves: so points are enumerated without gaps, and a slot's word is kept.  A
// solve (launches per level / this): N = 16 195 / 60 us, 31 (56 iterations) 957
// / 166, 64 300 / 104, 96 331 / 191 (161 and 302 with rows of 32 and 64 lanes,
// the reds corrected in a phase of their own and every second double read).
// More than two slots a thread: x in global memory and A p formed twice, which
// frees 20 to 40 registers (96 points: 215 us with A p kept and spills).
template <int RP>
__global__ __launch_bounds__(kCoarseWG) void k_solve_small(int problem, double lambda,
                                                           const double* b, const double* u,
                                                           double* xo, int N, unsigned half,
                                                           CoarseArgs c, Pcg a) {
  extern __shared__ double z0[];  // bordered; then the coarser levels
  __shared__ MatLds m;
  __shared__ double lds[3][16];
  constexpr bool XREG = RP <= 2;  // x in registers (with more slots they would spill)
  const int t = threadIdx.x, S = row_of(N), par = t & 1, side = 1 - 2 * par;
  const bool coarse = c.nlev + c.nmat > 0;
  const Coarse<3, 2> A(c, z0 + area_of(N), m);
  const double h = 1.0 / (double)(N + 1), H2 = h * h, ih2 = 1.0 / H2;
  double r[2][RP], p[2][RP], v[2][XREG ? RP : 1], x[2][XREG ? RP : 1];
  // offset of the red point, black is `side` next to it; bit 16: there is a red
  // point, 17: a black one, 18: the black one on the last row or column
  int word[RP];
#pragma unroll
  for (int q = 0; q < RP; ++q) {
    const Slot s = slot_of(t + q * kCoarseWG, N, half);
    const int o = s.red >= 0 ? s.red & 0xfffff : (s.blk & 0xfffff) - side;
    word[q] = (s.red < 0 && s.blk < 0 ? 0 : o) | (s.red >= 0) << 16 | (s.blk >= 0) << 17 |
              (s.blk >= 1 << 20) << 18;
  }
  // body(slot, offset, r, p, A p) over this thread's points of one colour
  auto points = [&](int col, auto&& body) {
#pragma unroll
    for (int q = 0; q < RP; ++q) {
      int w = word[q];
      fresh(w);
      if (w >> (16 + col) & 1) body(q, (w & 0xffff) + col * side, r[col][q], p[col][q], v[col][XREG ? q : 0]);
    }
  };
  // grid index of a point
  auto grid = [&](int col, int q) {
    int e = t + q * kCoarseWG;
    fresh(e);
    const int J = div_by(e >> 1, half), i = (e >> 1) - J * ((N + 1) >> 1);
    return (2 * J + par) * N + 2 * i + (col ? 1 - par : par);
  };
  for (int e = t; e < area_of(N) + c.off[c.nlev]; e += kCoarseWG) z0[e] = 0.0;
  double rr = 0.0;
#pragma unroll
  for (int col = 0; col < 2; ++col)
    points(col, [&](int q, int, double& rv, double& pv, double&) {
      const int g = grid(col, q);
      rv = rhs_at(problem, lambda, b, u[g], g);
      pv = 0.0;
      rr = fma(rv, rv, rr);
      if (XREG) x[col][XREG ? q : 0] = 0.0;
    });
  rr = block_sum<kCoarseWG>(rr, lds[0]);
  const double rr0 = rr;
  double rho_prev = 0.0;
  const int last = a.fixed >= 0 ? a.fixed : a.max_iter;
  int k = 0;
  while (k < last && (a.fixed >= 0 || !(rr <= a.tol2 * rr0))) {
    // the cycle: every diagonal entry of the fine grid is 4
    points(0, [&](int, int o, double& rv, double&, double&) { z0[o] = H2 * rv * 0.25; });
    __syncthreads();
    points(1, [&](int, int o, double& rv, double&, double&) {
      z0[o] = (H2 * rv + four(z0 + o, S)) * 0.25;
    });
    __syncthreads();
    if (coarse) {
      A.restrict_to(0, z0, N);
      __syncthreads();
      A.cycle();
      const double* zc = c.nlev ? A.z(0) : m.out;
      const int Sc = row_of(N >> 1);
#pragma unroll
      for (int q = 0; q < RP; ++q) {
        int w = word[q], e = t + q * kCoarseWG;
        fresh(w);
        fresh(e);
        if (w >> 17 & 1) {
          const int o = (w & 0xffff) + side, J = div_by(e >> 1, half);
          const int cc = (J + 1) * Sc + (e >> 1) - J * ((N + 1) >> 1) + 1;
          z0[o] = (H2 * r[1][q] +
                   (four(z0 + o, S) + interp_around(zc + cc, Sc, par, w >> 18 & 1))) * 0.25;
        }
      }
      __syncthreads();
    }
    points(0, [&](int, int o, double& rv, double&, double&) {
      z0[o] = (H2 * rv + four(z0 + o, S)) * 0.25;
    });
    // each thread reads back its own points only
    double acc = 0.0;
#pragma unroll
    for (int col = 0; col < 2; ++col)
      points(col, [&](int, int o, double& rv, double&, double&) { acc = fma(rv, z0[o], acc); });
    const double rho = block_sum<kCoarseWG>(acc, lds[1]);
    const double beta = k == 0 ? 0.0 : rho / rho_prev;
    rho_prev = rho;
#pragma unroll
    for (int col = 0; col < 2; ++col)
      points(col, [&](int, int o, double&, double& pv, double&) {
        pv = fma(beta, pv, z0[o]);
        z0[o] = pv;  // p, for q = A p (z is not needed any more)
      });
    __syncthreads();
    acc = 0.0;
#pragma unroll
    for (int col = 0; col < 2; ++col)
      points(col, [&](int, int o, double&, double& pv, double& q) {
        q = (4.0 * pv - four(z0 + o, S)) * ih2;
        acc = fma(pv, q, acc);
      });
    const double alpha = rho / block_sum<kCoarseWG>(acc, lds[2]);
    acc = 0.0;
#pragma unroll
    for (int col = 0; col < 2; ++col)
      points(col, [&](int q, int o, double& rv, double& pv, double& qv) {
        if (XREG) {
          double& xv = x[col][XREG ? q : 0];
          xv = fma(alpha, pv, xv);
        } else {
          double* xp = xo + grid(col, q);
          *xp = fma(alpha, pv, k == 0 ? 0.0 : *xp);
        }
        rv = fma(-alpha, XREG ? qv : (4.0 * pv - four(z0 + o, S)) * ih2, rv);
        acc = fma(rv, rv, acc);
      });
    rr = block_sum<kCoarseWG>(acc, lds[0]);
    ++k;
  }
  if (XREG || k == 0) {
#pragma unroll
    for (int col = 0; col < 2; ++col)
      points(col, [&](int q, int, double&, double&, double&) {
        xo[grid(col, q)] = XREG ? x[col][XREG ? q : 0] : 0.0;
      });
  }
  if (t == 0) {
    a.ist[I_DONE] = 1;
    a.ist[I_ITERS] = k;
    a.ist[I_CONV] = a.fixed >= 0 || rr <= a.tol2 * rr0 ? 1 : 0;
  }
}

__global__ void k_reset(int* ist) {
  if (threadIdx.x < I_COUNT) ist[threadIdx.x] = 0;
}

}  // namespace pde
}  // namespace aa

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

using namespace aa::pde;

struct aa_pde2d {
  int N;
  int problem;
  double lambda, tol;
  int max_iter, fixed;
  hipStream_t st;
  int nlev, first_lds;     // levels >= first_lds run in k_coarse
  int first_mat;           // levels >= first_mat are its matrix (nlev: none)
  Lev lev[kMaxLevels];
  double *r[2], *z, *p[2], *q, *sc, *p_rr, *p_rho, *p_pq, *mat;
  int* ist;
  int last_iters, last_conv, predicted;
};

namespace {

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// sizes of the hierarchy: halve while even; the coarse part must fit one
// workgroup's LDS (the first size of at most 32 points per side is reached)
int hierarchy(int64_t N, int* sizes) {
  int L = 0;
  int64_t n = N;
  while (true) {
    if (L >= kMaxLevels) return -1;
    sizes[L++] = (int)n;
    if (n % 2 != 0) break;
    n /= 2;
  }
  return L;
}

int first_level(const int* sizes, int L, int most) {
  for (int l = 0; l < L; ++l)
    if (sizes[l] <= most) return l;
  return -1;
}

size_t layout(int64_t N, int max_iter, const int* sizes, int L, aa_pde2d* c, char* base) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += align256(bytes);
    return p;
  };
  const size_t n = (size_t)N * (size_t)N;
  (void)max_iter;
  int* ist = (int*)take(I_COUNT * sizeof(int));
  double* sc = (double*)take(S_COUNT * sizeof(double));
  double* p_rr = (double*)take(kMaxWG * sizeof(double));
  double* p_rho = (double*)take(kMaxWG * sizeof(double));
  double* p_pq = (double*)take(kMaxWG * sizeof(double));
  double* mat = (double*)take(kMatN * kMatN * kMatN * kMatN * sizeof(double));
  double* r0 = (double*)take(n * 8);
  double* r1 = (double*)take(n * 8);
  double* z = (double*)take(n * 8);
  double* p0 = (double*)take(n * 8);
  double* p1 = (double*)take(n * 8);
  double* q = (double*)take(n * 8);
  if (c) {
    c->ist = ist;
    c->sc = sc;
    c->p_rr = p_rr;
    c->p_rho = p_rho;
    c->p_pq = p_pq;
    c->mat = mat;
    c->r[0] = r0;
    c->r[1] = r1;
    c->z = z;
    c->p[0] = p0;
    c->p[1] = p1;
    c->q = q;
  }
  const double h = 1.0 / (double)(N + 1);
  for (int l = 0; l < L; ++l) {
    const size_t nl = (size_t)sizes[l] * (size_t)sizes[l];
    double *lb = nullptr, *lz = z;
    if (l > 0) {
      lb = (double*)take(nl * 8);
      lz = (double*)take(nl * 8);
    }
    if (c) {
      const double H = h * (double)(1ll << l), dl = 1.0 + (double)(1ll << l);
      c->lev[l] = Lev{sizes[l], H * H, 1.0 / (2.0 + dl), 1.0 / (2.0 * dl), lb, lz};
    }
  }
  return off;
}

// workgroups of a tiled kernel on an N x N level
int tile_grid(int N) {
  const int64_t nt = N >= kTileBig ? (int64_t)tiles_of(N, 64) * tiles_of(N, 16)
                                   : (int64_t)tiles_of(N, 32) * tiles_of(N, 8);
  return (int)(nt < kMaxWG ? nt : kMaxWG);
}

Pcg pcg_args(const aa_pde2d* c) {
  Pcg a;
  a.sc = c->sc;
  a.ist = c->ist;
  a.p_rr = c->p_rr;
  a.p_rho = c->p_rho;
  a.p_pq = c->p_pq;
  a.np_fine = tile_grid(c->N);
  a.tol2 = c->tol * c->tol;
  a.max_iter = c->max_iter;
  a.fixed = c->fixed;
  return a;
}

CoarseArgs coarse_args(const aa_pde2d* c, int from, int to, int nmat) {
  CoarseArgs ca;
  memset(&ca, 0, sizeof(ca));
  ca.scale = 1.0;
  ca.nlev = to - from;
  for (int l = from; l < to; ++l) {
    const int n = c->lev[l].N, q = l - from;
    ca.N[q] = n;
    ca.inv[q][0] = 0.25;
    ca.inv[q][1] = c->lev[l].i1;
    ca.inv[q][2] = c->lev[l].i2;
    ca.half[q] = div_small((n + 1) / 2);
    ca.full[q] = div_small(n);
    ca.off[q + 1] = ca.off[q] + 2 * area_of(n);
  }
  if (nmat) ca.full_mat = div_small(nmat);
  ca.nmat = nmat;
  ca.mat = c->mat;
  return ca;
}

template <int MODE>
void launch_down(const aa_pde2d* c, int l, const DownFine& f, const Pcg& a, int k, int check) {
  const Lev &L = c->lev[l], &C = c->lev[l + 1];
  if (L.N >= kTileBig)
    hipLaunchKernelGGL((k_down<64, 16, MODE>), dim3(tile_grid(L.N)), dim3(kBX), 0, c->st, L, C, f,
                       a, k, check);
  else
    hipLaunchKernelGGL((k_down<32, 8, MODE>), dim3(tile_grid(L.N)), dim3(kBX), 0, c->st, L, C, f,
                       a, k, check);
}

template <bool FINE>
void launch_up(const aa_pde2d* c, int l, const double* r, const Pcg& a, int dot) {
  const Lev &L = c->lev[l], &C = c->lev[l + 1];
  if (L.N >= kTileBig)
    hipLaunchKernelGGL((k_up<64, 16, FINE>), dim3(tile_grid(L.N)), dim3(kBX), 0, c->st, L, r,
                       (const double*)C.z, C.N, a, dot);
  else
    hipLaunchKernelGGL((k_up<32, 8, FINE>), dim3(tile_grid(L.N)), dim3(kBX), 0, c->st, L, r,
                       (const double*)C.z, C.N, a, dot);
}

// One V-cycle into z: on r[0] (k = 0), or on r[k & 1] after the PCG update
// that forms it from the previous iteration's p, q and r (k > 0).  `pcg`: the
// stopping test before iteration k runs in the first kernel that follows the
// residual's norm, and rho_k = r . z is stored.
hipError_t launch_vcycle(const aa_pde2d* c, const Pcg& a, int k, int pcg, double* x) {
  const int fl = c->first_lds;
  const double* r = c->r[k & 1];
  for (int l = 0; l < fl; ++l) {
    const DownFine f{c->r[l == 0 && k > 0 ? (k + 1) & 1 : 0], c->r[k & 1], c->p[(k + 1) & 1], c->q,
                     x};
    if (l > 0)
      launch_down<DOWN_LEVEL>(c, l, f, a, k, pcg && l == 1);
    else if (k > 0)
      launch_down<DOWN_UPDATE>(c, l, f, a, k, 0);
    else
      launch_down<DOWN_FIRST>(c, l, f, a, k, 0);
  }
  const int to = c->first_mat;
  CoarseArgs ca = coarse_args(c, fl, to, to < c->nlev ? c->lev[to].N : 0);
  ca.in = fl == 0 ? r : c->lev[fl].b;
  if (fl == 0) ca.scale = c->lev[0].H2;
  ca.z_out = c->lev[fl].z;
  hipLaunchKernelGGL(k_coarse, dim3(1), dim3(kCoarseWG), 0, c->st, ca, a, k, pcg && fl <= 1);
  for (int l = fl - 1; l > 0; --l) launch_up<false>(c, l, nullptr, a, 0);
  if (fl > 0) launch_up<true>(c, 0, r, a, pcg);
  return hipGetLastError();
}

// PCG iteration k: the update of iteration k - 1 and the cycle, then p, q
hipError_t launch_iteration(const aa_pde2d* c, const Pcg& a, int k, double* x) {
  hipError_t e = launch_vcycle(c, a, k, 1, x);
  if (e != hipSuccess) return e;
  const int N = c->N;
  const double h = 1.0 / (double)(N + 1), ih2 = 1.0 / (h * h);
  double* pc = c->p[k & 1];
  const double* pp = c->p[(k + 1) & 1];
  if (N >= kTileBig)
    hipLaunchKernelGGL((k_dir<64, 16>), dim3(a.np_fine), dim3(kBX), 0, c->st,
                       (const double*)c->z, pp, pc, c->q, N, ih2, a, k);
  else
    hipLaunchKernelGGL((k_dir<32, 8>), dim3(a.np_fine), dim3(kBX), 0, c->st, (const double*)c->z,
                       pp, pc, c->q, N, ih2, a, k);
  return hipGetLastError();
}

aa_status hipst(hipError_t e) { return e == hipSuccess ? AA_OK : AA_EHIP; }

// the whole solve of a small grid in one launch
hipError_t launch_small(const aa_pde2d* c, const Pcg& a, int problem, const double* b,
                        const double* u, double* x) {
  const int N = c->N, coarse = c->nlev > 1 ? 1 : 0;
  const int to = c->first_mat;  // levels 1 .. to-1 in LDS, then the matrix
  const CoarseArgs ca = coarse_args(c, coarse, coarse ? to : 0,
                                    coarse && to < c->nlev ? c->lev[to].N : 0);
  const size_t lds = sizeof(double) * (size_t)(area_of(N) + ca.off[ca.nlev]);
  const int slots = 2 * ((N + 1) / 2) * ((N + 1) / 2);
  const unsigned half = div_small((N + 1) / 2);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kCoarseWG), lds, c->st, problem, c->lambda, b, u, x, N,
                       half, ca, a);
  };
  if (slots <= kCoarseWG)
    go(k_solve_small<1>);
  else if (slots <= 2 * kCoarseWG)
    go(k_solve_small<2>);
  else if (slots <= 3 * kCoarseWG)
    go(k_solve_small<3>);
  else
    go(k_solve_small<5>);
  return hipGetLastError();
}

// the PCG solve of A x = rhs(problem, u): enqueue iterations, read the state
// now and then (a first batch sized by the previous solve)
aa_status solve(aa_pde2d* c, int problem, const double* b, const double* u, double* x) {
  (void)hipGetLastError();
  const Pcg a = pcg_args(c);
  const int N = c->N;
  if (N <= kSmallN) {
    hipError_t e = launch_small(c, a, problem, b, u, x);
    int st[3] = {0, 0, 0};
    if (e == hipSuccess)
      e = hipMemcpyAsync(st, c->ist, sizeof(st), hipMemcpyDeviceToHost, c->st);
    if (e == hipSuccess) e = hipStreamSynchronize(c->st);
    if (e != hipSuccess || !st[I_DONE]) return AA_EHIP;
    c->last_iters = c->predicted = st[I_ITERS];
    c->last_conv = st[I_CONV];
    return AA_OK;
  }
  hipLaunchKernelGGL(k_init, dim3(a.np_fine), dim3(kBX), 0, c->st, problem, c->lambda, b, u, x,
                     c->r[0], N, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return AA_EHIP;
  const int last = c->fixed >= 0 ? c->fixed : c->max_iter;
  int k = 0;
  int batch = c->predicted + 1;
  int st[3] = {0, 0, 0};
  while (true) {
    for (int t = 0; t < batch && k <= last; ++t, ++k) {
      e = launch_iteration(c, a, k, x);
      if (e != hipSuccess) return AA_EHIP;
    }
    e = hipMemcpyAsync(st, c->ist, sizeof(st), hipMemcpyDeviceToHost, c->st);
    if (e == hipSuccess) e = hipStreamSynchronize(c->st);
    if (e != hipSuccess) return AA_EHIP;
    if (st[I_DONE]) break;
    if (k > last) return AA_EHIP;  // not reached: the test before iteration `last` stops
    batch = 2;
  }
  c->last_iters = st[I_ITERS];
  c->last_conv = st[I_CONV];
  c->predicted = st[I_ITERS];
  return AA_OK;
}

}  // namespace

extern "C" {

aa_status aa_pde2d_workspace_size(int64_t N, int max_iter, size_t* bytes) {
  if (!bytes || N < 1 || N > 65536 || max_iter < 1 || max_iter > 100000) return AA_EINVAL;
  int sizes[kMaxLevels];
  const int L = hierarchy(N, sizes);
  if (L < 1 || first_level(sizes, L, kCoarseN) < 0) return AA_EINVAL;
  *bytes = layout(N, max_iter, sizes, L, nullptr, nullptr);
  return AA_OK;
}

aa_status aa_pde2d_init(aa_pde2d** ctx, int64_t N, int problem, double lambda, double tol,
                        int max_iter, void* d_workspace, size_t bytes, void* stream) {
  if (!ctx) return AA_EINVAL;
  *ctx = nullptr;
  if (problem != AA_PDE_HEAT_NL1 && problem != AA_PDE_HEAT_NL2 && problem != AA_PDE_BRATU)
    return AA_EINVAL;
  if (!(tol >= 0.0) || !isfinite(lambda) || !d_workspace || ((uintptr_t)d_workspace & 255))
    return AA_EINVAL;
  size_t need = 0;
  aa_status s = aa_pde2d_workspace_size(N, max_iter, &need);
  if (s != AA_OK) return s;
  if (bytes < need) return AA_ENOSPACE;
  aa_pde2d* c = (aa_pde2d*)calloc(1, sizeof(aa_pde2d));
  if (!c) return AA_EINVAL;
  c->N = (int)N;
  c->problem = problem;
  c->lambda = lambda;
  c->tol = tol;
  c->max_iter = max_iter;
  c->fixed = -1;
  c->st = (hipStream_t)stream;
  int sizes[kMaxLevels];
  c->nlev = hierarchy(N, sizes);
  c->first_lds = first_level(sizes, c->nlev, kLdsN);
  c->first_mat = c->nlev;
  for (int l = c->first_lds + 1; l < c->nlev && c->first_mat == c->nlev; ++l)
    if (sizes[l] <= kMatN) c->first_mat = l;
  layout(N, max_iter, sizes, c->nlev, c, (char*)d_workspace);
  c->predicted = 8;
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, c->st, c->ist);
  if (c->first_mat < c->nlev) {
    const int n = c->lev[c->first_mat].N;
    hipLaunchKernelGGL(k_matrix, dim3(n * n), dim3(kCoarseWG), 0, c->st,
                       coarse_args(c, c->first_mat, c->nlev, 0), c->mat);
  }
  // every later call reads the matrix, on whatever stream the caller sets then:
  // wait for it here (a stream being captured runs nothing yet)
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && c->st) e = hipStreamIsCapturing(c->st, &cap);
  if (e == hipSuccess && c->first_mat < c->nlev && cap == hipStreamCaptureStatusNone)
    e = hipStreamSynchronize(c->st);
  if (e != hipSuccess) {
    free(c);
    return AA_EHIP;
  }
  *ctx = c;
  return AA_OK;
}

aa_status aa_pde2d_set_iters(aa_pde2d* c, int iters) {
  if (!c || iters < -1 || iters > c->max_iter) return AA_EINVAL;
  c->fixed = iters;
  return AA_OK;
}

aa_status aa_pde2d_apply(aa_pde2d* c, const double* d_b, const double* d_u, double* d_out) {
  if (!c || !d_u || !d_out) return AA_EINVAL;
  if (c->problem != AA_PDE_BRATU && !d_b) return AA_EINVAL;
  return solve(c, c->problem, d_b, d_u, d_out);
}

aa_status aa_pde2d_solve(aa_pde2d* c, const double* d_rhs, double* d_x) {
  if (!c || !d_rhs || !d_x) return AA_EINVAL;
  return solve(c, 0, nullptr, d_rhs, d_x);
}

aa_status aa_pde2d_vcycle(aa_pde2d* c, const double* d_r, double* d_z) {
  if (!c || !d_r || !d_z) return AA_EINVAL;
  (void)hipGetLastError();
  const size_t n = (size_t)c->N * (size_t)c->N;
  hipLaunchKernelGGL(k_reset, dim3(1), dim3(64), 0, c->st, c->ist);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(c->r[0], d_r, n * 8, hipMemcpyDeviceToDevice, c->st);
  if (e == hipSuccess) e = launch_vcycle(c, pcg_args(c), 0, 0, nullptr);
  if (e == hipSuccess) e = hipMemcpyAsync(d_z, c->z, n * 8, hipMemcpyDeviceToDevice, c->st);
  return hipst(e);
}

aa_status aa_pde2d_last(const aa_pde2d* c, int* h_iters, int* h_converged) {
  if (!c) return AA_EINVAL;
  if (h_iters) *h_iters = c->last_iters;
  if (h_converged) *h_converged = c->last_conv;
  return AA_OK;
}

aa_status aa_pde2d_set_stream(aa_pde2d* c, void* stream) {
  if (!c) return AA_EINVAL;
  c->st = (hipStream_t)stream;
  return AA_OK;
}

aa_status aa_pde2d_destroy(aa_pde2d* c) {
  free(c);
  return AA_OK;
}

}  // extern "C"
