// aa_problems.hip -- model fixed-point maps and seeded input generators.
//
// G(u) = u - omega (A u + c u^3 - f), A the (2 dim + 1)-point Dirichlet
// Laplacian on an s^dim grid (x fastest) scaled by 1/h^2: the 1D Poisson,
// 3D nonlinear and 2D batched workloads all use it (dim = 1, 3, 2).
#include <math.h>

#include "aa_passes.h"

namespace aa {

// Any size (more than 2^31 points, or more per side than the tiles address).
__global__ __launch_bounds__(256) void k_stencil(int dim, int64_t s, double ih2, double omega,
                                                 double c, const double* __restrict__ f,
                                                 const double* __restrict__ u,
                                                 double* __restrict__ out, int64_t n) {
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n;
       p += (int64_t)gridDim.x * blockDim.x)
    out[p] = stencil_point(u, f, dim, s, ih2, omega, c, p);
}

constexpr int kMarchWG = 1024, kMarchChunk = 16;

// One thread per point of a plane (3D), row (2D) or line segment (1D), marching
// `chunk` planes along the slowest dimension with the three planes' values in
// registers.  A plane's points are taken in memory order, so a workgroup's
// 1024 are a few whole rows and most of the y neighbours are its own reads.
// What bounds the map is the traffic beyond the eight L2s: consecutive
// workgroups run on different ones, so with one grid row per workgroup u was
// fetched five times (three rows, two planes); marching fetches it about 1.7
// times at s = 256: 140 -> 94 us there (4.3 TB/s of its 3 vectors), 39.7 -> 26.2
// at s = 160, 13.9 -> 9 at s = 101, 28.5 -> 21.5 for 2048^2 (workgroups of 512
// or 256 points and chunks of 8 or 32: 100 to 113 us at s = 256, the rest
// within 5 %).  Same arithmetic, in the same order, as stencil_point.  f
// and the output are streamed non-temporally.
template <int DIM>
__global__ __launch_bounds__(1024) void k_stencil_march(int s, double ih2, double omega, double c,
                                                        const double* __restrict__ f,
                                                        const double* __restrict__ u,
                                                        double* __restrict__ out, int plane,
                                                        int chunk) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;  // point of the plane
  if (q >= plane) return;
  const int x = DIM == 3 ? q % s : q, y = DIM == 3 ? q / s : 0;
  const int z0 = DIM == 1 ? 0 : blockIdx.y * chunk;
  const int z1 = DIM == 1 ? 1 : z0 + chunk < s ? z0 + chunk : s;
  int64_t p = (int64_t)z0 * plane + q;
  double lo = z0 > 0 ? u[p - plane] : 0.0, mid = u[p];
  for (int z = z0; z < z1; ++z, p += plane) {
    const bool more = DIM > 1 && z < s - 1;
    const double hi = more ? u[p + plane] : 0.0;
    const double fv = __builtin_nontemporal_load(f + p);
    double nb = 0.0;
    if (x > 0) nb += u[p - 1];
    if (x < s - 1) nb += u[p + 1];
    if (DIM == 3) {
      if (y > 0) nb += u[p - s];
      if (y < s - 1) nb += u[p + s];
    }
    if (z > 0) nb += lo;
    if (more) nb += hi;
    const double au = (2.0 * DIM * mid - nb) * ih2;
    __builtin_nontemporal_store(mid - omega * (au + c * mid * mid * mid - fv), out + p);
    lo = mid;
    mid = hi;
  }
}

hipError_t launch_stencil(int dim, int64_t s, double h, double omega, double c,
                          const double* f, const double* u, double* out, hipStream_t st) {
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  int64_t n = s;
  if (dim >= 2) n *= s;
  if (dim >= 3) n *= s;
  const double ih2 = 1.0 / (h * h);
  const int64_t plane = dim == 3 ? s * s : s;
  if (plane < (1 << 30)) {
    // workgroups of 1024 points from a quarter million points (256 below: more
    // of them on the chip), the shortest chunk that leaves one resident round,
    // at most 16 planes
    const int64_t wg = n >= 1024 * 256 ? kMarchWG : 256;
    const int block = (int)(plane < wg ? (plane + 63) / 64 * 64 : wg);
    const int64_t gx = (plane + block - 1) / block;
    const int64_t resident = 2048 * 256 / block;  // workgroups the chip holds
    int64_t chunk = dim == 1 ? 1 : (gx * s + resident - 1) / resident;
    chunk = chunk > kMarchChunk ? kMarchChunk : chunk;
    const int64_t gy = dim == 1 ? 1 : (s + chunk - 1) / chunk;
    if (gy <= 65535) {
      const dim3 g((unsigned)gx, (unsigned)gy), b((unsigned)block);
      if (dim == 1)
        hipLaunchKernelGGL(k_stencil_march<1>, g, b, 0, st, (int)s, ih2, omega, c, f, u, out,
                           (int)plane, (int)chunk);
      else if (dim == 2)
        hipLaunchKernelGGL(k_stencil_march<2>, g, b, 0, st, (int)s, ih2, omega, c, f, u, out,
                           (int)plane, (int)chunk);
      else
        hipLaunchKernelGGL(k_stencil_march<3>, g, b, 0, st, (int)s, ih2, omega, c, f, u, out,
                           (int)plane, (int)chunk);
      return hipGetLastError();
    }
  }
  int64_t blocks = (n + 255) / 256;
  int grid = (int)(blocks < 65536 ? blocks : 65536);
  hipLaunchKernelGGL(k_stencil, dim3(grid), dim3(256), 0, st, dim, s, ih2, omega, c, f, u, out, n);
  return hipGetLastError();
}

// The generators write far more than the caches hold and nothing reads it back
// at once: non-temporal stores.  (Ordinary stores leave the caches full of
// dirty lines, and the next kernel's reads then share HBM with their write-
// back: a 20-vector read pass ran 12 % slower right after a 512 MiB fill.)

// counter origin of stream (seed, stream_id)
static uint64_t stream_base(uint64_t seed, uint64_t stream_id) {
  return sm64_mix_host(sm64_mix_host(seed) + stream_id);
}

__global__ void k_fill_uniform(double* out, int64_t n, uint64_t base, double lo, double hi) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    __builtin_nontemporal_store(lo + (hi - lo) * u01(base + (uint64_t)i), out + i);
}

__global__ void k_fill_normal(double* out, int64_t n, uint64_t base, uint64_t offset) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    __builtin_nontemporal_store(normal_at(base, offset + (uint64_t)i), out + i);
}

// ---------------------------------------------------------------------------
// EM update of a three-component normal mixture's means (Sec. 5.3)
// ---------------------------------------------------------------------------

struct EmArgs {
  const double* x; int64_t N;      // samples
  const double* u;                 // current vector: the means are u[0..2]
  double coef[3];                  // alpha_i / (sqrt(2 pi) sigma_i)
  double inv2s2[3];                // 1 / (2 sigma_i^2)
  double* partials;                // [6][grid]: sum x w_i, then sum w_i
};

constexpr int kEmWG = 256;
constexpr int kEmMaxGrid = 1024;

// Per sample k: p_i = alpha_i / (sqrt(2 pi) sigma_i) exp(-(x_k - mu_i)^2 /
// (2 sigma_i^2)), w_i = p_i / sum_j p_j; each lane accumulates x_k w_i and
// w_i over its samples (grid stride), then one fixed-order reduction per
// workgroup writes the workgroup's six partial sums.
__global__ __launch_bounds__(kEmWG) void k_em_partials(EmArgs a) {
  const double m0 = a.u[0], m1 = a.u[1], m2 = a.u[2];
  double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int64_t k = (int64_t)blockIdx.x * kEmWG + threadIdx.x; k < a.N;
       k += (int64_t)gridDim.x * kEmWG) {
    const double x = a.x[k];
    const double d0 = x - m0, d1 = x - m1, d2 = x - m2;
    const double p0 = a.coef[0] * exp(-(d0 * d0) * a.inv2s2[0]);
    const double p1 = a.coef[1] * exp(-(d1 * d1) * a.inv2s2[1]);
    const double p2 = a.coef[2] * exp(-(d2 * d2) * a.inv2s2[2]);
    const double tot = p0 + p1 + p2;
    const double w0 = p0 / tot, w1 = p1 / tot, w2 = p2 / tot;
    acc[0] += x * w0;
    acc[1] += x * w1;
    acc[2] += x * w2;
    acc[3] += w0;
    acc[4] += w1;
    acc[5] += w2;
  }
  const double r = multi_reduce<8>(acc);  // lane l < 8: value l over the wave
  __shared__ double s_w[kEmWG / 64][8];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane < 8) s_w[w][lane] = r;
  __syncthreads();
  if (threadIdx.x < 6) {
    double t = 0.0;
    for (int q = 0; q < kEmWG / 64; ++q) t += s_w[q][threadIdx.x];
    a.partials[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
  }
}

// Every workgroup sums the G partials of the six values in the same fixed
// order (so all agree bit for bit; a wave takes the values c, c + 4), forms
// G(mu)_i = sum x w_i / sum w_i and writes its share of the replicas: entry e
// is G(mu)_{e mod 3}, two entries a store in memory order.  (One wave summing
// and a thread writing each replica's three entries 24 bytes apart took 17.5
// us for 500,000 replicas.)
__global__ __launch_bounds__(kEmWG) void k_em_broadcast(const double* __restrict__ partials,
                                                        int G, double* __restrict__ out,
                                                        int64_t n) {
  __shared__ double s_t[6];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int c = w; c < 6; c += kEmWG / 64) {
    double v = 0.0;
    for (int g = lane; g < G; g += 64) v += partials[(size_t)c * G + g];
    v = wave_sum(v);
    if (lane == 0) s_t[c] = v;
  }
  __syncthreads();
  const double g0 = s_t[0] / s_t[3], g1 = s_t[1] / s_t[4], g2 = s_t[2] / s_t[5];
  // entries 2 r and 2 r + 1; the launch's stride (pairs) is a multiple of
  // three, so a thread's phase never changes
  const int64_t first = (int64_t)blockIdx.x * kEmWG + threadIdx.x;
  const int ph = (int)((2 * first) % 3);
  const double a = ph == 0 ? g0 : ph == 1 ? g1 : g2, b = ph == 0 ? g1 : ph == 1 ? g2 : g0;
  const int64_t npair = n / 2, stride = (int64_t)gridDim.x * kEmWG;
  for (int64_t r = first; r < npair; r += stride)
    *reinterpret_cast<f64x2_any*>(out + 2 * r) = f64x2_any{a, b};
  if ((n & 1) && first == 0) out[n - 1] = g2;  // n is a multiple of three
}

hipError_t launch_em(const double alpha[3], const double sigma[3], const double* x, int64_t N,
                     const double* u, double* out, int64_t n, double* work, hipStream_t st) {
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  EmArgs a{};
  a.x = x;
  a.N = N;
  a.u = u;
  for (int i = 0; i < 3; ++i) {
    a.coef[i] = alpha[i] * 0.39894228040143267793994605993438 / sigma[i];
    a.inv2s2[i] = 1.0 / (2.0 * sigma[i] * sigma[i]);
  }
  a.partials = work;
  int64_t g = (N + kEmWG - 1) / kEmWG;
  const int G = (int)(g > kEmMaxGrid ? kEmMaxGrid : g);
  hipLaunchKernelGGL(k_em_partials, dim3(G), dim3(kEmWG), 0, st, a);
  // a multiple of three workgroups (the stores' stride), at most three a
  // compute unit
  int64_t gb = (n / 2 + kEmWG - 1) / kEmWG;
  const int GB = (int)((gb < 768 ? (gb < 1 ? 1 : gb) : 768) + 2) / 3 * 3;
  hipLaunchKernelGGL(k_em_broadcast, dim3(GB), dim3(kEmWG), 0, st, work, G, out, n);
  return hipGetLastError();
}

hipError_t launch_fill_uniform(double* out, int64_t n, uint64_t seed, uint64_t stream_id,
                               uint64_t offset, double lo, double hi, hipStream_t st) {
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  int64_t blocks = (n + 255) / 256;
  int grid = (int)(blocks < 65536 ? blocks : 65536);
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(k_fill_uniform, dim3(grid), dim3(256), 0, st, out, n,
                     stream_base(seed, stream_id) + offset, lo, hi);
  return hipGetLastError();
}

hipError_t launch_fill_normal(double* out, int64_t n, uint64_t seed, uint64_t stream_id,
                              uint64_t offset, hipStream_t st) {
  (void)hipGetLastError();  // drop a stale error left by an earlier call
  int64_t blocks = (n + 255) / 256;
  int grid = (int)(blocks < 65536 ? blocks : 65536);
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(k_fill_normal, dim3(grid), dim3(256), 0, st, out, n,
                     stream_base(seed, stream_id), offset);
  return hipGetLastError();
}

}  // namespace aa
