// aa_batch_api.hip -- host side of the batched C ABI (aa_batch_* in aa.h).
//
// The workspace holds the instance descriptors, their device-updated states,
// the schedule (instance order and work counter) and, per instance, G(x),
// f_{i-1}, G(x_{i-1}), Delta f, Q, the Delta g history and the small dense
// block.  aa_batch_run enqueues, per iteration, one launch of the persistent
// kernel (aa_batch.hip) and the passes of the wide instances
// (aa_batch_wide.hip); with a non-NULL stream the sequence for a given
// iteration count is captured once as a HIP graph and replayed.
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <numeric>
#include <vector>

#include "aa_internal.h"

using namespace aa;

struct aa_batch {
  int count = 0, variant = 0;
  unsigned flags = 0;
  double tol = 0.0;
  int64_t max_iter = 0;
  hipStream_t stream = nullptr;
  BInst* d_inst = nullptr;
  BState* d_state = nullptr;
  int* d_order = nullptr;
  unsigned* d_counter = nullptr;
  std::vector<int64_t> n;
  std::vector<int> m;
  std::vector<int> dim;
  int kbucket = 8;
  int mmax = 1;         // largest window of the batch
  bool gram = false;
  int grid = 0;        // persistent workgroups (0: 2 per compute unit)
  int order_mode = 0;  // 0: largest n*m first, 1: as given
  bool use_graph = true;
  hipGraphExec_t exec = nullptr;
  int exec_iters = 0;
  bool learned = false;
  float* d_feat = nullptr;  // [count x AA_MLP_FEATURES]
  float* d_out = nullptr;   // [count x AA_MLP_OUTPUTS]
  float* d_dout = nullptr;  // [count x AA_MLP_OUTPUTS]
  int pairs = 4;            // row pairs per lane per tile of the persistent kernel
  // instances with many workgroups each (aa_batch_wide.hip): those the cost
  // model takes out of the persistent kernel for good, and those the split
  // policy adds once few are active
  int64_t split_min_n = 65536;  // 0: never, nor the cost model's
  int split_active_max = 0;     // split when at most this many are active (0: CUs / 4)
  std::vector<int> cost_wide, split;
  std::vector<BInst> hinst;      // host copies of the descriptors
  int* d_skip = nullptr;         // [count] kWideNo: in the persistent kernel
  WideItem* d_items = nullptr;   // [items_cap]
  WideItem* d_list = nullptr;    // [count]
  int64_t items_cap = 0;
  int nitems = 0, nwide = 0;     // chunks and instances of the wide passes
  double* d_partials = nullptr;  // shared by them
};

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
int64_t ld_of(int64_t n) { return (n + 63) / 64 * 64; }

bool valid_instance(const aa_batch_instance& I) {
  if (I.m < 1 || I.m > 64 || I.dim < 1 || I.dim > 3 || I.s < 1) return false;
  int64_t n = I.s;
  if (I.dim >= 2) n *= I.s;
  if (I.dim >= 3) n *= I.s;
  if (n != I.n || !(I.h > 0.0) || !I.d_f || !I.d_x) return false;
  if (((uintptr_t)I.d_f % 16) != 0 || ((uintptr_t)I.d_x % 16) != 0) return false;
  return true;
}

size_t instance_bytes(int64_t n, int m, bool learned) {
  const size_t vec = align_up((size_t)ld_of(n) * sizeof(double));
  size_t b = (learned ? 6 : 4) * vec + 2 * (size_t)m * vec;  // g, f_prev, g_prev, W, (xc, gc), Q, ring
  b += 2 * align_up(sizeof(double) * m * m);  // R, T
  b += 3 * align_up(sizeof(double) * m);      // coef0, coef1, gamma
  b += align_up(sizeof(double) * 2 * m);      // Givens
  b += align_up(sizeof(double) * S_COUNT);    // scalars
  b += align_up(sizeof(int));                 // status
  return b;
}

// Reduction partials of the wide passes (every instance's widest reduction,
// value by chunk): 199 values x 8192 workgroups, as a single-instance context
// holds.
constexpr size_t kWidePartials = (size_t)(3 * AA_MAX_COLS + 4) * 8192;
constexpr int64_t kWideTile = 1024;     // rows of a tile of the wide passes
constexpr int64_t kWideChunks = 512;    // most chunks of an instance
constexpr int64_t kWideMinN = 512;      // rows from which the cost model takes an
constexpr double kWideMinBytes = 0.7e6; // instance, and bytes of the largest
constexpr int64_t kWideMaxN = 1 << 30;  // their row indices are 32 bits in the stencil

int64_t wide_tiles(int64_t n) { return (n + kWideTile - 1) / kWideTile; }

int64_t wide_items_cap(int count, const aa_batch_instance* inst) {
  int64_t t = 0;
  for (int j = 0; j < count; ++j) t += std::min(wide_tiles(inst[j].n), kWideChunks);
  return t;
}

size_t header_bytes(int count, const aa_batch_instance* inst, bool learned) {
  size_t b = align_up(sizeof(BInst) * count) + align_up(sizeof(BState) * count) +
             align_up(sizeof(int) * count) + align_up(sizeof(unsigned));
  b += align_up(sizeof(int) * count) + align_up(sizeof(WideItem) * wide_items_cap(count, inst)) +
       align_up(sizeof(WideItem) * count) + align_up(sizeof(double) * kWidePartials);
  if (learned)
    b += align_up(sizeof(float) * count * kFeat) + 2 * align_up(sizeof(float) * count * kOuts);
  return b;
}

int bucket(int m) { return m <= 8 ? 8 : m <= 16 ? 16 : m <= 32 ? 32 : 64; }

void drop_graph(aa_batch* b) {
  if (b->exec) (void)hipGraphExecDestroy(b->exec);
  b->exec = nullptr;
  b->exec_iters = 0;
}

// all: the wide instances too (plain mode leaves them out otherwise).
hipError_t enqueue_mode(aa_batch* b, int mode, float dscale, bool all = false) {
  BatchArgs a{};
  a.inst = b->d_inst;
  a.state = b->d_state;
  a.order = b->d_order;
  a.count = b->count;
  a.counter = b->d_counter;
  a.variant = b->variant;
  a.flags = b->flags;
  a.tol = b->tol;
  a.max_iter = b->max_iter;
  a.ov_iter = -1;
  a.mode = mode;
  a.skip = mode == BM_PLAIN && b->nwide > 0 && !all ? b->d_skip : nullptr;
  a.feat = b->d_feat;
  a.out = b->d_out;
  a.dout = b->d_dout;
  a.dscale = dscale;
  int grid = b->grid;
  if (grid <= 0) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
      (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    grid = 2 * cus;
  }
  if (grid > b->count) grid = b->count;
  return launch_batch(a, grid, b->kbucket, b->gram,
                      batch_stage_cols(b->mmax, b->variant, b->flags), b->stream, b->pairs);
}

// Values of an instance's widest reduction in the wide passes.
int64_t wide_values(const aa_batch* b, int j) {
  const int64_t m = b->m[j];
  return std::max(3 * m + 4, b->gram ? m * (m + 1) / 2 : (int64_t)0);
}

// Vectors of n doubles a recycled iteration moves (fused ICWY: the others
// differ by what the threshold below does not see).
double iter_bytes(const aa_batch* b, int j) {
  return 8.0 * (double)b->n[j] * (4.0 * b->m[j] + 18.0);
}

// The instances that gain from many workgroups: those with more bytes than a
// threshold, the one that makes an iteration shortest in this model of both
// kernels (fitted to 2D tables of 1 to 4096 instances of side 8 to 512).  The
// persistent kernel takes 45 us and its bytes at 20 GB/s (MGS, whose passes over
// single columns stay in the L2, at 40) for an instance, the batch as long as its
// largest (times 1.2 beside others), as its share of the 512 resident workgroups
// (times 1.7) or as its bytes at 4.8 TB/s; the wide passes take 4.5 us a launch, 0.05 us an instance and the bytes at 5.1 TB/s.
// Measured, us an iteration, persistent / wide: 8 instances of side 64 to 256
// 1700 / 115, 32 of 32 to 128 (DCGS-2) 372 / 104, 2000 of 16 to 48 454 / 359,
// 4096 of 32 to 512 20757 / 20047; one of side 24, 48 and 64 at m = 5 46 / 53, 59
// / 59 and 65 / 60, of side 32 at m = 20 92 / 89; MGS at m = 20 of side 64 136 /
// 188, of side 96 256 / 183.
void choose_wide(aa_batch* b) {
  std::vector<int> ord(b->count);
  std::iota(ord.begin(), ord.end(), 0);
  std::stable_sort(ord.begin(), ord.end(),
                   [&](int x, int y) { return iter_bytes(b, x) > iter_bytes(b, y); });
  constexpr double kFixed = 45e-6, kAll = 4.8e12, kResident = 512.0;
  const double kOne = b->variant == AA_MGS ? 40e9 : 20e9;
  constexpr double kLaunch = 4.5e-6, kInst = 0.05e-6, kWide = 5.1e12;
  double total = 0.0;
  for (int j : ord) total += iter_bytes(b, j);
  const double passes = 12.0 + (b->variant == AA_MGS ? 2.0 * b->mmax : 0.0);
  auto cost = [&](double wide, int next) {  // the first `next` instances are wide
    double t = next > 0 ? passes * kLaunch + next * kInst + wide / kWide : 0.0;
    if (next < b->count) {
      const double rest = total - wide;
      t += std::max({1.2 * (kFixed + iter_bytes(b, ord[next]) / kOne),
                     1.7 * ((b->count - next) * kFixed + rest / kOne) / kResident, rest / kAll});
    }
    return t;
  };
  // by 3 % at least; by 30 % where both kernels run one after the other (the
  // model is no better than that: 2000 instances of side 16 to 48 took 513 us
  // divided, 454 persistent)
  const double all = cost(0.0, 0);
  double best = all, wide = 0.0;
  int take = 0;
  for (int i = 0; i < b->count; ++i) {
    // below 512 rows (one pair a lane) a pass's workgroup is not even filled;
    // where the largest has less than 0.7 MB (48^2 at m = 5) the launches cost
    // more than its one workgroup
    if (b->n[ord[i]] < kWideMinN || b->n[ord[i]] >= kWideMaxN ||
        iter_bytes(b, ord[0]) < kWideMinBytes)
      break;
    wide += iter_bytes(b, ord[i]);
    const double t = cost(wide, i + 1);
    if (t < best && t < (i + 1 < b->count ? 0.7 : 0.97) * all) {
      best = t;
      take = i + 1;
    }
  }
  b->cost_wide.assign(ord.begin(), ord.begin() + take);
}

// The cost model's choice, none while aa_batch_set_split has switched off.
const std::vector<int>& cost_set(const aa_batch* b) {
  static const std::vector<int> none;
  return b->split_min_n > 0 ? b->cost_wide : none;
}

// Chunks of every wide instance (largest first), their partials, the tables.
// Chunks are as long as leaves about 4096 of them, at most 16 tiles, longer
// where the tables or the partials would not hold them; instances that even
// one chunk each does not fit stay in the persistent kernel.
aa_status plan_wide(aa_batch* b) {
  // a replay enqueued before may still run: it ends before its graph goes
  if (b->exec && hipStreamSynchronize(b->stream) != hipSuccess) return AA_EHIP;
  drop_graph(b);
  std::vector<int> set = b->split;
  for (int j : cost_set(b))
    if (std::find(b->split.begin(), b->split.end(), j) == b->split.end()) set.push_back(j);
  std::stable_sort(set.begin(), set.end(),
                   [&](int x, int y) { return iter_bytes(b, x) > iter_bytes(b, y); });
  size_t room = 0, keep = 0;
  while (keep < set.size() && room + wide_values(b, set[keep]) <= kWidePartials)
    room += wide_values(b, set[keep++]);
  set.resize(keep);
  int64_t tiles = 0;
  for (int j : set) tiles += wide_tiles(b->n[j]);
  int64_t per = std::min<int64_t>(16, std::max<int64_t>(1, tiles / 4096));
  auto chunks = [&](int j) {
    const int64_t t = wide_tiles(b->n[j]);
    const int64_t q = std::max(per, (t + kWideChunks - 1) / kWideChunks);
    return (t + q - 1) / q;
  };
  for (;; per *= 2) {
    int64_t items = 0;
    size_t part = 0;
    for (int j : set) {
      items += chunks(j);
      part += (size_t)(wide_values(b, j) * chunks(j));
    }
    if (items <= b->items_cap && part <= kWidePartials) break;
  }
  std::vector<int> skip(b->count, (int)kWideNo);
  std::vector<WideItem> items, list;
  size_t off = 0;
  for (int j : set) {
    const int c = (int)chunks(j);
    skip[j] = std::find(b->split.begin(), b->split.end(), j) != b->split.end() ? kWideSplit
                                                                               : kWideCost;
    b->hinst[j].sm.partials = b->d_partials + off;
    off += (size_t)(wide_values(b, j) * c);
    list.push_back(WideItem{j, 0, c});
    for (int q = 0; q < c; ++q) items.push_back(WideItem{j, q, c});
  }
  for (size_t t = 0; t < b->split.size();)
    if (skip[b->split[t]] != kWideSplit) b->split.erase(b->split.begin() + t);
    else ++t;
  b->nitems = (int)items.size();
  b->nwide = (int)list.size();
  auto put = [&](void* dst, const void* src, size_t bytes) {
    return bytes == 0 ||
           hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, b->stream) == hipSuccess;
  };
  const bool ok = put(b->d_skip, skip.data(), sizeof(int) * skip.size()) &&
                  put(b->d_items, items.data(), sizeof(WideItem) * items.size()) &&
                  put(b->d_list, list.data(), sizeof(WideItem) * list.size()) &&
                  put(b->d_inst, b->hinst.data(), sizeof(BInst) * b->hinst.size()) &&
                  hipStreamSynchronize(b->stream) == hipSuccess;
  return ok ? AA_OK : AA_EHIP;
}

hipError_t enqueue_wide(aa_batch* b) {
  WideArgs a{};
  a.inst = b->d_inst;
  a.state = b->d_state;
  a.items = b->d_items;
  a.list = b->d_list;
  a.split = b->d_skip;
  a.variant = b->variant;
  a.flags = b->flags;
  a.tol = b->tol;
  a.max_iter = b->max_iter;
  a.kgram = b->kbucket < 16 ? 16 : b->kbucket;
  return launch_wide(a, b->nitems, b->nwide, b->kbucket, b->mmax, b->gram,
                     batch_stage_cols(b->mmax, b->variant, b->flags), b->stream);
}

// End the split policy's choices (the cost model's stay).
aa_status merge_split(aa_batch* b) {
  if (b->split.empty()) return AA_OK;
  b->split.clear();
  return plan_wide(b);
}

// Split policy, evaluated when a run starts: once at most split_active_max
// instances are active (the persistent kernel no longer fills the chip), the
// active instances with n >= split_min_n leave it; split instances that have
// stopped are dropped from the list.
aa_status update_split(aa_batch* b) {
  if (b->split_min_n <= 0) return AA_OK;
  std::vector<BState> hs(b->count);
  if (hipMemcpyAsync(hs.data(), b->d_state, sizeof(BState) * b->count, hipMemcpyDeviceToHost,
                     b->stream) != hipSuccess ||
      hipStreamSynchronize(b->stream) != hipSuccess)
    return AA_EHIP;
  bool changed = false;
  for (size_t t = 0; t < b->split.size();) {
    if (!hs[b->split[t]].active) {
      b->split.erase(b->split.begin() + t);
      changed = true;
    } else {
      ++t;
    }
  }
  int active = 0;
  for (const BState& st : hs) active += st.active ? 1 : 0;
  int amax = b->split_active_max;
  if (amax <= 0) {
    // a workgroup an instance: with a quarter of the compute units in use an
    // iteration takes as long as the largest instance
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess)
      (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    amax = cus / 4 > 1 ? cus / 4 : 1;
  }
  if (active > 0 && active <= amax)
    for (int j = 0; j < b->count; ++j)
      if (hs[j].active && !hs[j].pending && hs[j].iter >= 1 && b->n[j] >= b->split_min_n &&
          b->n[j] < kWideMaxN &&
          std::find(b->split.begin(), b->split.end(), j) == b->split.end()) {
        b->split.push_back(j);
        changed = true;
      }
  return changed ? plan_wide(b) : AA_OK;
}

// all: every instance in the persistent kernel.
hipError_t enqueue(aa_batch* b, int iters, bool all = false) {
  for (int i = 0; i < iters; ++i) {
    if (all || b->nwide < b->count) {
      const hipError_t e = enqueue_mode(b, BM_PLAIN, 0.f, all);
      if (e != hipSuccess) return e;
    }
    if (!all && b->nwide > 0) {
      const hipError_t e = enqueue_wide(b);
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

}  // namespace

extern "C" {

aa_status aa_batch_workspace_size(int count, const aa_batch_instance* inst, int variant,
                                  unsigned flags, size_t* bytes) {
  if (count < 1 || !inst || !bytes || variant < AA_MGS || variant > AA_ICWY) return AA_EINVAL;
  if (flags & AA_ICWY_T_TRANSFORM) return AA_EINVAL;  // one-workgroup step: Gram refresh only
  const bool learned = (flags & AA_BATCH_LEARNED) != 0;
  for (int j = 0; j < count; ++j)
    if (!valid_instance(inst[j])) return AA_EINVAL;
  size_t tot = header_bytes(count, inst, learned);
  for (int j = 0; j < count; ++j) {
    if (learned && inst[j].m > kWin) return AA_EINVAL;  // features cover a 20-column window
    tot += instance_bytes(inst[j].n, inst[j].m, learned);
  }
  *bytes = tot;
  return AA_OK;
}

aa_status aa_batch_init(aa_batch** out, int count, const aa_batch_instance* inst, int variant,
                        unsigned flags, double tol, int64_t max_iter, void* d_ws,
                        size_t bytes, void* stream) {
  if (!out) return AA_EINVAL;
  *out = nullptr;
  size_t need = 0;
  aa_status s = aa_batch_workspace_size(count, inst, variant, flags, &need);
  if (s != AA_OK) return s;
  if (!d_ws || ((uintptr_t)d_ws % kAlign) != 0 || !(tol >= 0.0) || max_iter < 1)
    return AA_EINVAL;
  if (bytes < need) return AA_ENOSPACE;
  aa_batch* b = new (std::nothrow) aa_batch();
  if (!b) return AA_EINVAL;
  b->count = count;
  b->variant = variant;
  b->flags = flags;
  b->tol = tol;
  b->max_iter = max_iter;
  b->stream = (hipStream_t)stream;
  char* base = (char*)d_ws;
  size_t o = 0;
  b->d_inst = (BInst*)(base + o); o = align_up(o + sizeof(BInst) * count);
  b->d_state = (BState*)(base + o); o = align_up(o + sizeof(BState) * count);
  b->d_order = (int*)(base + o); o = align_up(o + sizeof(int) * count);
  b->d_counter = (unsigned*)(base + o); o = align_up(o + sizeof(unsigned));
  b->d_skip = (int*)(base + o); o = align_up(o + sizeof(int) * count);
  b->items_cap = wide_items_cap(count, inst);
  b->d_items = (WideItem*)(base + o); o = align_up(o + sizeof(WideItem) * b->items_cap);
  b->d_list = (WideItem*)(base + o); o = align_up(o + sizeof(WideItem) * count);
  b->d_partials = (double*)(base + o); o = align_up(o + sizeof(double) * kWidePartials);
  b->learned = (flags & AA_BATCH_LEARNED) != 0;
  if (b->learned) {
    b->d_feat = (float*)(base + o); o = align_up(o + sizeof(float) * count * kFeat);
    b->d_out = (float*)(base + o); o = align_up(o + sizeof(float) * count * kOuts);
    b->d_dout = (float*)(base + o); o = align_up(o + sizeof(float) * count * kOuts);
  }
  std::vector<BInst> hi(count);
  std::vector<BState> hs(count);
  int mmax = 1;
  for (int j = 0; j < count; ++j) {
    const aa_batch_instance& A = inst[j];
    BInst& I = hi[j];
    const int64_t ld = ld_of(A.n);
    const size_t vec = align_up((size_t)ld * sizeof(double));
    const int m = A.m;
    I.n = A.n; I.ld = ld; I.m = m; I.dim = A.dim; I.s = A.s;
    I.h = A.h; I.omega = A.omega; I.c = A.c;
    I.f = A.d_f; I.x = A.d_x;
    I.g = (double*)(base + o); o += vec;
    I.f_prev = (double*)(base + o); o += vec;
    I.g_prev = (double*)(base + o); o += vec;
    I.W = (double*)(base + o); o += vec;
    if (b->learned) {
      I.xc = (double*)(base + o); o += vec;
      I.gc = (double*)(base + o); o += vec;
    }
    I.Q = (double*)(base + o); o += vec * m;
    I.ring = (double*)(base + o); o += vec * m;
    Small& sm = I.sm;
    sm.R = (double*)(base + o); o = align_up(o + sizeof(double) * m * m);
    sm.T = (double*)(base + o); o = align_up(o + sizeof(double) * m * m);
    sm.coef0 = (double*)(base + o); o = align_up(o + sizeof(double) * m);
    sm.coef1 = (double*)(base + o); o = align_up(o + sizeof(double) * m);
    sm.gamma = (double*)(base + o); o = align_up(o + sizeof(double) * m);
    sm.givens = (double*)(base + o); o = align_up(o + sizeof(double) * 2 * m);
    sm.scal = (double*)(base + o); o = align_up(o + sizeof(double) * S_COUNT);
    sm.status = (int*)(base + o); o = align_up(o + sizeof(int));
    sm.partials = nullptr;
    sm.cap = m;
    sm.stop = nullptr;  // batched instances stop by their own per-instance test
    BState& st = hs[j];
    st.iter = 0; st.conv_iter = -1; st.k = 0; st.m_i = 0; st.active = 1; st.status = 0;
    st.res_norm = st.res0_norm = 0.0;
    st.g_evals = st.accepted = 0;
    st.loss = 0.0;
    st.pending = st.g_valid = 0;
    b->n.push_back(A.n);
    b->m.push_back(m);
    b->dim.push_back(A.dim);
    mmax = std::max(mmax, m);
  }
  b->kbucket = bucket(mmax);
  b->mmax = mmax;
  b->gram = batch_needs_gram(variant, flags);
  b->hinst = hi;
  choose_wide(b);
  hipError_t e = hipMemcpyAsync(b->d_state, hs.data(), sizeof(BState) * count,
                                hipMemcpyHostToDevice, b->stream);
  // plan_wide stores the descriptors and waits
  if (e != hipSuccess || plan_wide(b) != AA_OK ||
      launch_batch_init(b->d_inst, count, b->d_counter, b->stream) != hipSuccess) {
    delete b;
    return AA_EHIP;
  }
  if (aa_batch_set_schedule(b, 0, 0, 1) != AA_OK) {
    delete b;
    return AA_EHIP;
  }
  *out = b;
  return AA_OK;
}

aa_status aa_batch_set_schedule(aa_batch* b, int grid, int order, int use_graph) {
  if (!b || grid < 0 || grid > 65536 || order < 0 || order > 1) return AA_EINVAL;
  std::vector<int> ord(b->count);
  std::iota(ord.begin(), ord.end(), 0);
  if (order == 0)
    std::stable_sort(ord.begin(), ord.end(), [&](int a, int c) {
      return b->n[a] * b->m[a] > b->n[c] * b->m[c];
    });
  if (hipMemcpyAsync(b->d_order, ord.data(), sizeof(int) * b->count, hipMemcpyHostToDevice,
                     b->stream) != hipSuccess ||
      hipStreamSynchronize(b->stream) != hipSuccess)
    return AA_EHIP;
  b->grid = grid;
  b->order_mode = order;
  b->use_graph = use_graph != 0;
  drop_graph(b);
  return AA_OK;
}

aa_status aa_batch_set_split(aa_batch* b, int64_t min_n, int active_max) {
  if (!b || min_n < 0 || active_max < 0) return AA_EINVAL;
  const bool was_on = b->split_min_n > 0, on = min_n > 0;
  b->split_min_n = min_n;
  b->split_active_max = active_max;
  if (on == was_on) return AA_OK;
  if (!on) b->split.clear();
  return plan_wide(b);
}

aa_status aa_batch_split_count(const aa_batch* b, int* count) {
  if (!b || !count) return AA_EINVAL;
  *count = (int)b->split.size();
  return AA_OK;
}

aa_status aa_batch_set_tiles(aa_batch* b, int pairs) {
  if (!b || (pairs != 2 && pairs != 4)) return AA_EINVAL;
  b->pairs = pairs;
  drop_graph(b);
  return AA_OK;
}

aa_status aa_batch_autotune(aa_batch* b, int iters, const char* cache_path,
                            aa_batch_schedule* best) {
  if (!b || iters < 1) return AA_EINVAL;
  // the split policy's instances go back first: the schedule is chosen for
  // the batch as it starts
  if (merge_split(b) != AA_OK) return AA_EHIP;
  // The schedule is the persistent kernel's.  A learned batch's entry points run
  // every instance there, a plain run those that are not wide; so do the trials.
  const bool all = b->learned;
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
    return AA_EHIP;
  const int cus = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
  // FNV-1a over the workload: variant, flags, every instance's (n, m, dim) and
  // whether the trials leave it out
  std::vector<char> out(b->count, 0);
  if (!all)
    for (int j : cost_set(b)) out[j] = 1;
  uint64_t sig = 1469598103934665603ull;
  auto mix = [&](uint64_t v) {
    for (int i = 0; i < 8; ++i) {
      sig ^= (v >> (8 * i)) & 0xffu;
      sig *= 1099511628211ull;
    }
  };
  mix(3u);  // cache format: grid, order, row pairs; instances left out
  mix((uint64_t)b->variant);
  mix((uint64_t)b->flags);
  for (int j = 0; j < b->count; ++j) {
    mix((uint64_t)b->n[j]);
    mix((uint64_t)b->m[j]);
    mix((uint64_t)b->dim[j]);
    mix((uint64_t)out[j]);
  }
  char sigs[32];
  snprintf(sigs, sizeof sigs, "%016llx", (unsigned long long)sig);
  const bool graph = b->use_graph;
  if (cache_path) {
    // the last line matching this device and workload wins
    bool hit = false;
    aa_batch_schedule got{0, 0, 0.0, 0, 4};
    if (FILE* fh = fopen(cache_path, "r")) {
      char line[512], arch[128], s2[64];
      int g = 0, o = 0, pr = 0;
      double ms = 0.0;
      while (fgets(line, sizeof line, fh))
        if (sscanf(line, "%127s %63s %d %d %d %lf", arch, s2, &g, &o, &pr, &ms) == 6 &&
            strcmp(arch, prop.gcnArchName) == 0 && strcmp(s2, sigs) == 0 && g >= 0 && o >= 0 &&
            o <= 1 && (pr == 2 || pr == 4)) {
          hit = true;
          got = aa_batch_schedule{g, o, ms, 0, pr};
        }
      fclose(fh);
    }
    if (hit) {
      aa_status st = aa_batch_set_tiles(b, got.pairs);
      if (st == AA_OK) st = aa_batch_set_schedule(b, got.grid, got.order, graph);
      if (st != AA_OK) return st;
      if (best) *best = got;
      return AA_OK;
    }
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    return AA_EHIP;
  }
  aa_status st = AA_OK;
  aa_batch_schedule win{0, 0, 1e300, 0, 4};
  auto trial = [&](float& ms) {
    return hipEventRecord(e0, b->stream) == hipSuccess && enqueue(b, iters, all) == hipSuccess &&
           hipEventRecord(e1, b->stream) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
           hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
  };
  if (!all && b->nwide == b->count) {
    // no instance in the persistent kernel: nothing to choose.  The schedule
    // stays, timed once, and is no entry of the cache.
    float ms = 0.f;
    const bool ok = trial(ms);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (!ok) return AA_EHIP;
    if (best) *best = aa_batch_schedule{b->grid, b->order_mode, ms / iters, 1, b->pairs};
    return AA_OK;
  }
  // tiles (row pairs per lane: 4 or 2) x persistent workgroups per compute
  // unit x instance order
  for (int pr = 4; pr >= 2 && st == AA_OK; pr -= 2) {
    b->pairs = pr;
    for (int per = 1; per <= 4 && st == AA_OK; ++per) {
      const int g = std::min(per * cus, b->count);
      if (per > 1 && g == std::min((per - 1) * cus, b->count)) break;  // capped: no new candidate
      for (int o = 0; o <= 1 && st == AA_OK; ++o) {
        st = aa_batch_set_schedule(b, g, o, 0);
        if (st != AA_OK) break;
        float ms = 0.f;
        if (!trial(ms)) {
          st = AA_EHIP;
          break;
        }
        win.trials += 1;
        if (ms / iters < win.ms_per_iter) {
          win.grid = g;
          win.order = o;
          win.pairs = pr;
          win.ms_per_iter = ms / iters;
        }
      }
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (st != AA_OK) return st;
  b->pairs = win.pairs;
  st = aa_batch_set_schedule(b, win.grid, win.order, graph);
  if (st != AA_OK) return st;
  if (cache_path) {
    if (FILE* fh = fopen(cache_path, "a")) {
      fprintf(fh, "%s %s %d %d %d %.6f\n", prop.gcnArchName, sigs, win.grid, win.order,
              win.pairs, win.ms_per_iter);
      fclose(fh);
    }
  }
  if (best) *best = win;
  return AA_OK;
}

aa_status aa_batch_run(aa_batch* b, int iters) {
  if (!b || iters < 0) return AA_EINVAL;
  if (iters == 0) return AA_OK;
  if (b->split_min_n > 0) {
    const aa_status s = update_split(b);
    if (s != AA_OK) return s;
  }
  if (!b->use_graph || b->stream == nullptr) return enqueue(b, iters) == hipSuccess ? AA_OK : AA_EHIP;
  if (b->exec_iters != iters) {
    drop_graph(b);
    hipGraph_t g = nullptr;
    if (hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
      return AA_EHIP;
    hipError_t e = enqueue(b, iters);
    hipError_t e2 = hipStreamEndCapture(b->stream, &g);
    if (e != hipSuccess || e2 != hipSuccess || !g) {
      if (g) (void)hipGraphDestroy(g);
      return AA_EHIP;
    }
    e = hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess) {
      b->exec = nullptr;
      return AA_EHIP;
    }
    b->exec_iters = iters;
  }
  return hipGraphLaunch(b->exec, b->stream) == hipSuccess ? AA_OK : AA_EHIP;
}

aa_status aa_batch_read(aa_batch* b, aa_batch_state* states, int* active) {
  if (!b) return AA_EINVAL;
  std::vector<BState> hs(b->count);
  if (hipMemcpyAsync(hs.data(), b->d_state, sizeof(BState) * b->count, hipMemcpyDeviceToHost,
                     b->stream) != hipSuccess ||
      hipStreamSynchronize(b->stream) != hipSuccess)
    return AA_EHIP;
  if (states) memcpy(states, hs.data(), sizeof(BState) * b->count);
  if (active) {
    int a = 0;
    for (const BState& st : hs) a += st.active ? 1 : 0;
    *active = a;
  }
  return AA_OK;
}

aa_status aa_batch_run_learned(aa_batch* b, aa_mlp* net, int iters) {
  if (!b || !net || iters < 0 || !b->learned) return AA_EINVAL;
  if (mlp_stream(net) != b->stream || mlp_max_batch(net) < b->count) return AA_EINVAL;
  if (merge_split(b) != AA_OK) return AA_EHIP;  // the learned step is one-workgroup only
  for (int i = 0; i < iters; ++i) {
    if (enqueue_mode(b, BM_PHASE_A, 0.f) != hipSuccess) return AA_EHIP;
    aa_status s = aa_mlp_forward(net, b->count, b->d_feat, b->d_out);
    if (s != AA_OK) return s;
    if (enqueue_mode(b, BM_GUARD, 0.f) != hipSuccess) return AA_EHIP;
  }
  return AA_OK;
}

aa_status aa_batch_train(aa_batch* b, aa_mlp* net, int iters, float lr) {
  if (!b || !net || iters < 0 || !b->learned || !(lr >= 0.f)) return AA_EINVAL;
  if (mlp_stream(net) != b->stream || mlp_max_batch(net) < b->count) return AA_EINVAL;
  if (merge_split(b) != AA_OK) return AA_EHIP;
  const float dscale = 1.0f / (float)b->count;
  for (int i = 0; i < iters; ++i) {
    if (enqueue_mode(b, BM_PHASE_A, 0.f) != hipSuccess) return AA_EHIP;
    aa_status s = aa_mlp_forward(net, b->count, b->d_feat, b->d_out);
    if (s != AA_OK) return s;
    if (enqueue_mode(b, BM_TRAIN, dscale) != hipSuccess) return AA_EHIP;
    s = aa_mlp_backward(net, b->count, b->d_dout);
    if (s != AA_OK) return s;
    s = aa_mlp_adam(net, lr, 0.9f, 0.999f, 1e-8f);
    if (s != AA_OK) return s;
  }
  return AA_OK;
}

aa_status aa_batch_read_learning(aa_batch* b, float* feat, float* out, float* dout) {
  if (!b || !b->learned) return AA_EINVAL;
  const size_t c = (size_t)b->count;
  if ((feat && hipMemcpyAsync(feat, b->d_feat, sizeof(float) * c * kFeat, hipMemcpyDeviceToHost,
                              b->stream) != hipSuccess) ||
      (out && hipMemcpyAsync(out, b->d_out, sizeof(float) * c * kOuts, hipMemcpyDeviceToHost,
                             b->stream) != hipSuccess) ||
      (dout && hipMemcpyAsync(dout, b->d_dout, sizeof(float) * c * kOuts, hipMemcpyDeviceToHost,
                              b->stream) != hipSuccess) ||
      hipStreamSynchronize(b->stream) != hipSuccess)
    return AA_EHIP;
  return AA_OK;
}

aa_status aa_batch_destroy(aa_batch* b) {
  if (!b) return AA_OK;
  drop_graph(b);
  delete b;
  return AA_OK;
}

}  // extern "C"
