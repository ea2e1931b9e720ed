// Verification step that follows drafting (paper Sec. 2): the target model
// scores the drafted tokens in one pass, and the drafts are kept while they
// pass the test -- greedy: the target's own arg-max equals the draft;
// sampled: the rejection rule r < min(1, p_target(x) / p_draft(x)), with the
// replacement drawn from max(0, p_target - p_draft) at the first rejection,
// or one extra token from p_target when all pass.  Trees (greedy): the
// longest root path whose every node is the target's choice at its parent.
//
// Logits rows are V-wide fp32 (0.5 MB at V = 128256), so the work is a
// stream over them, bound by HBM: each row is split over several workgroups,
// which reduce their slices to (max z, sum exp(z - max)), z = logit / T
// (sampled), or to the arg-max (greedy).  A sampled call then decides per
// sequence and sums the weights of the one row it draws from, again a slice
// per workgroup, and one workgroup per sequence walks the slice that holds
// the draw: 8B vocabulary, batch 16, K 5 (90 MB), 75.7 -> 34.3 us per call
// (one workgroup per sequence summing and walking its whole row took 39 us
// alone).  Draws use the drafter's inverse CDF in token-id order.
#include <cstdarg>
#include <cstdio>
#include <mutex>

#include "device.h"
#include "prism_draft.h"

namespace prism {

constexpr int VSPLIT = 8;        // slices per row at least
constexpr int VSPLIT_MAX = 32;   // and at most (8, 16 or 32)
constexpr int VSPLIT_WGS = 1024; // as long as the slices of all rows stay within this many
constexpr int VER_UNROLL = 4;

// Slices per row of a call over `rows` rows: 8 (16032 ids of the 8B
// vocabulary, four batches of 16-byte loads per thread) once that fills the
// chip, more for few rows, where the call is the latency of one slice.
static int row_slices(int rows) {
  int n = VSPLIT;
  while (n < VSPLIT_MAX && rows * n * 2 <= VSPLIT_WGS) n *= 2;
  return n;
}

struct SoftStat {     // one slice of one row: softmax statistics of z = logit / T
  float mx, sum;
};
struct BestStat {     // arg-max (the lowest id if several)
  float best;
  int arg;
};

// slice of a row: ids [lo, hi), both multiples of 4 (V is a multiple of 16)
__device__ __forceinline__ void slice_of(int V, int part, int parts, int &lo, int &hi) {
  const int per = (((V + parts - 1) / parts) + 3) & ~3;
  lo = min(V, part * per);
  hi = min(V, lo + per);
}

// Softmax statistics of rows0 rows of x0, then of the rows of x1.  A thread
// keeps a running (max, sum) and takes 16 values at a time: one rescale per
// batch and one exponential per value.  (Rescaling value by value, with both
// sides of the branch run, cost two: 19 us for 49 MB.)
__global__ __launch_bounds__(256) void k_rows_soft(const float *__restrict__ x0, int rows0,
                                                   const float *__restrict__ x1, int V, float inv_t,
                                                   SoftStat *out) {
  __shared__ float sh[8];
  const int row = blockIdx.y, part = blockIdx.x, parts = gridDim.x, tid = threadIdx.x;
  int lo, hi;
  slice_of(V, part, parts, lo, hi);
  const float *r = row < rows0 ? x0 + (size_t)row * V : x1 + (size_t)(row - rows0) * V;
  float m = -INFINITY, s = 0.f;
  for (int i0 = lo + 4 * tid; i0 < hi; i0 += 4 * 256 * VER_UNROLL) {
    f32x4 v[VER_UNROLL];
#pragma unroll
    for (int u = 0; u < VER_UNROLL; ++u) {
      const int i = i0 + u * 4 * 256;
      v[u] = *(const f32x4 *)(r + (i < hi ? i : i0));
      if (i >= hi) v[u] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    }
    float mn = m;
#pragma unroll
    for (int u = 0; u < VER_UNROLL; ++u) {
      v[u] *= inv_t;
      mn = fmaxf(mn, fmaxf(fmaxf(v[u].x, v[u].y), fmaxf(v[u].z, v[u].w)));
    }
    const float ref = mn == -INFINITY ? 0.f : mn;   // only -inf so far: every term is 0
    s *= expf(m - ref);
#pragma unroll
    for (int u = 0; u < VER_UNROLL; ++u)
      s += (expf(v[u].x - ref) + expf(v[u].y - ref)) + (expf(v[u].z - ref) + expf(v[u].w - ref));
    m = mn;
  }
  const float M = block_max<4>(m, sh);
  const float S = block_sum<4>(m == -INFINITY ? 0.f : s * expf(m - M), sh);
  if (tid == 0) out[(size_t)row * parts + part] = SoftStat{M, S};
}

// Arg-max of each row's slice.  A thread's ids ascend, so a strictly larger
// value is taken; a thread that saw none above -inf looks for its first -inf.
__global__ __launch_bounds__(256) void k_rows_best(const float *__restrict__ x, int V, BestStat *out) {
  __shared__ float shv[8];
  __shared__ int shi[8];
  const int row = blockIdx.y, part = blockIdx.x, parts = gridDim.x, tid = threadIdx.x;
  int lo, hi;
  slice_of(V, part, parts, lo, hi);
  const float *r = x + (size_t)row * V;
  float bv = -INFINITY;
  int bi = NO_TOKEN;
  for (int i0 = lo + 4 * tid; i0 < hi; i0 += 4 * 256 * VER_UNROLL) {
    f32x4 v[VER_UNROLL];
#pragma unroll
    for (int u = 0; u < VER_UNROLL; ++u) {   // all loads first
      const int i = i0 + u * 4 * 256;
      v[u] = *(const f32x4 *)(r + (i < hi ? i : i0));   // past the end: i0 again, never larger
    }
#pragma unroll
    for (int u = 0; u < VER_UNROLL; ++u) {
      const int i = i0 + u * 4 * 256;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool take = v[u][q] > bv;
        bv = take ? v[u][q] : bv;
        bi = take ? i + q : bi;
      }
    }
  }
  if (bi == NO_TOKEN)
    for (int i0 = lo + 4 * tid; i0 < hi && bi == NO_TOKEN; i0 += 4 * 256)
      for (int q = 3; q >= 0; --q)
        if (r[i0 + q] == -INFINITY) bi = i0 + q;
  block_argmax<4>(bv, bi, shv, shi);
  if (tid == 0) out[(size_t)row * parts + part] = BestStat{bv, bi};
}

// merges of one row's slices, in slice order
struct RowSum {
  float M, S;
};
template <int P>
__device__ __forceinline__ RowSum merge_soft_n(const SoftStat *st) {
  SoftStat v[P];
#pragma unroll
  for (int p = 0; p < P; ++p) v[p] = st[p];   // all loads first
  float M = -INFINITY, S = 0.f;
#pragma unroll
  for (int p = 0; p < P; ++p) M = fmaxf(M, v[p].mx);
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (v[p].mx != -INFINITY) S += v[p].sum * expf(v[p].mx - M);
  return RowSum{M, S};
}
__device__ __forceinline__ RowSum merge_soft(const SoftStat *st, int parts) {   // row_slices
  if (parts == VSPLIT) return merge_soft_n<VSPLIT>(st);
  if (parts == 2 * VSPLIT) return merge_soft_n<2 * VSPLIT>(st);
  return merge_soft_n<VSPLIT_MAX>(st);
}
__device__ __forceinline__ int merge_best(const BestStat *st, int parts) {
  float bv = -INFINITY;
  int bi = NO_TOKEN;
#pragma unroll 8
  for (int p = 0; p < parts; ++p) {
    const BestStat v = st[p];
    if (better(v.best, v.arg, bv, bi)) { bv = v.best; bi = v.arg; }
  }
  return bi;
}

constexpr int VER_MAXK = 64;      // drafts per sequence (max_steps <= 63)
constexpr int DRAW_SLICES = 32;   // slices of the row a sequence draws from

// What a sequence draws from, left by its decision: the target row n, alone
// (mode 0) or less the draft row (mode 1, the residual at a rejection), their
// softmax statistics, and the weight of each slice in id order.
struct Draw {
  int n, mode;
  RowSum t, d;
  float sum[DRAW_SLICES];
};

struct VerifyChainArgs {
  int K, V, parts;
  float inv_t;                   // 0: greedy
  const float *tl, *dl;          // [B, K+1, V], [B, K, V]
  const SoftStat *ts, *ds;       // sampled: [B*(K+1)][parts], [B*K][parts]
  const BestStat *best;          // greedy: [B*(K+1)][parts]
  Draw *draw;                    // sampled: [B]
  const int32_t *drafts;         // [B, K]
  const float *u;                // [B, K+1]
  int32_t *n_acc, *next;         // [B]
  uint32_t *err;
};

// Weights of ids i..i+3 of a sequence's draw (0 past the row): p_target up to
// its normaliser, or max(0, p_target - p_draft).
__device__ __forceinline__ f32x4 draw_weights(const Draw &w, int mode, const f32x4 &t, const f32x4 &d,
                                              float it) {
  f32x4 v;
  if (mode == 1) {
    const float ist = 1.f / w.t.S, isd = 1.f / w.d.S;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      v[q] = fmaxf(0.f, expf(t[q] * it - w.t.M) * ist - expf(d[q] * it - w.d.M) * isd);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = expf(t[q] * it - w.t.M);
  }
  return v;
}

// this thread's share of the weights of ids [lo, hi), the loads of a batch
// issued together
__device__ __forceinline__ float slice_weight(const VerifyChainArgs &a, const Draw &w, int mode,
                                              const float *trow, const float *drow, int lo, int hi) {
  float acc = 0.f;
  for (int i0 = lo + 4 * (int)threadIdx.x; i0 < hi; i0 += 4 * 256 * VER_UNROLL) {
    f32x4 t[VER_UNROLL], d[VER_UNROLL];
#pragma unroll
    for (int u = 0; u < VER_UNROLL; ++u) {
      const int i = i0 + u * 4 * 256;
      t[u] = *(const f32x4 *)(trow + (i < hi ? i : i0));
      d[u] = mode == 1 ? *(const f32x4 *)(drow + (i < hi ? i : i0)) : t[u];
    }
#pragma unroll
    for (int u = 0; u < VER_UNROLL; ++u) {
      if (i0 + u * 4 * 256 >= hi) continue;
      const f32x4 v = draw_weights(w, mode, t[u], d[u], a.inv_t);
      acc += (v.x + v.y) + (v.z + v.w);
    }
  }
  return acc;
}

// One workgroup per (slice, sequence): the sequence's decision (every
// workgroup takes it from the row statistics), and the weight of its slice
// of the row drawn from.
__global__ __launch_bounds__(256) void k_verify_decide(VerifyChainArgs a) {
  __shared__ Draw w;
  __shared__ RowSum s_t[VER_MAXK + 1], s_d[VER_MAXK];
  __shared__ float sh[8];
  const int b = blockIdx.y, part = blockIdx.x, tid = threadIdx.x;
  const int K = a.K, V = a.V;
  // lane i of wave 0: draft i and its rows; wave 1: the target rows' statistics
  float lt = 0.f, ld = 0.f, r = 0.f;
  int x = -1;
  if (tid < K) {
    x = a.drafts[(size_t)b * K + tid];
    r = a.u[(size_t)b * (K + 1) + tid];
    if (x < 0 || x >= V) x = -1;
    if (x < 0 && part == 0) atomicOr(a.err, ERRF_TOKEN);
    if (x >= 0) {
      lt = a.tl[((size_t)b * (K + 1) + tid) * V + x];
      ld = a.dl[((size_t)b * K + tid) * V + x];
    }
    s_d[tid] = merge_soft(a.ds + ((size_t)b * K + tid) * a.parts, a.parts);
  } else if (tid >= 64 && tid - 64 <= K) {
    s_t[tid - 64] = merge_soft(a.ts + ((size_t)b * (K + 1) + tid - 64) * a.parts, a.parts);
  }
  __syncthreads();
  if (tid < 64) {   // K <= 63: the first draft not kept is one ballot
    bool stop = tid >= K;
    if (tid < K && x >= 0) {
      const float pt = expf(lt * a.inv_t - s_t[tid].M) / s_t[tid].S;
      const float pd = expf(ld * a.inv_t - s_d[tid].M) / s_d[tid].S;
      stop = !(r < fminf(1.f, pt / pd));
    } else if (tid < K) {
      stop = true;   // an invalid draft is never kept
    }
    const int n = __ffsll((long long)__ballot(stop)) - 1;   // lane K always stops
    const int xn = __shfl(x, n, 64);
    if (tid == 0) {
      w.n = n;
      w.mode = n < K && xn >= 0 ? 1 : 0;
      w.t = s_t[n];
      w.d = n < K ? s_d[n] : s_t[n];
    }
  }
  __syncthreads();
  const float *trow = a.tl + ((size_t)b * (K + 1) + w.n) * V;
  const float *drow = w.mode == 1 ? a.dl + ((size_t)b * K + w.n) * V : trow;
  int lo, hi;
  slice_of(V, part, DRAW_SLICES, lo, hi);
  const float sum = block_sum<4>(slice_weight(a, w, w.mode, trow, drow, lo, hi), sh);
  if (tid == 0) {
    Draw *o = a.draw + b;
    o->sum[part] = sum;
    if (part == 0) {
      o->n = w.n;
      o->mode = w.mode;
      o->t = w.t;
      o->d = w.d;
    }
  }
}

// the first of n in-order sums that carries the running total past goal: its
// index and the total before it; none (rounding): the last positive one, with
// the goal moved to +inf
__device__ __forceinline__ void pick_in_order(const float *sums, int n, float goal, int &pick, float &at,
                                              float &g) {
  float run = 0.f;
  pick = -1;
  at = 0.f;
  g = goal;
  for (int i = 0; i < n; ++i) {
    if (sums[i] > 0.f && run + sums[i] > goal) { pick = i; at = run; return; }
    run += sums[i];
  }
  for (int i = n - 1; i >= 0; --i)
    if (sums[i] > 0.f) { pick = i; break; }
  g = INFINITY;
}

// One workgroup per sequence: the slice that holds u * total, then inside it
// 4096 ids at a time (16 consecutive ones per thread) an in-order prefix over
// the threads, and the thread that holds the goal walks its 16.  Rounding
// that leaves no crossing takes the highest id of positive weight of the
// slice.  A residual of no weight (identical distributions) draws from the
// target row instead.
__global__ __launch_bounds__(256) void k_verify_draw(VerifyChainArgs a) {
  __shared__ Draw w;
  __shared__ float sh[8], s_wave[4];
  __shared__ int s_found, s_last, s_pick;
  __shared__ float s_at, s_goal;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int K = a.K, V = a.V;
  for (int i = tid; i < (int)(sizeof(Draw) / 4); i += 256) ((int *)&w)[i] = ((const int *)(a.draw + b))[i];
  const float u = fminf(fmaxf(a.u[(size_t)b * (K + 1) + K], 0.f), 1.f);
  __syncthreads();
  const float *trow = a.tl + ((size_t)b * (K + 1) + w.n) * V;
  int mode = w.mode;
  for (;;) {
    if (tid == 0) {
      float total = 0.f, at, g;
      int pick;
#pragma unroll
      for (int i = 0; i < DRAW_SLICES; ++i) total += w.sum[i];
      pick_in_order(w.sum, DRAW_SLICES, u * total, pick, at, g);
      s_pick = pick;
      s_at = at;
      s_goal = g;
      s_found = s_last = -1;
    }
    __syncthreads();
    if (s_pick >= 0 || mode == 0) break;    // uniform
    mode = 0;
    for (int p = 0; p < DRAW_SLICES; ++p) {
      int lo, hi;
      slice_of(V, p, DRAW_SLICES, lo, hi);
      const float sum = block_sum<4>(slice_weight(a, w, 0, trow, trow, lo, hi), sh);
      if (tid == 0) w.sum[p] = sum;
    }
    __syncthreads();
  }
  if (s_pick >= 0) {   // uniform
    const float *drow = mode == 1 ? a.dl + ((size_t)b * K + w.n) * V : trow;
    int lo, hi;
    slice_of(V, s_pick, DRAW_SLICES, lo, hi);
    float run = s_at;
    const float goal = s_goal;
    for (int c = lo; c < hi && s_found < 0; c += 4096) {   // s_found: uniform past the barrier
      const int i0 = c + 16 * tid;
      f32x4 t[4], d[4], v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = i0 + 4 * q < hi ? i0 + 4 * q : lo;
        t[q] = *(const f32x4 *)(trow + i);
        d[q] = mode == 1 ? *(const f32x4 *)(drow + i) : t[q];
      }
      float ls = 0.f;
      int last = -1;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v[q] = i0 + 4 * q < hi ? draw_weights(w, mode, t[q], d[q], a.inv_t) : f32x4{0.f, 0.f, 0.f, 0.f};
        ls += (v[q].x + v[q].y) + (v[q].z + v[q].w);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v[q][e] > 0.f) last = i0 + 4 * q + e;
      }
      float x = ls;   // inclusive prefix over the lanes, then over the waves, in order
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const float y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
      }
      if (lane == 63) s_wave[wave] = x;
      __syncthreads();
      float base = run;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (q < wave) base += s_wave[q];
        run += s_wave[q];
      }
      if (last >= 0) atomicMax(&s_last, last);
      // the lowest thread past the goal (ids ascend with the thread)
      const unsigned long long hit = __ballot(ls > 0.f && base + x > goal);
      if (hit && lane == __ffsll((long long)hit) - 1) {
        float at = base + x - ls;
        int id = -1;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (id < 0 && v[q][e] > 0.f && at + v[q][e] > goal) id = i0 + 4 * q + e;
            at += v[q][e];
          }
        atomicMin((unsigned *)&s_found, (unsigned)(id >= 0 ? id : last));   // -1: the largest unsigned
      }
      __syncthreads();
    }
  }
  if (tid == 0) {
    a.n_acc[b] = w.n;
    a.next[b] = s_pick < 0 ? -1 : s_found >= 0 ? s_found : s_last;
  }
}

// Greedy: one wave per sequence, lane i takes row i's arg-max; the first
// draft that is not its row's choice is one ballot.
__global__ __launch_bounds__(64) void k_verify_greedy(VerifyChainArgs a) {
  const int b = blockIdx.x, lane = threadIdx.x, K = a.K;   // K <= 63
  const int arg = lane <= K ? merge_best(a.best + ((size_t)b * (K + 1) + lane) * a.parts, a.parts) : -1;
  int x = -1;
  if (lane < K) {
    x = a.drafts[(size_t)b * K + lane];
    if (x < 0 || x >= a.V) {
      atomicOr(a.err, ERRF_TOKEN);
      x = -1;
    }
  }
  const int n = __ffsll((long long)__ballot(lane >= K || x < 0 || x != arg)) - 1;
  const int next = __shfl(arg, n, 64);
  if (lane == 0) {
    a.n_acc[b] = n;
    a.next[b] = next;
  }
}

struct VerifyTreeArgs {
  int nodes, V, parts;
  const BestStat *ts;            // [B*(nodes+1)][parts]
  const int32_t *tokens, *parent;   // [B, nodes]
  int32_t *n_acc, *path, *next;  // [B], [B, nodes], [B]
};

// one wave per tree; lane j holds node j (v <= 64), so each step of the walk
// is one ballot over the nodes: the first child of the current position
// whose token is the target's choice there
__global__ __launch_bounds__(64) void k_verify_tree(VerifyTreeArgs a) {
  __shared__ int s_arg[MAX_VERIFY_NODES + 1];
  const int b = blockIdx.x, lane = threadIdx.x, v = a.nodes;
  for (int j = lane; j <= v; j += 64) s_arg[j] = merge_best(a.ts + ((size_t)b * (v + 1) + j) * a.parts, a.parts);
  const int tok = lane < v ? a.tokens[(size_t)b * v + lane] : -1;
  const int par = lane < v ? a.parent[(size_t)b * v + lane] : -2;
  __syncthreads();
  int at = -1, n = 0;
  int32_t *path = a.path + (size_t)b * v;
  while (n < v) {   // a path has at most v nodes (also bounds a malformed parent table)
    const int want = s_arg[at + 1];
    const unsigned long long m = __ballot(lane < v && par == at && tok == want);
    if (!m) break;
    at = __ffsll((long long)m) - 1;
    if (lane == 0) path[n] = at;
    ++n;
  }
  for (int j = n + lane; j < v; j += 64) path[j] = -1;
  if (lane == 0) {
    a.n_acc[b] = n;
    a.next[b] = s_arg[at + 1];
  }
}

// Bytes of the statistics of a call over `rows` rows, and its draws: 8 per
// (row, slice), where few rows take more slices (row_slices), and a Draw per
// sequence of at least 3 rows (sampled, K >= 1).
static_assert(sizeof(Draw) <= 3 * VSPLIT * sizeof(SoftStat), "draws fit beside the statistics");
size_t verify_stats_bytes(int rows) {
  const size_t entries = (size_t)rows * VSPLIT;
  return 2 * sizeof(SoftStat) * (entries > VSPLIT_WGS ? entries : VSPLIT_WGS);
}

// ---------------------------------------------------------------------------
// Chain verification that allocates nothing, for callers that cannot call
// hipMalloc (graph capture, serving loops): the per-slice row statistics and
// the kernels' error word live in this file-scope device array, one copy per
// GPU, held until the process ends.  Its device address comes from
// hipGetSymbolAddress, once per device (in prism_create, or at the first
// call on a device); host code never passes the array's own name.
constexpr int VSTATIC_ROWS = 8192;   // logits rows statistics are kept for
constexpr size_t VSTATIC_BYTES = 256 + (size_t)VSTATIC_ROWS * VSPLIT * 2 * sizeof(SoftStat);
static __device__ __align__(256) unsigned char scratch[VSTATIC_BYTES];

namespace {
constexpr int SCRATCH_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[SCRATCH_DEVICES] = {};

prism_status static_fail(prism_status st, const char *fmt, ...) {
  char buf[256];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  set_global_error(buf);
  return st;
}
}  // namespace

hipError_t verify_scratch(void **out) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= SCRATCH_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace prism

extern "C" prism_status prism_verify_chain_static(int32_t vocab, int32_t batch, int32_t K,
                                                  float temperature, const float *d_target_logits,
                                                  const float *d_draft_logits,
                                                  const int32_t *d_draft_tokens,
                                                  const float *d_uniforms, int32_t *d_n_accepted,
                                                  int32_t *d_next_token, void *stream) {
  using namespace prism;
  if (vocab < 16 || vocab % 16)
    return static_fail(PRISM_ERR_SHAPE, "vocab %d must be a positive multiple of 16", vocab);
  if (batch < 1 || K < 1 || K >= VER_MAXK)
    return static_fail(PRISM_ERR_INVALID_ARG, "batch %d / K %d out of range (K < %d)", batch,
                       K, VER_MAXK);
  if (!(temperature >= 0.f) || (temperature > 0.f && !std::isfinite(1.f / temperature)))
    return static_fail(PRISM_ERR_INVALID_ARG, "temperature %g", (double)temperature);
  const bool sampled = temperature > 0.f;
  if (!d_target_logits || !d_draft_tokens || !d_n_accepted || !d_next_token ||
      (sampled && (!d_draft_logits || !d_uniforms)))
    return static_fail(PRISM_ERR_INVALID_ARG, "NULL pointer");
  const long rows = (long)batch * (K + 1) + (sampled ? (long)batch * K : 0);
  if (rows > VSTATIC_ROWS)
    return static_fail(PRISM_ERR_SHAPE,
                       "%ld logits rows exceed the %d the static scratch holds "
                       "(batch * (K + 1), plus batch * K when sampled)",
                       rows, VSTATIC_ROWS);
  void *base = nullptr;
  hipError_t e = verify_scratch(&base);
  if (e != hipSuccess)
    return static_fail(PRISM_ERR_HIP, "hipGetSymbolAddress: %s", hipGetErrorString(e));
  uint32_t *err = (uint32_t *)base;                    // written by the kernels, never read
  void *stats = (unsigned char *)base + 256;
  launch_verify_chain(batch, K, vocab, sampled ? 1.f / temperature : 0.f, d_target_logits,
                      d_draft_logits, d_draft_tokens, d_uniforms, d_n_accepted, d_next_token,
                      stats, err, (hipStream_t)stream);
  e = hipGetLastError();
  if (e != hipSuccess) return static_fail(PRISM_ERR_HIP, "launch: %s", hipGetErrorString(e));
  return PRISM_OK;
}

namespace prism {

void launch_verify_chain(int B, int K, int V, float inv_t, const float *tl, const float *dl,
                         const int32_t *drafts, const float *u, int32_t *n_acc, int32_t *next,
                         void *stats, uint32_t *err, hipStream_t s) {
  VerifyChainArgs a{};
  a.K = K; a.V = V; a.inv_t = inv_t;
  a.tl = tl; a.dl = dl; a.drafts = drafts; a.u = u;
  a.n_acc = n_acc; a.next = next; a.err = err;
  const int rt = B * (K + 1), rd = B * K;
  if (inv_t > 0.f) {   // sampled: the target and draft rows' softmax statistics
    a.parts = row_slices(rt + rd);
    SoftStat *st = (SoftStat *)stats;
    a.ts = st;
    a.ds = st + (size_t)rt * a.parts;
    const size_t entries = (size_t)(rt + rd) * a.parts;
    a.draw = (Draw *)(st + entries);
    hipLaunchKernelGGL(k_rows_soft, dim3(a.parts, rt + rd), dim3(256), 0, s, tl, rt, dl, V, inv_t, st);
    hipLaunchKernelGGL(k_verify_decide, dim3(DRAW_SLICES, B), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_verify_draw, dim3(B), dim3(256), 0, s, a);
  } else {             // greedy: the target rows' arg-max only
    a.parts = row_slices(rt);
    a.best = (const BestStat *)stats;
    hipLaunchKernelGGL(k_rows_best, dim3(a.parts, rt), dim3(256), 0, s, tl, V, (BestStat *)stats);
    hipLaunchKernelGGL(k_verify_greedy, dim3(B), dim3(64), 0, s, a);
  }
}

void launch_verify_tree(int B, int nodes, int V, const float *tl, const int32_t *tokens,
                        const int32_t *parent, int32_t *n_acc, int32_t *path, int32_t *next,
                        void *stats, hipStream_t s) {
  const int rows = B * (nodes + 1), parts = row_slices(rows);
  BestStat *ts = (BestStat *)stats;
  hipLaunchKernelGGL(k_rows_best, dim3(parts, rows), dim3(256), 0, s, tl, V, ts);
  VerifyTreeArgs a{nodes, V, parts, ts, tokens, parent, n_acc, path, next};
  hipLaunchKernelGGL(k_verify_tree, dim3(B), dim3(64), 0, s, a);
}

}  // namespace prism
