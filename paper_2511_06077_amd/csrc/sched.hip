// Varlen scheduler: device offsets -> attention work units.
//
// The ragged batch is packed without padding and segmented by per-request
// offsets (App. A.4, index-based ragged target attention).  Each request's
// history rows are covered by whole 32-row blocks of the packed history
// ([floor(h0/32), ceil(h1/32))); the blocks are cut into at most max_chunks
// chunks of about `chunk_blocks` blocks, and the request's targets into groups
// of `group` (at most kWideGroup).  One unit = (target group, chunk).  Units of groups with at
// most 32 targets are listed first, the wider ones after them, so kernels
// specialised on the group width each get one contiguous range.  With
// deal = G > 0, each range holds its units in descending order of history
// blocks (32 size buckets, any order inside a bucket), every complete round
// of G units after the first in reverse order: a persistent kernel of G
// workgroups that deals units round-robin (unit w, w + G, ...) then pairs
// large units with small ones.  Every
// target's chunk count is recorded so the combine step knows how many partial
// results to merge.
//
// With `order`, entry u is unit u's rank in request, group and chunk order (the
// chunks of one target group have consecutive ranks).
//
// One workgroup of 1024 threads.  Up to 1024 requests: a thread per request
// counts its units, then the threads share the units (each finds its request
// by a binary search over the counts' prefix sums) and the targets' chunk
// counts.  One thread writing all its request's units and targets took 14 us
// for one request of 16 chunks and 40 targets, 27 us for 16 requests of 256
// targets.  More requests: each thread owns a contiguous run of them.
// Invalid segments produce no units and set the workspace status, so no later
// kernel reads outside the buffers whatever the offsets hold.  Only requests
// with m_lo..m_hi targets get units (a batch can be split between two forms
// of the attention, each with its own schedule); every request is validated.
//
// The per-call weight repacking lives here too: a forward's schedules (one
// workgroup each) and its repacking run as one launch, side by side.
#include <algorithm>

#include "common.h"
#include "fast.h"
#include "internal.h"

namespace stca {

namespace {

constexpr int kSchedThreads = 1024;

struct ReqPlan {
  int32_t h0, h1, t0, t1, nch, cb, ng, bl;
  bool ok;
};

__device__ ReqPlan plan_request(const int32_t* hoff, const int32_t* toff, int r, int64_t n_hist,
                                int64_t n_tgt, int chunk_blocks, int group, int m_lo, int m_hi, int max_chunks) {
  ReqPlan p{};
  p.h0 = hoff[r];
  p.h1 = hoff[r + 1];
  p.t0 = toff[r];
  p.t1 = toff[r + 1];
  p.ok = p.h0 >= 0 && p.h0 <= p.h1 && p.h1 <= n_hist && p.t0 >= 0 && p.t0 <= p.t1 && p.t1 <= n_tgt &&
         (p.t1 == p.t0 || p.h1 > p.h0);
  p.nch = 0;
  p.ng = 0;
  if (!p.ok || p.t1 == p.t0 || p.t1 - p.t0 < m_lo || p.t1 - p.t0 > m_hi) return p;
  p.bl = p.h0 / kBlockTokens;
  const int32_t bh = static_cast<int32_t>(ceil_div(p.h1, kBlockTokens));
  const int32_t nb = bh - p.bl;
  int32_t nch = static_cast<int32_t>(ceil_div(nb, chunk_blocks));
  nch = nch < 1 ? 1 : (nch > max_chunks ? max_chunks : nch);
  p.cb = static_cast<int32_t>(ceil_div(nb, nch));
  p.nch = static_cast<int32_t>(ceil_div(nb, p.cb));  // no empty chunk
  p.ng = static_cast<int32_t>(ceil_div(p.t1 - p.t0, group));
  return p;
}

__device__ __forceinline__ int group_size(const ReqPlan& p, int g, int group) {
  return min(group, p.t1 - (p.t0 + g * group));
}

// Exclusive prefix sum over the workgroup: an inclusive scan inside each
// wave by shuffles, then one scan of the 16 wave totals by the first wave.
// scan[kSchedThreads - 1] holds the total afterwards.
__device__ int64_t block_scan(int64_t* scan, int64_t mine) {
  constexpr int kWaves = kSchedThreads / 64;
  __shared__ int64_t wsum[kWaves];
  const int tid = threadIdx.x, lane = tid % 64, w = tid / 64;
  int64_t v = mine;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int64_t t = __shfl_up(v, off, 64);
    if (lane >= off) v += t;
  }
  if (lane == 63) wsum[w] = v;
  __syncthreads();
  if (w == 0) {
    int64_t x = lane < kWaves ? wsum[lane] : 0;
#pragma unroll
    for (int off = 1; off < kWaves; off <<= 1) {
      const int64_t t = __shfl_up(x, off, 64);
      if (lane >= off) x += t;
    }
    if (lane < kWaves) wsum[lane] = x;  // inclusive prefix of the wave totals
  }
  __syncthreads();
  const int64_t excl = (w > 0 ? wsum[w - 1] : 0) + v - mine;
  if (tid == kSchedThreads - 1) scan[tid] = wsum[kWaves - 1];
  __syncthreads();
  return excl;
}

// Size buckets of the by-size order: bucket of a unit of `size` blocks.
constexpr int kSizeBuckets = 32;
__device__ __forceinline__ int size_bucket(int size, int chunk_blocks) {
  return min(kSizeBuckets - 1, static_cast<int>((int64_t)size * kSizeBuckets / (chunk_blocks + 1)));
}

// One schedule: launch_sched's arguments.
struct SchedJob {
  const int32_t *hoff, *toff;
  int R;
  int64_t n_hist, n_tgt;
  int chunk_blocks, group, m_lo, m_hi, max_chunks, by_size;
  unsigned deal;
  Unit* units;
  int64_t max_units;
  int32_t* tchunks;
  WsHeader* hdr;
  int32_t* order;
};

struct SchedLds {
  int64_t scan[kSchedThreads];
  int bad;
  unsigned cursor[2][kSizeBuckets];  // by_size: units, then next rank, per (class, bucket)
  // up to kSchedThreads requests: first unit of each request within its class
  // (then the total), first target, chunk count
  int32_t pn[kSchedThreads + 1], pw[kSchedThreads + 1], toff[kSchedThreads], nch[kSchedThreads];
};

__device__ void sched_body(const SchedJob& S, SchedLds& L) {
  const int tid = threadIdx.x;
  const int R = S.R, group = S.group;
  const int64_t n_tgt = S.n_tgt;
  const bool few = R <= kSchedThreads;
  if (tid == 0)
    L.bad = (S.hoff[0] != 0 || S.toff[0] != 0 || S.hoff[R] != S.n_hist || S.toff[R] != n_tgt) ? 1 : 0;
  if (tid < 2 * kSizeBuckets) L.cursor[tid / kSizeBuckets][tid % kSizeBuckets] = 0;
  if (!few)
    for (int64_t t = tid; t < n_tgt; t += kSchedThreads) S.tchunks[t] = 0;
  __syncthreads();

  auto plan = [&](int r) {
    return plan_request(S.hoff, S.toff, r, S.n_hist, n_tgt, S.chunk_blocks, group, S.m_lo, S.m_hi, S.max_chunks);
  };
  const int per = static_cast<int>(ceil_div(R, kSchedThreads));
  const int rb = tid * per;
  const int re = min(R, rb + per);
  int64_t narrow = 0, wide = 0;
  bool any_bad = false;
  for (int r = rb; r < re; ++r) {
    const ReqPlan p = plan(r);
    any_bad |= !p.ok;
    if (p.ng > 0) {
      // every group but the last is full
      const int last_wide = group_size(p, p.ng - 1, group) > 32 ? 1 : 0;
      const int64_t w = (int64_t)(group > 32 ? p.ng - 1 : 0) + last_wide;
      wide += w * p.nch;
      narrow += (p.ng - w) * p.nch;
    }
    if (few) {
      L.toff[r] = p.t0;
      L.nch[r] = p.nch;
    } else if (S.by_size) {  // units per (class, size bucket)
      const int32_t bh = static_cast<int32_t>(ceil_div(p.h1, kBlockTokens));
      for (int g = 0; g < p.ng; ++g)
        for (int c = 0; c < p.nch; ++c) {
          const int b0 = p.bl + c * p.cb;
          atomicAdd(&L.cursor[group_size(p, g, group) > 32][size_bucket(min(b0 + p.cb, bh) - b0, S.chunk_blocks)], 1u);
        }
    }
  }
  if (any_bad) atomicOr(&L.bad, 1);
  int64_t un = block_scan(L.scan, narrow);
  const int64_t total_narrow = L.scan[kSchedThreads - 1];
  __syncthreads();
  const int64_t uwc = block_scan(L.scan, wide);
  const int64_t total = total_narrow + L.scan[kSchedThreads - 1];
  int64_t uw = total_narrow + uwc;
  // (units that all go out in the first round need no order; `order` asks for it)
  const bool by_size = S.by_size && (S.order || !few || total > S.deal);

  // the place of the unit of rank ur: with by_size, rank k in the class's
  // descending order; complete rounds of `deal` units are dealt in alternating
  // directions, so that a workgroup taking a large unit in one round takes a
  // small one in the next
  auto place = [&](int cls, int size, int64_t ur) -> int64_t {
    if (!by_size) return ur;
    const unsigned k = atomicAdd(&L.cursor[cls][size_bucket(size, S.chunk_blocks)], 1u);
    const unsigned nc = static_cast<unsigned>(cls ? total - total_narrow : total_narrow);
    const unsigned j = k / S.deal, i = k - j * S.deal;
    const bool back = (j & 1) && (j + 1) * S.deal <= nc;
    return (cls ? total_narrow : 0) + static_cast<int64_t>(j) * S.deal + (back ? S.deal - 1 - i : i);
  };
  auto emit = [&](const ReqPlan& p, int r, int g, int c, int64_t ur) {
    const int32_t bh = static_cast<int32_t>(ceil_div(p.h1, kBlockTokens));
    Unit v;
    v.r = r;
    v.t0 = p.t0 + g * group;
    v.nt = group_size(p, g, group);
    v.c = c;
    v.b0 = p.bl + c * p.cb;
    v.b1 = min(v.b0 + p.cb, bh);
    v.l0 = p.h0;
    v.l1 = p.h1;
    const int64_t u = place(v.nt > 32 ? 1 : 0, v.b1 - v.b0, ur);
    if (u >= S.max_units) return;
    S.units[u] = v;
    if (S.order) S.order[u] = static_cast<int32_t>(ur);
  };
  // each bucket's rank range within its class, from the largest bucket down
  auto bucket_ranks = [&]() {
    if (tid < 2) {
      unsigned pos = 0u;
      for (int k = kSizeBuckets - 1; k >= 0; --k) {
        const unsigned n = L.cursor[tid][k];
        L.cursor[tid][k] = pos;
        pos += n;
      }
    }
    __syncthreads();
  };
  // last entry of the non-decreasing a[0..R) that is <= k (a[0] <= k)
  auto find = [&](const int32_t* a, int32_t k) {
    int lo = 0, hi = R;
    while (hi - lo > 1) {
      const int mid = (lo + hi) / 2;
      if (a[mid] <= k) lo = mid;
      else hi = mid;
    }
    return lo;
  };
  if (few) {
    if (tid < R) {
      L.pn[tid] = static_cast<int32_t>(un);
      L.pw[tid] = static_cast<int32_t>(uwc);
    }
    __syncthreads();
    const bool bad = L.bad != 0;
    // (request, group, chunk) of the unit of rank i
    auto locate = [&](int64_t i, int& r, int& g, int& c) {
      const bool cls = i >= total_narrow;
      const int32_t k = static_cast<int32_t>(cls ? i - total_narrow : i);
      r = find(cls ? L.pw : L.pn, k);
      const ReqPlan p = plan(r);
      const int32_t local = k - (cls ? L.pw : L.pn)[r];
      // groups wider than 32: only the last of a request may be narrow
      const bool last = group > 32 && !cls;
      g = last ? p.ng - 1 : local / max(p.nch, 1);
      c = last ? local : local % max(p.nch, 1);
      return p;
    };
    if (by_size) {
      for (int64_t i = tid; i < total; i += kSchedThreads) {
        int r, g, c;
        const ReqPlan p = locate(i, r, g, c);
        const int32_t bh = static_cast<int32_t>(ceil_div(p.h1, kBlockTokens));
        const int b0 = p.bl + c * p.cb;
        atomicAdd(&L.cursor[i >= total_narrow][size_bucket(min(b0 + p.cb, bh) - b0, S.chunk_blocks)], 1u);
      }
      __syncthreads();
      bucket_ranks();
    }
    for (int64_t i = tid; i < total; i += kSchedThreads) {
      int r, g, c;
      const ReqPlan p = locate(i, r, g, c);
      emit(p, r, g, c, i);
    }
    if (!bad) {
      for (int64_t t = tid; t < n_tgt; t += kSchedThreads)
        S.tchunks[t] = L.nch[find(L.toff, static_cast<int32_t>(t))];
    } else {  // offsets that may not ascend: request by request
      for (int64_t t = tid; t < n_tgt; t += kSchedThreads) S.tchunks[t] = 0;
      __syncthreads();
      if (tid < R) {
        const ReqPlan p = plan(tid);
        if (p.nch > 0)
          for (int t = p.t0; t < p.t1; ++t) S.tchunks[t] = p.nch;
      }
    }
  } else {
    if (by_size) bucket_ranks();
    for (int r = rb; r < re; ++r) {
      const ReqPlan p = plan(r);
      if (p.nch == 0) continue;
      for (int g = 0; g < p.ng; ++g) {
        int64_t& ur = group_size(p, g, group) > 32 ? uw : un;
        for (int c = 0; c < p.nch; ++c, ++ur) emit(p, r, g, c, ur);
      }
      for (int t = p.t0; t < p.t1; ++t) S.tchunks[t] = p.nch;
    }
  }
  if (tid == 0) {
    S.hdr->n_units = static_cast<int32_t>(total < S.max_units ? total : S.max_units);
    S.hdr->n_narrow = static_cast<int32_t>(total_narrow < S.max_units ? total_narrow : S.max_units);
    S.hdr->status = (L.bad || total > S.max_units) ? STCA_ERR_INVALID_ARG : STCA_OK;
    S.hdr->range = 0;  // set by later kernels of the call that find an fp16 overflow
  }
}

__global__ __launch_bounds__(kSchedThreads) void sched_kernel(SchedJob S) {
  __shared__ SchedLds L;
  sched_body(S, L);
}

// ------------------------------------------------------------- repacking
template <typename V8>
struct elem_of;
template <>
struct elem_of<bf16x8> {
  typedef __bf16 type;
};
template <>
struct elem_of<f16x8> {
  typedef _Float16 type;
};

// W: [K][N] bf16 row-major -> P: [N/32][K/16][64][8], kept bf16 (V8 = bf16x8)
// or converted to fp16 (V8 = f16x8, exact for every bf16 value inside fp16's
// range); vector g of it.
template <typename V8>
__device__ __forceinline__ void pack_one(const bf16_bits* __restrict__ w, V8* __restrict__ P, int K, int N,
                                         int64_t g, bool trans) {
  const int lane = g % 64;
  const int64_t rest = g / 64;
  const int ks = rest % (K / 16);
  const int nb = rest / (K / 16);
  const int n = nb * 32 + lane % 32;
  const int k0 = ks * 16 + 8 * (lane / 32);
  V8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e)
    r[e] = static_cast<typename elem_of<V8>::type>(
        to_f32(w[trans ? (int64_t)n * K + k0 + e : (int64_t)(k0 + e) * N + n]));
  P[g] = r;
}

__device__ __forceinline__ int64_t pack_groups(const PackJob& b) { return (int64_t)(b.N / 32) * (b.K / 16) * 64; }

__device__ __forceinline__ void pack_layer(const PackJob& b, int layer, int64_t g) {
  const int64_t groups = pack_groups(b);
  const bf16_bits* w = static_cast<const bf16_bits*>(b.src) + (int64_t)layer * b.K * b.N;
  if (b.to_f16)
    pack_one(w, static_cast<f16x8*>(b.dst) + (int64_t)layer * groups, b.K, b.N, g, b.trans != 0);
  else
    pack_one(w, static_cast<bf16x8*>(b.dst) + (int64_t)layer * groups, b.K, b.N, g, b.trans != 0);
}

// Several weights in one launch (blockIdx.z = job).
__global__ void pack_many_kernel(PackJobs J) {
  const PackJob& b = J.job[blockIdx.z];
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < pack_groups(b)) pack_layer(b, blockIdx.y, g);
}

// A call's schedules (workgroups 0 .. n_sched - 1) and its repacking (the
// rest: kSchedThreads vectors each of one job and layer) in one launch: they
// are independent, and each alone leaves the chip nearly idle (one request:
// 14 + 7 us as two launches, the schedule's 10 together).
struct SetupArgs {
  SchedJob sched[kMaxSetupScheds];
  int n_sched, n_jobs, n_layers;
  PackJobs pack;
  int32_t* zero;  // n_zero words to clear (arrival counters of the call's later launches)
  int64_t n_zero;
};
__global__ __launch_bounds__(kSchedThreads) void setup_kernel(SetupArgs A) {
  __shared__ SchedLds L;
  const int bid = blockIdx.x;
  for (int64_t i = (int64_t)bid * kSchedThreads + threadIdx.x; i < A.n_zero; i += (int64_t)gridDim.x * kSchedThreads)
    A.zero[i] = 0;
  if (bid < A.n_sched) {
    sched_body(A.sched[bid], L);
    return;
  }
  int64_t i = bid - A.n_sched;
  for (int j = 0; j < A.n_jobs; ++j) {
    const PackJob& b = A.pack.job[j];
    const int64_t per = ceil_div(pack_groups(b), kSchedThreads), n = per * A.n_layers;
    if (i < n) {
      const int64_t g = i % per * kSchedThreads + threadIdx.x;
      if (g < pack_groups(b)) pack_layer(b, static_cast<int>(i / per), g);
      return;
    }
    i -= n;
  }
}

bool make_job(const SchedSpec& s, SchedJob* j) {
  if (s.group < 1 || s.group > kWideGroup || s.deal < 0) return false;
  *j = {s.hoff, s.toff, s.R, s.n_hist, s.n_tgt, s.chunk_blocks, s.group, s.m_lo, s.m_hi, s.max_chunks,
        s.deal > 0 ? 1 : 0,
        static_cast<unsigned>(s.deal > 0 ? s.deal : 1), s.units, s.max_units, s.tchunks, s.hdr, s.order};
  return true;
}

}  // namespace

hipError_t launch_sched(const SchedSpec& s, hipStream_t st) {
  SchedJob j;
  if (!make_job(s, &j)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(sched_kernel, dim3(1), dim3(kSchedThreads), 0, st, j);
  return hipGetLastError();
}

hipError_t launch_setup(const SchedSpec* sched, int n_sched, const PackJobs& jobs, int n_jobs, int n_layers,
                        hipStream_t st, int32_t* zero, int64_t n_zero) {
  if (n_sched < 0 || n_sched > kMaxSetupScheds || n_jobs < 0 || n_jobs > kMaxPackJobs) return hipErrorInvalidValue;
  SetupArgs A{};
  for (int i = 0; i < n_sched; ++i)
    if (!make_job(sched[i], &A.sched[i])) return hipErrorInvalidValue;
  A.n_sched = n_sched;
  A.n_jobs = n_jobs;
  A.n_layers = n_layers;
  A.pack = jobs;
  A.zero = zero;
  A.n_zero = zero ? n_zero : 0;
  int64_t blocks = n_sched;
  for (int j = 0; j < n_jobs; ++j)
    blocks += n_layers * ceil_div((int64_t)(jobs.job[j].N / 32) * (jobs.job[j].K / 16) * 64, kSchedThreads);
  hipLaunchKernelGGL(setup_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kSchedThreads), 0, st, A);
  return hipGetLastError();
}

hipError_t fast_pack_many(const PackJobs& jobs, int n_jobs, int n_layers, hipStream_t st) {
  if (n_jobs < 1 || n_jobs > kMaxPackJobs) return hipErrorInvalidValue;
  int64_t groups = 0;
  for (int j = 0; j < n_jobs; ++j)
    groups = std::max<int64_t>(groups, (int64_t)(jobs.job[j].N / 32) * (jobs.job[j].K / 16) * 64);
  dim3 g(static_cast<unsigned>(ceil_div(groups, 256)), n_layers, n_jobs);
  hipLaunchKernelGGL(pack_many_kernel, g, dim3(256), 0, st, jobs);
  return hipGetLastError();
}

// Host mirror of plan_request for exact unit counts when host offsets exist.
int64_t host_count_units(const int32_t* hoff, const int32_t* toff, int R, int chunk_blocks, int group, int m_lo,
                         int m_hi, int max_chunks, int64_t* wide) {
  int64_t n = 0, nw = 0;
  for (int r = 0; r < R; ++r) {
    const int64_t h0 = hoff[r], h1 = hoff[r + 1], m = toff[r + 1] - static_cast<int64_t>(toff[r]);
    if (m == 0 || m < m_lo || m > m_hi) continue;
    const int64_t nb = ceil_div(h1, kBlockTokens) - h0 / kBlockTokens;
    int64_t nch = ceil_div(nb, chunk_blocks);
    nch = nch < 1 ? 1 : (nch > max_chunks ? max_chunks : nch);
    nch = ceil_div(nb, ceil_div(nb, nch));
    const int64_t ng = ceil_div(m, group);
    n += nch * ng;
    // every group but the last is full
    if (group > 32) nw += nch * (ng - 1 + (m - (ng - 1) * group > 32 ? 1 : 0));
  }
  if (wide) *wide = nw;
  return n;
}

}  // namespace stca
