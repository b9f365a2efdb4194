// graph.hip -- set-up and per-iteration bookkeeping kernels around the sweep:
// validation, degree classes, initial labels and flags (Algorithm 1: every
// vertex in its own community and unprocessed), the frontier of flagged
// vertices ("for all unprocessed i ... mark i processed"), the hub slice plan,
// the publishing of labels and changes, and fp64 modularity (Eq. 1).
#include <algorithm>
#include <mutex>

#include "lpa_device.h"
#include "lpa_mlp.h"
#include "lpa_record.h"

namespace lpa {

namespace {

constexpr int kBT = 256;

__device__ __forceinline__ void set_error(DevStats* st, unsigned int bit) {
  atomicOr(&st->error, bit);
}

template <typename T>
__global__ void k_fill(T* p, T v, int64_t count) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

int grid_for(int64_t n, int per_block, int cap) {
  const int64_t g = (n + per_block - 1) / per_block;
  return (int)(g < 1 ? 1 : (g > cap ? cap : g));
}

}  // namespace

// ---- init ---------------------------------------------------------------------
__global__ void k_init(int64_t n, const int32_t* init, const int32_t* inv, int32_t* C,
                       uint8_t* F, DevStats* st) {
  // ident: every label equals its internal id, so the first sweep may take
  // a neighbour's id for its label
  if (blockIdx.x == 0 && threadIdx.x == 0) st->ident = (init || inv) ? 0 : 1;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t u = inv ? (int64_t)inv[i] : i;
    const int32_t c = init ? init[u] : (int32_t)u;
    if (c < 0 || (int64_t)c >= n) set_error(st, 4u);
    C[i] = c;
    F[i] = 1;
  }
}

hipError_t launch_init(int64_t n, const int32_t* init, const int32_t* inv, int32_t* C,
                       uint8_t* F, DevStats* st, hipStream_t s) {
  hipLaunchKernelGGL(k_init, dim3(grid_for(n, kBT, 8192)), dim3(kBT), 0, s, n, init, inv, C, F,
                     st);
  return hipGetLastError();
}

// ---- run control ---------------------------------------------------------------
// k_run_begin zeroes the counters and stores the run's parameters; every
// per-iteration kernel returns at once when stop is set; k_iter_end records
// the iteration's statistics and applies the stop rule of Algorithm 1 (after
// an iteration that is not Pick-Less with changed < tolerance * N), or, in a
// batched run, stops when every graph has stopped.
__global__ void k_run_begin(DevStats* st, double tol, int cap, int rho, int batched,
                            int graphs, LearnParams lp, unsigned int seq) {
  // the counters and their copies; the history stays that of the last run
  // (lpa_learned_history) until an iteration of this one ends
  uint32_t* w = reinterpret_cast<uint32_t*>(st);
  for (uint32_t i = threadIdx.x; i < sizeof(DevStats) / sizeof(uint32_t); i += blockDim.x)
    w[i] = 0u;
  uint32_t* c = reinterpret_cast<uint32_t*>(reinterpret_cast<DevState*>(st)->slot);
  for (uint32_t i = threadIdx.x; i < sizeof(DevState::slot) / sizeof(uint32_t); i += blockDim.x)
    c[i] = 0u;
  __syncthreads();
  if (threadIdx.x == 0) {
    st->tol = tol;
    st->cap = cap;
    st->rho = rho;
    st->iter = 0;
    st->stop = cap <= 0 ? 1 : 0;
    st->batched = batched;
    st->graphs_left = (unsigned int)graphs;
    st->learn = lp.learn;
    st->pred_cmin = lp.cmin < 1 ? 1 : lp.cmin;
    st->pred_cmax = lp.cmax < 1 || lp.cmax >= kClassHub ? kClassHub - 1 : lp.cmax;
    st->pred_start = lp.pstart < 1 ? 1 : lp.pstart;
    st->guard = lp.guard;
    st->trace = lp.trace;
    st->z_theta = lp.z_theta;
    st->fn_bound = lp.fn_bound;
    st->trace_rate = lp.trace_rate;
    st->trace_seed = lp.trace_seed;
    st->trace_cap = lp.trace_cap;
    st->cand = 1;
    st->seq = seq;
  }
  begin_iteration(st);  // thread 0 wrote what it reads
}

hipError_t launch_run_begin(DevStats* st, double tol, int cap, int rho, int batched,
                            int graphs, const LearnParams& lp, unsigned int seq,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_run_begin, dim3(1), dim3(1024), 0, s, st, tol, cap, rho, batched, graphs,
                     lp, seq);
  return hipGetLastError();
}

__global__ void k_arm_flags(uint8_t* F, int64_t n, const DevStats* st) {
  if (st->stop) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    F[i] = 1;
}

hipError_t launch_arm_flags(uint8_t* F, int64_t n, const DevStats* st, hipStream_t s) {
  hipLaunchKernelGGL(k_arm_flags, dim3(grid_for(n, kBT, 8192)), dim3(kBT), 0, s, F, n, st);
  return hipGetLastError();
}

// How this iteration's flags are set: 0 pushed, 1 pulled, 2 left to
// lpa_get_flags (the run stops after this iteration: k_iter_end's test, same
// operands).  fw: entries in the rows of the changed vertices.
__device__ __forceinline__ unsigned int flag_decision(const DevStats* st, const FlagRule& r,
                                                      unsigned long long fw,
                                                      unsigned long long changed,
                                                      unsigned long long skipped) {
  if (!st->batched &&
      ((!st->pl && (double)(changed + skipped) < st->tol * (double)r.n) || st->iter + 1 >= st->cap))
    return 2u;
  if (r.force) return r.force == 2 ? 1u : 0u;
  return (unsigned long long)r.pdiv * fw >= (unsigned long long)r.m ? 1u : 0u;
}

// FOLD: no k_flag_decide has added up the counters' copies (a work-queue run,
// k_flags); otherwise only the pull kernels have added to them since.  rule.m
// >= 0: record k_flags' decision too.  next: no k_hub_plan begins the next
// iteration.
template <bool FOLD>
__global__ __launch_bounds__(1024) void k_iter_end(DevStats* st, DevIterStats* hist, int64_t n,
                                                   unsigned long long* progress, FlagRule rule,
                                                   int next) {
  if (st->stop) return;
  if constexpr (FOLD) {
    fold_stats(st);
  } else if (threadIdx.x < kStatSlots) {
    unsigned long long* p =
        &reinterpret_cast<DevState*>(st)->slot[threadIdx.x][kStatPullScanned];
    unsigned long long t = *p;
    *p = 0ull;
    for (int ofs = kStatSlots / 2; ofs > 0; ofs >>= 1) t += __shfl_xor(t, ofs, kStatSlots);
    if (threadIdx.x == 0) st->pull_scanned = t;
  }
  __shared__ int ended_sh;
  if (threadIdx.x == 0) {
    unsigned long long changed = 0, edges = 0;
    for (int c = 0; c < kNumClasses; ++c) {
      changed += st->changed[c];
      edges += st->edges[c];
    }
    if (rule.m >= 0) {
      unsigned long long fw = 0;
      for (int c = 0; c < kNumClasses; ++c) fw += st->flagw[c];
      st->pull_mode = flag_decision(st, rule, fw, changed, st->skipped);
      st->flags_deferred = st->pull_mode == 2u ? 1u : 0u;
    }
    changed -= st->reverted;  // Cross-Check reverts do not count as changes
    const int l = st->iter;
    // learned skipping: a plain iteration with predictions checks the vertices
    // predicted unchanged; too many of them changing turns skipping off
    if (st->predict && !st->skipping && st->npred > 0 &&
        (double)st->fneg > st->fn_bound * (double)st->npred)
      st->fallback = 1;
    DevIterStats& h = hist[l];
    h.iteration = l;
    h.pick_less = st->pl;
    h.changed = (long long)changed;
    h.processed = (long long)st->processed;
    h.edges = (long long)edges;
    h.skipped = (long long)st->skipped;
    h.npred = (long long)st->npred;
    h.fneg = st->skipping ? 0ll : (long long)st->fneg;
    h.skipping = st->skipping;
    h.fallback = st->fallback;
    int stop = 0;
    if (st->batched) stop = st->graphs_left == 0u;
    // Algorithm 1's test on changed + skipped: the skipped vertices bound what
    // a plain sweep of this iteration could have changed in addition
    else stop = !st->pl && (double)(changed + st->skipped) < st->tol * (double)n;
    // near the stop (changed < 2 tol N) the next iteration is a plain sweep
    st->cand = (double)changed < 2.0 * st->tol * (double)n ? 1 : 0;
    st->iter = l + 1;
    const int ended = (stop || l + 1 >= st->cap) ? 1 : 0;
    st->stop = ended;
    // for the host, which launches on while iterations run: the word alone is
    // read there, so that no other write has to be visible with it
    __hip_atomic_store(progress,
                       (unsigned long long)st->seq << 32 | (unsigned int)ended << 31 |
                           (unsigned int)(l + 1),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    ended_sh = ended;
  }
  __syncthreads();
  if (next && !ended_sh) begin_iteration(st);
}

hipError_t launch_iter_end(DevStats* st, DevIterStats* hist, int64_t n, bool fold,
                           unsigned long long* progress, const FlagRule* rule, bool next,
                           hipStream_t s) {
  const FlagRule r = rule ? *rule : FlagRule{-1, 0, 0, 0};
  if (fold)
    hipLaunchKernelGGL(k_iter_end<true>, dim3(1), dim3(1024), 0, s, st, hist, n, progress, r,
                       next ? 1 : 0);
  else
    hipLaunchKernelGGL(k_iter_end<false>, dim3(1), dim3(64), 0, s, st, hist, n, progress, r,
                       next ? 1 : 0);
  return hipGetLastError();
}

// ---- batched runs: per-graph stop rule ------------------------------------------
// One workgroup per graph: count the graph's changed vertices, apply Algorithm
// 1's stop test with the graph's own vertex count, and clear the flags of a
// graph that stops so that none of its vertices is processed again.  All
// graphs share the iteration counter, so each follows its solo schedule.
__global__ __launch_bounds__(kBT) void k_batch_step(BatchArgs b, const uint8_t* chg,
                                                    uint8_t* F, DevStats* st) {
  __shared__ unsigned int cnt[kBT / 64];
  __shared__ int fin;
  if (st->stop) return;
  for (int32_t g = blockIdx.x; g < b.G; g += gridDim.x) {
    if (b.done[g]) continue;
    const int64_t v0 = b.v_off[g], v1 = b.v_off[g + 1];
    unsigned int c = 0;
    for (int64_t v = v0 + threadIdx.x; v < v1; v += kBT) c += chg[v];
    for (int ofs = 32; ofs > 0; ofs >>= 1) c += __shfl_xor(c, ofs);
    if ((threadIdx.x & 63) == 0) cnt[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long t = 0;
      for (int q = 0; q < kBT / 64; ++q) t += cnt[q];
      b.changed_last[g] = (long long)t;
      const int l = st->iter;
      const bool f = (!st->pl && (double)t < st->tol * (double)(v1 - v0)) || l + 1 >= st->cap;
      if (f) {
        b.done[g] = 1;
        b.iters[g] = l + 1;
      } else {
        atomicAdd(&st->graphs_left, 1u);
      }
      fin = f;
    }
    __syncthreads();
    if (fin)
      for (int64_t v = v0 + threadIdx.x; v < v1; v += kBT) F[v] = 0;
    __syncthreads();
  }
}

hipError_t launch_batch_step(const BatchArgs& b, const uint8_t* chg, uint8_t* F, DevStats* st,
                             hipStream_t s) {
  const int g = b.G < 8192 ? (b.G > 0 ? b.G : 1) : 8192;
  hipLaunchKernelGGL(k_batch_step, dim3(g), dim3(kBT), 0, s, b, chg, F, st);
  return hipGetLastError();
}

__global__ void k_batch_reset(BatchArgs b) {
  for (int32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < b.G; g += gridDim.x * blockDim.x) {
    b.done[g] = b.v_off[g + 1] == b.v_off[g];  // an empty graph performs no iteration
    b.iters[g] = 0;
    b.changed_last[g] = 0;
  }
}

hipError_t launch_batch_reset(const BatchArgs& b, hipStream_t s) {
  hipLaunchKernelGGL(k_batch_reset, dim3(grid_for(b.G, kBT, 1024)), dim3(kBT), 0, s, b);
  return hipGetLastError();
}

// every CSR entry of graph g must point into graph g (error bit 16)
template <typename OffT>
__global__ void k_batch_validate(const OffT* off, const int32_t* tgt, BatchArgs b, int64_t n,
                                 DevStats* st) {
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x) {
    int32_t lo = 0, hi = b.G - 1;  // graph holding v: largest g with v_off[g] <= v
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (b.v_off[mid] <= v) lo = mid; else hi = mid - 1;
    }
    const int64_t a0 = b.v_off[lo], a1 = b.v_off[lo + 1];
    for (int64_t e = (int64_t)off[v]; e < (int64_t)off[v + 1]; ++e)
      if ((int64_t)tgt[e] < a0 || (int64_t)tgt[e] >= a1) {
        set_error(st, 16u);
        break;
      }
  }
}

hipError_t launch_batch_validate(bool off64, const void* off, const int32_t* tgt,
                                 const BatchArgs& b, int64_t n, DevStats* st, hipStream_t s) {
  const int g = grid_for(n, kBT, 8192);
  if (off64)
    hipLaunchKernelGGL(k_batch_validate<int64_t>, dim3(g), dim3(kBT), 0, s,
                       (const int64_t*)off, tgt, b, n, st);
  else
    hipLaunchKernelGGL(k_batch_validate<int32_t>, dim3(g), dim3(kBT), 0, s,
                       (const int32_t*)off, tgt, b, n, st);
  return hipGetLastError();
}

// ---- validation (error bits: 1 offsets, 2 targets, 8 weights) ----------------
template <typename OffT>
__global__ void k_validate(const OffT* off, const int32_t* tgt, const float* w,
                           int64_t n, int64_t m, DevStats* st) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t0 == 0 && ((int64_t)off[0] != 0 || (int64_t)off[n] != m)) set_error(st, 1u);
  for (int64_t i = t0; i < n; i += stride)
    if (off[i] > off[i + 1]) set_error(st, 1u);
  for (int64_t e = t0; e < m; e += stride) {
    const int32_t j = tgt[e];
    if (j < 0 || (int64_t)j >= n) set_error(st, 2u);
    if (w) {
      const uint32_t b = __float_as_uint(w[e]);
      // reject negative (sign bit set, including -0.0), infinities and NaN
      if ((b >> 31) || ((b >> 23) & 0xFFu) == 0xFFu) set_error(st, 8u);
    }
  }
}

hipError_t launch_validate(bool off64, const void* off, const int32_t* tgt,
                           const float* w, int64_t n, int64_t m, DevStats* st,
                           hipStream_t s) {
  const int g = grid_for(m > n ? m : n, kBT, 8192);
  if (off64)
    hipLaunchKernelGGL(k_validate<int64_t>, dim3(g), dim3(kBT), 0, s,
                       (const int64_t*)off, tgt, w, n, m, st);
  else
    hipLaunchKernelGGL(k_validate<int32_t>, dim3(g), dim3(kBT), 0, s,
                       (const int32_t*)off, tgt, w, n, m, st);
  return hipGetLastError();
}

// Any weight other than 1.0f: other[0] receives 1 (else the weights are unit
// weights, and the kernels need not read them).  Any that is not a whole number
// of at most 2^18: other[1] receives 1 (else 64 of them sum exactly in any order).
__global__ void k_unit_weights(const float* w, int64_t m, unsigned int* other) {
  constexpr int U = 4;  // loads in flight
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  bool any = false, rounds = false;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < m; e += U * stride) {
    float x[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      x[u] = e + u * stride < m ? __builtin_nontemporal_load(&w[e + u * stride]) : 1.0f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      any |= __float_as_uint(x[u]) != 0x3F800000u;
      rounds |= !(x[u] >= 0.0f && x[u] <= 262144.0f && x[u] == truncf(x[u]));
    }
  }
  if (__any(any) && (threadIdx.x & 63) == 0) other[0] = 1u;
  if (__any(rounds) && (threadIdx.x & 63) == 0) other[1] = 1u;
}

hipError_t launch_unit_weights(const float* w, int64_t m, unsigned int* other, hipStream_t s) {
  hipError_t e = launch_fill_u32(other, 0u, 2, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_unit_weights, dim3(grid_for(m, kBT, 8192)), dim3(kBT), 0, s, w, m, other);
  return hipGetLastError();
}

// Rows with strictly increasing targets (sorted, no repeated neighbour):
// mark the first entry of every non-empty row, then flag any entry whose
// successor in the same row is not larger.  bad receives 1 on a violation.
template <typename OffT>
__global__ void k_mark_row_starts(const OffT* off, int64_t n, uint8_t* mark) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    if (off[i] < off[i + 1]) mark[off[i]] = 1;
}

__global__ void k_rows_strict(const int32_t* tgt, const uint8_t* mark, int64_t m,
                              unsigned int* bad) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e + 1 < m;
       e += (int64_t)gridDim.x * blockDim.x)
    if (!mark[e + 1] && tgt[e] >= tgt[e + 1]) *bad = 1u;
}

hipError_t launch_rows_strict(bool off64, const void* off, const int32_t* tgt, int64_t n,
                              int64_t m, uint8_t* mark, unsigned int* bad, hipStream_t s) {
  hipError_t e = launch_fill_u8(mark, 0, m, s);
  if (e != hipSuccess) return e;
  e = launch_fill_u32(bad, 0u, 1, s);
  if (e != hipSuccess) return e;
  if (off64)
    hipLaunchKernelGGL(k_mark_row_starts<int64_t>, dim3(grid_for(n, kBT, 8192)), dim3(kBT), 0,
                       s, (const int64_t*)off, n, mark);
  else
    hipLaunchKernelGGL(k_mark_row_starts<int32_t>, dim3(grid_for(n, kBT, 8192)), dim3(kBT), 0,
                       s, (const int32_t*)off, n, mark);
  hipLaunchKernelGGL(k_rows_strict, dim3(grid_for(m, kBT, 16384)), dim3(kBT), 0, s, tgt, mark, m,
                     bad);
  return hipGetLastError();
}

// Label-read probe: one pass that only reads every CSR entry's target and
// its neighbour's label, in the order the sweep kernels read them (8 entries
// in flight per lane).  Its rate bounds any sweep that must read them.
__global__ __launch_bounds__(256) void k_label_read_probe(const int32_t* tgt, int64_t m,
                                                          const int32_t* C, uint32_t* sink) {
  constexpr int U = 8;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t T = (int64_t)gridDim.x * 256;
  uint32_t acc = 0;
  int64_t e = t;
  for (; e + (U - 1) * T < m; e += U * T) {
    int32_t j[U];
#pragma unroll
    for (int u = 0; u < U; ++u) j[u] = __builtin_nontemporal_load(&tgt[e + u * T]);
#pragma unroll
    for (int u = 0; u < U; ++u) acc += (uint32_t)C[j[u]];
  }
  for (; e < m; e += T) acc += (uint32_t)C[__builtin_nontemporal_load(&tgt[e])];
  sink[t] = acc;
}

hipError_t launch_label_read_probe(const int32_t* tgt, int64_t m, const int32_t* C,
                                   uint32_t* sink, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_label_read_probe, dim3(grid), dim3(256), 0, s, tgt, m, C, sink);
  return hipGetLastError();
}

__global__ void k_check_labels(int64_t n, const int32_t* lab, DevStats* st) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    if (lab[i] < 0 || (int64_t)lab[i] >= n) set_error(st, 4u);
}

hipError_t launch_check_labels(int64_t n, const int32_t* lab, DevStats* st, hipStream_t s) {
  hipLaunchKernelGGL(k_check_labels, dim3(grid_for(n, kBT, 8192)), dim3(kBT), 0, s, n, lab, st);
  return hipGetLastError();
}

// ---- degree classes -------------------------------------------------------------
struct Bounds { int32_t hi[kNumClasses]; };

template <typename OffT>
__global__ void k_classify(const OffT* off, int64_t n, Bounds b, uint8_t* cls,
                           unsigned long long* counts, int32_t* hub_out,
                           unsigned int* hub_count) {
  __shared__ unsigned int cnt[kNumClasses];
  if (threadIdx.x < kNumClasses) cnt[threadIdx.x] = 0;
  __syncthreads();
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x) {
    const int64_t d = (int64_t)off[v + 1] - (int64_t)off[v];
    int c = kClassHub;
    if (d == 0) {
      c = 0;
    } else {
      for (int q = 1; q < kClassHub; ++q)
        if (d <= b.hi[q]) { c = q; break; }
    }
    cls[v] = (uint8_t)c;
    atomicAdd(&cnt[c], 1u);
    if (c == kClassHub) hub_out[atomicAdd(hub_count, 1u)] = (int32_t)v;
  }
  __syncthreads();
  if (threadIdx.x < kNumClasses && cnt[threadIdx.x])
    atomicAdd(&counts[threadIdx.x], (unsigned long long)cnt[threadIdx.x]);
}

hipError_t launch_classify(bool off64, const void* off, int64_t n, const int32_t* bounds,
                           uint8_t* cls, unsigned long long* counts, int32_t* hub_out,
                           unsigned int* hub_count, hipStream_t s) {
  Bounds b;
  for (int q = 0; q < kNumClasses; ++q) b.hi[q] = bounds[q];
  const int g = grid_for(n, kBT, 8192);
  if (off64)
    hipLaunchKernelGGL(k_classify<int64_t>, dim3(g), dim3(kBT), 0, s, (const int64_t*)off,
                       n, b, cls, counts, hub_out, hub_count);
  else
    hipLaunchKernelGGL(k_classify<int32_t>, dim3(g), dim3(kBT), 0, s, (const int32_t*)off,
                       n, b, cls, counts, hub_out, hub_count);
  return hipGetLastError();
}

template <typename OffT>
__global__ void k_gather_degrees(const OffT* off, const int32_t* vids, int32_t h, int64_t* deg) {
  for (int32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < h; i += gridDim.x * blockDim.x)
    deg[i] = (int64_t)off[vids[i] + 1] - (int64_t)off[vids[i]];
}

hipError_t launch_gather_degrees(bool off64, const void* off, const int32_t* vids, int32_t h,
                                 int64_t* deg, hipStream_t s) {
  const int g = grid_for(h, kBT, 4096);
  if (off64)
    hipLaunchKernelGGL(k_gather_degrees<int64_t>, dim3(g), dim3(kBT), 0, s, (const int64_t*)off, vids, h, deg);
  else
    hipLaunchKernelGGL(k_gather_degrees<int32_t>, dim3(g), dim3(kBT), 0, s, (const int32_t*)off, vids, h, deg);
  return hipGetLastError();
}

// Position of each hub slice's middle entry in the id order by entry mass:
// the row offset of its target (the entries of all rows before it).  Slices
// are listed as (hub index, slice index) pairs.
template <typename OffT>
__global__ void k_slice_keys(const OffT* off, const int32_t* tgt, const int32_t* hub_vid,
                             const uint32_t* sl, int64_t ns, int chunk, int64_t* key) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= ns) return;
  const int32_t v = hub_vid[sl[2 * i]];
  const int64_t c = sl[2 * i + 1];
  const int64_t o = (int64_t)off[v], d = (int64_t)off[v + 1] - o;
  const int64_t e0 = c * chunk;
  const int64_t n = d - e0 < chunk ? d - e0 : chunk;
  key[i] = (int64_t)off[tgt[o + e0 + n / 2]];
}

hipError_t launch_slice_keys(bool off64, const void* off, const int32_t* tgt,
                             const int32_t* hub_vid, const uint32_t* sl, int64_t ns, int chunk,
                             int64_t* key, hipStream_t s) {
  const int g = grid_for(ns, kBT, 1 << 20);
  if (off64)
    hipLaunchKernelGGL(k_slice_keys<int64_t>, dim3(g), dim3(kBT), 0, s, (const int64_t*)off, tgt,
                       hub_vid, sl, ns, chunk, key);
  else
    hipLaunchKernelGGL(k_slice_keys<int32_t>, dim3(g), dim3(kBT), 0, s, (const int32_t*)off, tgt,
                       hub_vid, sl, ns, chunk, key);
  return hipGetLastError();
}

hipError_t launch_fill_u8(uint8_t* p, uint8_t v, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_fill<uint8_t>, dim3(grid_for(count, kBT, 8192)), dim3(kBT), 0, s, p, v, count);
  return hipGetLastError();
}
hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_fill<uint32_t>, dim3(grid_for(count, kBT, 8192)), dim3(kBT), 0, s, p, v, count);
  return hipGetLastError();
}
hipError_t launch_fill_f32(float* p, float v, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_fill<float>, dim3(grid_for(count, kBT, 8192)), dim3(kBT), 0, s, p, v, count);
  return hipGetLastError();
}
hipError_t launch_fill_f64(double* p, double v, int64_t count, hipStream_t s) {
  hipLaunchKernelGGL(k_fill<double>, dim3(grid_for(count, kBT, 8192)), dim3(kBT), 0, s, p, v, count);
  return hipGetLastError();
}
hipError_t launch_fill_u64(unsigned long long* p, unsigned long long v, int64_t count,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_fill<unsigned long long>, dim3(grid_for(count, kBT, 8192)), dim3(kBT), 0,
                     s, p, v, count);
  return hipGetLastError();
}

// ---- hub plan: reset the iteration counters, take the flagged hubs, queue
// their slices and their label buckets.  One workgroup of 1024 threads. -------
template <typename OffT>
__global__ __launch_bounds__(1024) void k_hub_plan(HubArgs a, int32_t* C, uint8_t* F) {
  __shared__ uint32_t ws[16], wb[16];
  __shared__ uint32_t run_s, run_b;
  __shared__ uint32_t nproc;
  const int tid = threadIdx.x;
  DevStats* st = a.st;
  if (st->stop) return;
  begin_iteration(st);
  if (tid == 0) {
    run_s = 0; run_b = 0; nproc = 0;
  }
  if (a.witems && tid < kXcds) a.wctr[tid * kQueueCtrStride] = 0u;
  __syncthreads();
  const OffT* off = reinterpret_cast<const OffT*>(a.off);
  // each hub's slice count (0 unless flagged), kB tiles of 1024 hubs at a
  // time, so that the dependent loads of kB hubs per thread (hub vertex, its
  // flag, its row offsets) are in flight together; thread tid takes hubs
  // tid mod 1024 in both passes and reads back only what it wrote
  constexpr int kB = 4;
  for (int32_t t0 = 0; t0 < a.H; t0 += 1024 * kB) {
    int32_t hv[kB];
    uint8_t hf[kB];
#pragma unroll
    for (int q = 0; q < kB; ++q) {
      const int32_t h = t0 + q * 1024 + tid;
      hv[q] = h < a.H ? a.hub_vid[h] : -1;
    }
#pragma unroll
    for (int q = 0; q < kB; ++q) hf[q] = hv[q] >= 0 ? F[hv[q]] : (uint8_t)0;
#pragma unroll
    for (int q = 0; q < kB; ++q) {
      const int32_t h = t0 + q * 1024 + tid;
      if (h >= a.H) continue;
      const int32_t v = hv[q];
      a.hub_best[h] = 0ull;
      a.hub_ovf[h] = 0;
      uint32_t nch = 0;
      if (hf[q]) {
        F[v] = 0;
        a.hub_old[h] = C[v];
        const int64_t d = (int64_t)off[v + 1] - (int64_t)off[v];
        nch = (uint32_t)((d + a.chunk - 1) / a.chunk);
        atomicAdd(&nproc, 1u);
      }
      a.hub_nch[h] = (int32_t)nch;
    }
  }
  // queue the flagged hubs' slices and buckets: a scan of both counts over
  // each tile of 1024 hubs (within each wave by shuffles, then over the
  // waves' totals); the next tile's counts are loaded during this one's
  const int lane = tid & 63, wv = tid >> 6;
  uint32_t rs = 0, rb = 0;  // slices and buckets queued by earlier tiles
  int32_t nch_n = tid < a.H ? a.hub_nch[tid] : 0;
  int32_t lgb_n = tid < a.H ? a.hub_lgb[tid] : 0;
  for (int32_t tile = 0; tile < a.H; tile += 1024) {
    const int32_t h = tile + tid;
    const uint32_t nch = (uint32_t)nch_n;
    const uint32_t nbk = nch ? 1u << lgb_n : 0u;
    if (h + 1024 < a.H) {
      nch_n = a.hub_nch[h + 1024];
      lgb_n = a.hub_lgb[h + 1024];
    } else {
      nch_n = 0;
      lgb_n = 0;
    }
    uint32_t xs = nch, xb = nbk;  // inclusive scans within the wave
#pragma unroll
    for (int ofs = 1; ofs < 64; ofs <<= 1) {
      const uint32_t ys = __shfl_up(xs, ofs), yb = __shfl_up(xb, ofs);
      if (lane >= ofs) {
        xs += ys;
        xb += yb;
      }
    }
    if (lane == 63) {
      ws[wv] = xs;
      wb[wv] = xb;
    }
    __syncthreads();
    uint32_t bs = 0, bb = 0, ts = 0, tb = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      if (w < wv) {
        bs += ws[w];
        bb += wb[w];
      }
      ts += ws[w];
      tb += wb[w];
    }
    const uint32_t fs = rs + bs + xs - nch;
    const uint32_t fb = rb + bb + xb - nbk;
    for (uint32_t c = 0; c < nch; ++c) {
      a.items[2 * (uint64_t)(fs + c)] = (uint32_t)h;
      a.items[2 * (uint64_t)(fs + c) + 1] = c;
    }
    for (uint32_t b = 0; b < nbk; ++b) {
      a.bitems[2 * (uint64_t)(fb + b)] = (uint32_t)h;
      a.bitems[2 * (uint64_t)(fb + b) + 1] = b;
      a.bsize[fb + b] = 0u;
    }
    if (nbk) a.hub_bq[h] = (int32_t)fb;
    rs += ts;
    rb += tb;
    __syncthreads();  // ws and wb are rewritten by the next tile
  }
  if (tid == 0) {
    run_s = rs;
    run_b = rb;
  }
  __syncthreads();
  if (tid == 0) {
    st->hub_items = run_s;
    st->hub_bitems = run_b;
    st->processed = nproc;
    st->hub_all = (int32_t)nproc == a.H ? 1u : 0u;
  }
}

hipError_t launch_hub_plan(bool off64, const HubArgs& a, int32_t* C, uint8_t* F,
                           hipStream_t s) {
  if (off64)
    hipLaunchKernelGGL(k_hub_plan<int64_t>, dim3(1), dim3(1024), 0, s, a, C, F);
  else
    hipLaunchKernelGGL(k_hub_plan<int32_t>, dim3(1), dim3(1024), 0, s, a, C, F);
  return hipGetLastError();
}

// ---- frontier: append flagged vertices to their class list, clear flags ------
struct ListPtrs { int32_t* p[kNumClasses]; };

// Words per thread and step by vertex count: few words spread a small graph's
// steps over the chip, many keep the count of global atomics down (1 M
// vertices: 22 us with one word, 13 with four, 20 with eight; 10 000: 5.7 us
// with one, 16 with eight).
constexpr int64_t kFrontierOneWord = (int64_t)1 << 18, kFrontierFourWords = (int64_t)1 << 22;

// kWords words of four vertices per thread and block step: the block's
// appends cost one global atomic per class and step.  A wave whose 256
// vertices are all listed in one class skips the placing, and four vertices
// of one class are stored at once.  67 M vertices (8192 x 8192 lattice), per
// launch: 212 -> 174 us; the flags, classes and list entries alone take 106.
template <int kWords>
__global__ __launch_bounds__(kBT) void k_frontier(int64_t n_all, int64_t n_later, uint8_t* F,
                                                  const uint8_t* cls, ListPtrs lists,
                                                  uint8_t* chg_clear, DevStats* st) {
  constexpr int64_t kStep = (int64_t)kBT * kWords * 4;
  static_assert(kStep <= 65536, "places within a step are kept in 16 bits");
  __shared__ uint32_t cnt[kNumClasses];
  __shared__ int32_t* out[kNumClasses];  // where this step's vertices of a class go
  if (st->stop) return;
  // vertices scanned: all in the first iteration, then n_later (the
  // vertices of degree 0, last in the internal order, are flagged only by
  // the initialisation)
  const int64_t n = st->iter == 0 ? n_all : n_later;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  uint32_t proc = 0;
  for (int64_t chunk = (int64_t)blockIdx.x * kStep; chunk < n; chunk += (int64_t)gridDim.x * kStep) {
    if (tid < kNumClasses) cnt[tid] = 0;
    __syncthreads();
    // word k of this thread holds vertices v0[k] .. v0[k] + 3 (coalesced)
    int64_t v0[kWords];
    uint32_t f4[kWords], c4[kWords];
#pragma unroll
    for (int k = 0; k < kWords; ++k) {
      v0[k] = chunk + ((int64_t)k * kBT + tid) * 4;
      f4[k] = 0u;
      c4[k] = 0u;
      if (v0[k] + 3 < n) {
        f4[k] = *reinterpret_cast<const uint32_t*>(F + v0[k]);
        c4[k] = *reinterpret_cast<const uint32_t*>(cls + v0[k]);
        *reinterpret_cast<uint32_t*>(chg_clear + v0[k]) = 0u;
        if (f4[k]) *reinterpret_cast<uint32_t*>(F + v0[k]) = 0u;
      } else {
        for (int q = 0; q < 4 && v0[k] + q < n; ++q) {
          f4[k] |= (uint32_t)F[v0[k] + q] << (8 * q);
          c4[k] |= (uint32_t)cls[v0[k] + q] << (8 * q);
          chg_clear[v0[k] + q] = 0;
          F[v0[k] + q] = 0;
        }
      }
    }
    // class of each vertex to be listed (byte q of c4; 0: none) and its place
    // among those of its class (half q & 1 of pos[q >> 1]), in vertex order
    // within the wave's 256 vertices of word k: the sweeps' loads and stores
    // by listed vertex then fall on consecutive addresses where consecutive
    // vertices are listed.  (Placed byte by byte of the words instead, 64
    // lanes spanned 256 vertices: 0.88 against 0.48 ms per sweep of the 67 M
    // short rows of an 8192 x 8192 lattice, 0.29 against 0.18 ms per label
    // copy; R-MAT 26 56.0 against 54.5 ms per run.)
    uint32_t pos[kWords][2];
#pragma unroll
    for (int k = 0; k < kWords; ++k) {
      const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)c4[k]);
      const bool all4 = ((f4[k] - 0x01010101u) & ~f4[k] & 0x80808080u) == 0u;
      pos[k][0] = pos[k][1] = 0u;
      if (__all(all4 && c4[k] == first) && first == (first & 0xFFu) * 0x01010101u &&
          first != 0u && (first & 0xFFu) != (uint32_t)kClassHub) {
        // all 256 vertices listed, in one class
        uint32_t b = 0;
        if (lane == 0) b = atomicAdd(&cnt[first & 0xFFu], 256u);
        b = (uint32_t)__builtin_amdgcn_readfirstlane((int)b) + 4u * (uint32_t)lane;
        pos[k][0] = b | (b + 1u) << 16;
        pos[k][1] = (b + 2u) | (b + 3u) << 16;
        proc += 4u;
        continue;
      }
      uint32_t todo = 0u;  // q with a vertex still to be placed
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool f = ((f4[k] >> (8 * q)) & 0xFFu) != 0u;
        const uint32_t c = (c4[k] >> (8 * q)) & 0xFFu;
        proc += f ? 1u : 0u;
        if (f && c != 0u && c != (uint32_t)kClassHub) todo |= 1u << q;
        else c4[k] &= ~(0xFFu << (8 * q));
      }
      unsigned long long left = __ballot(todo != 0u);
      // one LDS atomic per class present in the wave
      while (left) {
        const int src = __ffsll((long long)left) - 1;
        const uint32_t mine = todo ? (c4[k] >> (8 * (__ffs((int)todo) - 1))) & 0xFFu : 0u;
        const uint32_t cc = (uint32_t)__builtin_amdgcn_readlane((int)mine, src);
        uint32_t total = 0, before = 0;
        uint32_t in4 = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bool in = ((c4[k] >> (8 * q)) & 0xFFu) == cc;
          const unsigned long long m = __ballot(in);
          total += (uint32_t)__popcll(m);
          before += lane_rank(m);
          in4 |= in ? 1u << q : 0u;
        }
        todo &= ~in4;
        uint32_t b = 0;
        if (lane == 0) b = atomicAdd(&cnt[cc], total);
        b = (uint32_t)__builtin_amdgcn_readfirstlane((int)b) + before;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (in4 & (1u << q)) pos[k][q >> 1] |= b++ << (16 * (q & 1));
        left = __ballot(todo != 0u);
      }
    }
    __syncthreads();
    if (tid < kNumClasses && cnt[tid])
      out[tid] = lists.p[tid] + atomicAdd(&st->active[tid].n, cnt[tid]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kWords; ++k) {
      const uint32_t c0 = c4[k] & 0xFFu;
      if (c0 != 0u && c4[k] == c0 * 0x01010101u) {
        // four of one class: their places follow one another
        const int32_t v = (int32_t)v0[k];
        const int4 four = make_int4(v, v + 1, v + 2, v + 3);
        __builtin_memcpy(out[c0] + (pos[k][0] & 0xFFFFu), &four, sizeof(four));
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t c = (c4[k] >> (8 * q)) & 0xFFu;
          if (c) out[c][pos[k][q >> 1] >> (16 * (q & 1)) & 0xFFFFu] = (int32_t)(v0[k] + q);
        }
      }
    }
    __syncthreads();
  }
  // one atomic per workgroup for the processed count (cnt is free after the
  // last step's barrier; every thread of the workgroup gets here)
  uint32_t x = proc;
  for (int ofs = 32; ofs > 0; ofs >>= 1) x += __shfl_xor(x, ofs);
  if ((tid & 63) == 0) cnt[tid >> 6] = x;
  __syncthreads();
  if (tid == 0) {
    uint32_t t = 0;
    for (int q = 0; q < kBT / 64; ++q) t += cnt[q];
    if (t) atomicAdd(&stat_slot(st)[kStatProcessed], (unsigned long long)t);
  }
}

hipError_t launch_frontier(int64_t n, int64_t n_later, uint8_t* F, const uint8_t* cls,
                           int32_t* const* lists, uint8_t* chg_clear, DevStats* st, hipStream_t s) {
  ListPtrs lp;
  for (int q = 0; q < kNumClasses; ++q) lp.p[q] = lists[q];
  if (n <= kFrontierOneWord)
    hipLaunchKernelGGL(k_frontier<1>, dim3(grid_for(n, kBT * 4, 2048)), dim3(kBT), 0, s, n,
                       n_later, F, cls, lp, chg_clear, st);
  else if (n <= kFrontierFourWords)
    hipLaunchKernelGGL(k_frontier<4>, dim3(grid_for(n, kBT * 16, 2048)), dim3(kBT), 0, s, n,
                       n_later, F, cls, lp, chg_clear, st);
  else
    hipLaunchKernelGGL(k_frontier<8>, dim3(grid_for(n, kBT * 32, 2048)), dim3(kBT), 0, s, n,
                       n_later, F, cls, lp, chg_clear, st);
  return hipGetLastError();
}

// ---- frontier with the change predictor (learned variant) ------------------------
// One wave per 64 consecutive vertices.  The flagged vertices of classes 1..8
// are compacted within the wave and, when this iteration predicts, run through
// the network 16 at a time (one MFMA tile of samples, operands held in
// registers for the whole kernel).  In a skipping iteration a vertex whose
// logit is below z_theta keeps its flag and is not listed; in a plain one it
// is listed and marked (record byte 6, bit 7) so that the sweep counts it if
// it changes.  Trace samples (features of a listed vertex) are appended here;
// their targets are filled in after the sweep.
namespace {

__device__ __forceinline__ double sample_draw(unsigned long long seed, int l, int64_t v) {
  unsigned long long z = seed + 0x9E3779B97F4A7C15ull *
                                    (1ull + (((unsigned long long)(uint32_t)l << 32) |
                                             (unsigned long long)v));
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (double)(z >> 11) * (1.0 / 9007199254740992.0);
}

}  // namespace

constexpr int kLearnWaves = 4;
constexpr int kLearnChunks = 4;  // 64-vertex chunks per wave and block step

__global__ __launch_bounds__(kLearnWaves * 64) void k_frontier_learned(
    int64_t n_all, int64_t n_later, uint8_t* F, const uint8_t* cls, ListPtrs lists,
    uint8_t* chg_clear, DevStats* st, unsigned long long* rec, const MlpTiles* tiles,
    TraceArgs tr) {
  __shared__ uint8_t lst_all[kLearnWaves][64];
  __shared__ uint8_t dec_all[kLearnWaves][64];
  __shared__ unsigned long long slot_all[kLearnWaves][16];
  __shared__ uint32_t cnt[kNumClasses];
  __shared__ uint32_t cbase[kNumClasses];
  // the network's operand tiles, read from LDS at each use: held in
  // registers they would leave room for two waves per SIMD
  __shared__ MlpTiles wl;
  if (st->stop) return;
  const int64_t n = st->iter == 0 ? n_all : n_later;  // as in k_frontier
  const int tid = threadIdx.x;
  const int wv = tid >> 6;
  const int lane = tid & 63;
  const int g = lane >> 4;
  uint8_t* lst = lst_all[wv];
  uint8_t* dec = dec_all[wv];
  unsigned long long* slot = slot_all[wv];
  const int l = st->iter;
  const int cap = st->cap, rho = st->rho;
  const bool predict = st->predict != 0;
  const bool skipping = st->skipping != 0;
  // rows of other classes are never predicted or traced
  const int cmin = st->pred_cmin, cmax = st->pred_cmax;
  const bool tracing = st->trace != 0 && l >= st->pred_start && tr.X != nullptr;
  const float z_theta = st->z_theta;
  const double rate = st->trace_rate;
  const unsigned long long seed = st->trace_seed, tcap = st->trace_cap;
  if (predict) {
    static_assert(sizeof(MlpTiles) % 4 == 0, "tiles are copied as words");
    const uint32_t* src = reinterpret_cast<const uint32_t*>(tiles);
    uint32_t* dst = reinterpret_cast<uint32_t*>(&wl);
    for (int q = tid; q < (int)(sizeof(MlpTiles) / 4); q += kLearnWaves * 64) dst[q] = src[q];
  }
  __syncthreads();
  const MlpFromTiles W{wl, lane, g};
  uint32_t proc = 0, skipped = 0, npred = 0;
  constexpr int64_t kStep = (int64_t)kLearnWaves * kLearnChunks * 64;
  // the whole workgroup walks the same steps of kStep vertices (barriers
  // inside); the listed vertices of a step are appended with one atomic per
  // class and workgroup, as in the plain frontier
  for (int64_t step0 = (int64_t)blockIdx.x * kStep; step0 < n;
       step0 += (int64_t)gridDim.x * kStep) {
    if (tid < kNumClasses) cnt[tid] = 0;
    __syncthreads();
    int8_t cq[kLearnChunks];
    uint32_t pos[kLearnChunks];
    // flags, classes and records of the wave's chunks, loaded together (the
    // records of listed vertices reach their tile lanes by shuffles)
    uint8_t fq[kLearnChunks], cl[kLearnChunks];
    unsigned long long rq[kLearnChunks];
#pragma unroll
    for (int q = 0; q < kLearnChunks; ++q) {
      const int64_t v = step0 + ((int64_t)wv * kLearnChunks + q) * 64 + lane;
      fq[q] = 0;
      cl[q] = 0;
      rq[q] = kRecordInit;
      if (v < n) {
        fq[q] = F[v];
        cl[q] = cls[v];
        if (predict || tracing) rq[q] = rec[v];
        chg_clear[v] = 0;
      }
    }
#pragma unroll
    for (int q = 0; q < kLearnChunks; ++q) {
      const int64_t base = step0 + ((int64_t)wv * kLearnChunks + q) * 64;
      const int64_t v = base + lane;
      const uint8_t f = fq[q], c = cl[q];
      const bool cand = f && c >= cmin && c <= cmax && (predict || tracing);
      const unsigned long long cm = __ballot(cand);
      const uint32_t ncand = __popcll(cm);
      if (cand) lst[lane_rank(cm)] = (uint8_t)lane;
      dec[lane] = 0;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      for (uint32_t r0 = 0; r0 < ncand; r0 += 16) {  // uniform trip count
        const uint32_t si = r0 + (uint32_t)(lane & 15);
        const bool has = si < ncand;
        const int src = has ? lst[si] : 0;
        const int64_t u = base + src;
        const uint32_t rlo = (uint32_t)__shfl((int)(uint32_t)rq[q], src);
        const uint32_t rhi = (uint32_t)__shfl((int)(uint32_t)(rq[q] >> 32), src);
        const unsigned long long rr =
            has ? (((unsigned long long)rhi << 32) | rlo) : kRecordInit;
        float x[4];
        rec_features(rr, l, cap, rho, g, x);
        bool pred = false;
        if (predict) {
          const float z = mlp_logit16_src(W, x);
          pred = has && z < z_theta;
        }
        const bool skip = pred && skipping;
        if (lane < 16 && has) dec[src] = (uint8_t)((pred ? 1 : 0) | (skip ? 2 : 0));
        if (tracing) {
          const int64_t uid = tr.inv ? (int64_t)tr.inv[u] : u;  // the caller's id
          const bool take = has && !skip && sample_draw(seed, l, uid) < rate;
          if (lane < 16) slot[lane] = take ? atomicAdd(&st->trace_n, 1ull) : ~0ull;
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
          const unsigned long long qq = slot[lane & 15];
          if (take && qq < tcap && g < 3) {
#pragma unroll
            for (int j = 0; j < 4; ++j) tr.X[qq * kMlpIn + 4 * g + j] = x[j];
            if (g == 0) {
              tr.v[qq] = (int32_t)uid;
              tr.l[qq] = l;
            }
          }
          __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      const uint8_t dd = dec[lane];
      const bool skip = (dd & 2) != 0;
      const bool keep = f && !skip;
      if (dd & 1) {
        ++npred;
        // plain iteration: mark for the false-negative count of the sweep
        if (!skip) rec[v] = rq[q] | (0x80ull << 48);
      }
      if (skip) ++skipped;
      cq[q] = -1;
      if (keep) {
        F[v] = 0;
        ++proc;
        if (c >= 1 && c < kClassHub) {
          cq[q] = (int8_t)c;
          pos[q] = atomicAdd(&cnt[c], 1u);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
    __syncthreads();
    if (tid < kNumClasses) cbase[tid] = cnt[tid] ? atomicAdd(&st->active[tid].n, cnt[tid]) : 0u;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kLearnChunks; ++q)
      if (cq[q] >= 0)
        lists.p[cq[q]][cbase[cq[q]] + pos[q]] =
            (int32_t)(step0 + ((int64_t)wv * kLearnChunks + q) * 64 + lane);
    __syncthreads();
  }
  // one atomic per counter and workgroup (cnt and cbase are free after the
  // last step's barrier; every thread of the workgroup gets here)
  const uint32_t tp = wave_sum_u32(proc), ts = wave_sum_u32(skipped), tn = wave_sum_u32(npred);
  if (lane == 0) {
    cnt[wv] = tp;
    cnt[kLearnWaves + wv] = ts;
    cbase[wv] = tn;
  }
  __syncthreads();
  if (tid == 0) {
    uint32_t sp = 0, ss = 0, sn = 0;
    for (int q = 0; q < kLearnWaves; ++q) {
      sp += cnt[q];
      ss += cnt[kLearnWaves + q];
      sn += cbase[q];
    }
    unsigned long long* slot = stat_slot(st);
    if (sp) atomicAdd(&slot[kStatProcessed], (unsigned long long)sp);
    if (ss) atomicAdd(&slot[kStatSkipped], (unsigned long long)ss);
    if (sn) atomicAdd(&slot[kStatNpred], (unsigned long long)sn);
  }
}

hipError_t launch_frontier_learned(int64_t n, int64_t n_later, uint8_t* F, const uint8_t* cls,
                                   int32_t* const* lists, uint8_t* chg_clear, DevStats* st,
                                   unsigned long long* rec, const MlpTiles* tiles,
                                   const TraceArgs& tr, int grid, hipStream_t s) {
  ListPtrs lp;
  for (int q = 0; q < kNumClasses; ++q) lp.p[q] = lists[q];
  hipLaunchKernelGGL(k_frontier_learned, dim3(grid), dim3(kLearnWaves * 64), 0, s, n, n_later,
                     F, cls, lp, chg_clear, st, rec, tiles, tr);
  return hipGetLastError();
}

// Targets of this iteration's trace samples: 1 if the vertex changed label.
__global__ void k_trace_label(const DevStats* st, const uint8_t* chg, TraceArgs tr) {
  if (st->stop || !st->trace) return;
  const unsigned long long end = st->trace_n < st->trace_cap ? st->trace_n : st->trace_cap;
  for (unsigned long long i = st->trace_first + blockIdx.x * (unsigned long long)blockDim.x +
                              threadIdx.x;
       i < end; i += (unsigned long long)gridDim.x * blockDim.x)
    tr.y[i] = chg[tr.perm ? tr.perm[tr.v[i]] : tr.v[i]] ? 1.0f : 0.0f;
}

hipError_t launch_trace_label(const DevStats* st, const uint8_t* chg, const TraceArgs& tr,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_trace_label, dim3(256), dim3(256), 0, s, st, chg, tr);
  return hipGetLastError();
}

// ---- neighbour flags ------------------------------------------------------------
// The sweep records each changed vertex in chg.  Every CSR neighbour of a
// changed vertex is then flagged for the next iteration (Sec. 4 item 4), in
// one of two equivalent ways on a symmetric CSR:
//   push: each changed vertex writes the flag byte of each neighbour;
//   pull: each vertex reads the change bytes of its neighbours and stops at
//         the first changed one.
// Push costs one scattered byte store (a line's read-modify-write) per entry
// of a changed row; pull costs a read per entry up to the first changed
// neighbour, about 1/p entries per vertex when the changed rows hold a share
// p of the entries.  On R-MAT scale 26 the two cost the same near p = 1/16
// (push of a quarter of the entries: 18.6 ms; pull at p near 1/2: 2.7 ms), so
// k_flag_decide picks pull when the changed rows hold at least 1/pdiv of the
// CSR entries (lpa_tuning.pull_divisor, default 16), push otherwise; the
// kernels of the other way return at once.
__global__ __launch_bounds__(1024) void k_flag_decide(DevStats* st, FlagRule rule) {
  if (st->stop) return;
  fold_stats(st);
  if (threadIdx.x != 0) return;
  unsigned long long fw = 0, changed = 0;
  for (int c = 0; c < kNumClasses; ++c) {
    fw += st->flagw[c];
    changed += st->changed[c];
  }
  st->pull_mode = flag_decision(st, rule, fw, changed - st->reverted, st->skipped);
  // its flags matter only to a later lpa_get_flags, which sets them then
  if (st->pull_mode == 2u) st->flags_deferred = 1u;
}

hipError_t launch_flag_decide(DevStats* st, const FlagRule& rule, hipStream_t s) {
  hipLaunchKernelGGL(k_flag_decide, dim3(1), dim3(1024), 0, s, st, rule);
  return hipGetLastError();
}

// ---- Cross-Check (Sec. 4.1) ---------------------------------------------------
__global__ void k_cc_save(const int32_t* C, int32_t* Cp, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    Cp[i] = C[i];
}

// One round of revert decisions.  A changed vertex (caller id u, new label c)
// reverts when vertex c, at its place in id order, does not hold label c:
// for c < u that is c's final label (its previous label if it reverts), for
// c > u its new label.  The decisions depend only on those of smaller ids, so
// repeating rounds until none changes reaches the id-order result.
__global__ void k_cc_round(const int32_t* C, const int32_t* Cp, const uint8_t* chg, uint8_t* R,
                           const int32_t* perm, const int32_t* inv, int64_t n, DevStats* st) {
  bool moved = false;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    if (!chg[i]) continue;
    const int32_t c = C[i];                       // new label = a caller id
    const int64_t u = inv ? (int64_t)inv[i] : i;  // this vertex's caller id
    const int64_t ci = perm ? (int64_t)perm[c] : (int64_t)c;  // vertex c, internal
    int32_t lab = C[ci];
    if ((int64_t)c < u && chg[ci] && R[ci]) lab = Cp[ci];
    const uint8_t r = lab != c ? 1 : 0;
    if (r != R[i]) {
      R[i] = r;
      moved = true;
    }
  }
  if (__any(moved) && (threadIdx.x & 63) == 0) st->cc_moved = 1u;
}

__global__ void k_cc_apply(int32_t* C, const int32_t* Cp, uint8_t* chg, uint8_t* R, int64_t n,
                           DevStats* st) {
  uint32_t rev = 0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    if (chg[i] && R[i]) {
      C[i] = Cp[i];
      chg[i] = 0;
      R[i] = 0;
      ++rev;
    }
  }
  for (int ofs = 32; ofs > 0; ofs >>= 1) rev += __shfl_xor(rev, ofs);
  if ((threadIdx.x & 63) == 0 && rev) atomicAdd(&st->reverted, (unsigned long long)rev);
}

__global__ void k_cc_clear_moved(DevStats* st) {
  if (threadIdx.x == 0 && blockIdx.x == 0) st->cc_moved = 0u;
}

hipError_t launch_cc_save(const int32_t* C, int32_t* Cp, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_cc_save, dim3(grid_for(n, kBT, 8192)), dim3(kBT), 0, s, C, Cp, n);
  return hipGetLastError();
}
hipError_t launch_cc_round(const int32_t* C, const int32_t* Cp, const uint8_t* chg, uint8_t* R,
                           const int32_t* perm, const int32_t* inv, int64_t n, DevStats* st,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_cc_clear_moved, dim3(1), dim3(64), 0, s, st);
  hipLaunchKernelGGL(k_cc_round, dim3(grid_for(n, kBT, 8192)), dim3(kBT), 0, s, C, Cp, chg, R,
                     perm, inv, n, st);
  return hipGetLastError();
}
hipError_t launch_cc_apply(int32_t* C, const int32_t* Cp, uint8_t* chg, uint8_t* R, int64_t n,
                           DevStats* st, hipStream_t s) {
  hipLaunchKernelGGL(k_cc_apply, dim3(grid_for(n, kBT, 8192)), dim3(kBT), 0, s, C, Cp, chg, R,
                     n, st);
  return hipGetLastError();
}

__global__ void k_flags_resume(DevStats* st) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    st->stop = 0;
    st->pull_mode = 1u;
  }
}
__global__ void k_flags_done(DevStats* st) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    st->stop = 1;
    st->pull_mode = 2u;
    st->flags_deferred = 0u;
  }
}
hipError_t launch_flags_resume(DevStats* st, hipStream_t s) {
  hipLaunchKernelGGL(k_flags_resume, dim3(1), dim3(64), 0, s, st);
  return hipGetLastError();
}
hipError_t launch_flags_done(DevStats* st, hipStream_t s) {
  hipLaunchKernelGGL(k_flags_done, dim3(1), dim3(64), 0, s, st);
  return hipGetLastError();
}

// push: classes 1..4 with 8 lanes per vertex, classes 5..8 with a workgroup
// per vertex (hub rows: k_push_hubs, one workgroup per slice)
template <typename OffT>
__device__ __forceinline__ void push_lists(const OffT* off, const int32_t* tgt,
                                           const ListPtrs& lists, const uint8_t* chg, uint8_t* F,
                                           const DevStats* st) {
  const int lane = threadIdx.x & 63;
  const int k = lane & 7;
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int c = 1; c <= 4; ++c) {
    const int64_t cnt = st->active[c];
    const int32_t* list = lists.p[c];
    for (int64_t base = wave * 8; base < cnt; base += nwaves * 8) {
      const int64_t idx = base + (lane >> 3);
      if (idx >= cnt) continue;
      const int32_t v = list[idx];
      if (!chg[v]) continue;
      const int64_t o = (int64_t)off[v], d = (int64_t)off[v + 1] - o;
      for (int64_t e = k; e < d; e += 8) F[tgt[o + e]] = 1;
    }
  }
  for (int c = 5; c < kClassHub; ++c) {
    const int64_t cnt = st->active[c];
    const int32_t* list = lists.p[c];
    for (int64_t item = blockIdx.x; item < cnt; item += gridDim.x) {
      const int32_t v = list[item];
      if (!chg[v]) continue;
      const int64_t o = (int64_t)off[v], d = (int64_t)off[v + 1] - o;
      for (int64_t e = threadIdx.x; e < d; e += blockDim.x) F[tgt[o + e]] = 1;
    }
  }
}

template <typename OffT>
__global__ __launch_bounds__(kBT) void k_push_lists(const OffT* off, const int32_t* tgt,
                                                    ListPtrs lists, const uint8_t* chg,
                                                    uint8_t* F, DevStats* st) {
  if (st->stop || st->pull_mode) return;
  push_lists(off, tgt, lists, chg, F, st);
}

hipError_t launch_push_lists(bool off64, const void* off, const int32_t* tgt,
                             int32_t* const* lists, const uint8_t* chg, uint8_t* F,
                             DevStats* st, int grid, hipStream_t s) {
  ListPtrs lp;
  for (int q = 0; q < kNumClasses; ++q) lp.p[q] = lists[q];
  if (off64)
    hipLaunchKernelGGL(k_push_lists<int64_t>, dim3(grid), dim3(kBT), 0, s,
                       (const int64_t*)off, tgt, lp, chg, F, st);
  else
    hipLaunchKernelGGL(k_push_lists<int32_t>, dim3(grid), dim3(kBT), 0, s,
                       (const int32_t*)off, tgt, lp, chg, F, st);
  return hipGetLastError();
}

template <typename OffT>
__global__ __launch_bounds__(kBT) void k_push_hubs(HubArgs a) {
  if (a.st->stop || a.st->pull_mode) return;
  const uint32_t nitems = a.st->hub_items;
  const OffT* off = reinterpret_cast<const OffT*>(a.off);
  for (uint32_t it = blockIdx.x; it < nitems; it += gridDim.x) {
    const int32_t h = (int32_t)a.items[2 * (uint64_t)it];
    const int32_t c = (int32_t)a.items[2 * (uint64_t)it + 1];
    const int32_t v = a.hub_vid[h];
    if (!a.chg[v]) continue;
    const int64_t o = (int64_t)off[v], d = (int64_t)off[v + 1] - o;
    const int64_t e0 = (int64_t)c * a.chunk;
    const int64_t n = (d - e0 < a.chunk) ? d - e0 : a.chunk;
    for (int64_t e = threadIdx.x; e < n; e += blockDim.x) a.F[a.tgt[o + e0 + e]] = 1;
  }
}

hipError_t launch_push_hubs(bool off64, const HubArgs& a, int grid, hipStream_t s) {
  if (off64)
    hipLaunchKernelGGL(k_push_hubs<int64_t>, dim3(grid), dim3(kBT), 0, s, a);
  else
    hipLaunchKernelGGL(k_push_hubs<int32_t>, dim3(grid), dim3(kBT), 0, s, a);
  return hipGetLastError();
}

// pull: non-hub rows with one lane, then 16 lanes per vertex; hub rows with one
// workgroup per hub.
namespace {
// whether x holds on any lane of the 16-lane group g = lane / 16
__device__ __forceinline__ bool group_any16(bool x, int g) {
  return ((uint32_t)(__ballot(x) >> (16 * g)) & 0xFFFFu) != 0u;
}
}  // namespace

// After the sweep, over the change bytes: in deterministic mode (APPLY) the
// changed vertices' labels go from Cn to C -- the sweeps wrote Cn for them
// only --, and when the flags are pulled the bytes are packed into bits (bit v
// % 32 of word v / 32; pack, 2 ahead of k_flags' decision): the pull kernels' reads land at data-dependent
// vertices, and the bitmap (n / 8 bytes) keeps far more of them in one cache
// line than the bytes do.  One vertex per lane, so that the copies of a wave
// fall on consecutive addresses.  It is bound by the bytes read and the
// labels moved: 157 us on the 8192 x 8192 lattice where nearly all change,
// against 176 us for a copy of every listed vertex's label and 18 us for the
// packing.
template <bool APPLY>
__global__ __launch_bounds__(kBT) void k_publish(const DevStats* st, const uint8_t* chg, int64_t n,
                                                 const int32_t* Cn, int32_t* C, uint32_t* bits,
                                                 int pack) {
  if (st->stop) return;
  const bool packed = pack == 2 || (pack && st->pull_mode == 1u);
  if (!APPLY && !packed) return;
  constexpr int U = 8;  // 64-vertex groups per wave step, all in flight
  const int lane = threadIdx.x & 63;
  const int64_t wave = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  const int64_t nw = (n + 31) / 32;
  for (int64_t base = wave * 64 * U; base < n; base += nwaves * 64 * U) {
    uint8_t c[U];
    int32_t l[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t v = base + u * 64 + lane;
      c[u] = v < n ? chg[v] : (uint8_t)0;
    }
    if constexpr (APPLY) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c[u]) l[u] = Cn[base + u * 64 + lane];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c[u]) C[base + u * 64 + lane] = l[u];
    }
    if (packed) {
      // lane i holds word i of the step's 2 U
      uint32_t word = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const unsigned long long m = __ballot(c[u] != 0);
        if ((lane >> 1) == u) word = (lane & 1) ? (uint32_t)(m >> 32) : (uint32_t)m;
      }
      const int64_t w = base / 32 + lane;
      if (lane < 2 * U && w < nw) bits[w] = word;
    }
  }
}

hipError_t launch_publish(const DevStats* st, const uint8_t* chg, int64_t n, const int32_t* Cn,
                          int32_t* C, uint32_t* bits, bool apply, int pack, hipStream_t s) {
  const int g = grid_for(n, kBT * 8, 2048);
  if (apply)
    hipLaunchKernelGGL(k_publish<true>, dim3(g), dim3(kBT), 0, s, st, chg, n, Cn, C, bits,
                       pack);
  else
    hipLaunchKernelGGL(k_publish<false>, dim3(g), dim3(kBT), 0, s, st, chg, n, Cn, C, bits,
                       pack);
  return hipGetLastError();
}

__device__ __forceinline__ bool chg_bit(const uint32_t* bits, int32_t j) {
  return (bits[j >> 5] >> (j & 31)) & 1u;
}

// tgt[p .. p + 3]: one 16-byte load, or entry by entry where the row is one of
// the array's first few and p is negative (entries before `lo`, the row's
// start, are read as -1).  In a row of fewer entries the load takes in the end
// of the row before; those entries are not looked at.
__device__ __forceinline__ int4 load_four(const int32_t* tgt, int64_t p, int64_t lo) {
  int4 j;
  if (p >= 0) {
    __builtin_memcpy(&j, tgt + p, sizeof(j));
  } else {
    j.x = -1;
    j.y = p + 1 >= lo ? tgt[p + 1] : -1;
    j.z = p + 2 >= lo ? tgt[p + 2] : -1;
    j.w = p + 3 >= lo ? tgt[p + 3] : -1;
  }
  return j;
}

constexpr int kPullSmallWords = 8192, kPullBigWords = 38912;
// Vertices per wave and step.  A small graph has waves to spare: 16, so that
// the rows left unresolved take one round of the wave (10 000 vertices, longest
// pull of a run: 13.5 -> 7.8 us; 20 011: 20.5 -> 17.3).
template <int WORDS>
__host__ __device__ constexpr int pull_rows(int64_t n) {
  return WORDS == kPullSmallWords && n <= 65536 ? 16 : 64;
}

// WORDS > 0: the bits are copied to LDS first (n <= 32 WORDS), where a lookup
// costs a few cycles a wave instead of the address unit's 64 (LFR, 1 M
// vertices, 20 M entries: 87 -> 61 us in the longest pull of a run).  From
// memory it is bound by the latency of offset, entries and bits one after the
// other, so by the waves in flight: eight per SIMD, the whole grid resident at
// once (8192 x 8192 lattice: 0.41 ms per launch; with the last four entries
// read one by one 0.43, with two vertices per lane and six waves 0.48).
//
// DECIDE (k_flags): graphs of up to 1.2 M vertices without hubs take the
// decision, the pushing and the pulling in one launch, each workgroup adding
// up the counters' copies for itself (k_iter_end folds them): a launch that
// returns at once still takes 4.6 us of an iteration of a captured run.  With
// the next iteration begun by k_iter_end, three launches fewer an iteration: a
// 10 000-vertex run 0.38 -> 0.33 ms, LFR 1M 1.60 -> 1.57 ms.
struct PushArgs {
  ListPtrs lists;
  const uint8_t* chg;
  FlagRule rule;
};
template <typename OffT, int BT, int WORDS, bool DECIDE>
__global__ __launch_bounds__(BT, WORDS ? 1 : 8) void k_pull_flags(const OffT* off, const int32_t* tgt,
                                                   int64_t n, const uint8_t* cls,
                                                   const uint32_t* bits, uint8_t* F,
                                                   DevStats* st, PushArgs pa) {
  if (st->stop || (!DECIDE && st->pull_mode != 1u)) return;
  __shared__ __align__(16) uint32_t copy[WORDS + 1];
  if constexpr (DECIDE) {
    __shared__ unsigned int mode_sh;
    unsigned long long(*part)[kStatWords] =
        reinterpret_cast<unsigned long long(*)[kStatWords]>(copy);
    static_assert(WORDS * 4 >= BT / 64 * kStatWords * 8, "the copies' sums fit the bits' LDS");
    const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
    const unsigned long long(*slot)[kStatWords] = reinterpret_cast<const DevState*>(st)->slot;
    unsigned long long x = 0;
    for (int q = wv; q < kStatSlots; q += BT / 64) x += slot[q][l];
    part[wv][l] = x;
    __syncthreads();
    if (wv == 0) {
      for (int q = 1; q < BT / 64; ++q) x += part[q][l];
      const bool cls_word = l < 3 * kNumClasses;
      const unsigned long long fw = wave_sum_u64(cls_word && l % 3 == kStatFlagw ? x : 0ull);
      const unsigned long long ch = wave_sum_u64(cls_word && l % 3 == kStatChanged ? x : 0ull);
      const unsigned long long sk = wave_sum_u64(l == kStatSkipped ? x : 0ull);
      if (l == 0) mode_sh = flag_decision(st, pa.rule, fw, ch, sk);
    }
    __syncthreads();
    const unsigned int mode = mode_sh;
    if (mode == 2u) return;
    if (mode == 0u) {
      push_lists(off, tgt, pa.lists, pa.chg, F, st);
      return;
    }
  }
  // the word after the copied ones stands for the vertices from n on, which have
  // no entries and never change (the internal order's last; one is a target
  // only if the CSR is not symmetric)
  [[maybe_unused]] const int last = (int)((n + 31) / 32);
  if constexpr (WORDS > 0) {
    for (int w = threadIdx.x; w < last; w += BT) copy[w] = bits[w];
    if (threadIdx.x == 0) copy[last] = 0u;
    __syncthreads();
  }
  auto changed = [&](int32_t j) {
    if constexpr (WORDS > 0) return ((copy[min(j >> 5, last)] >> (j & 31)) & 1u) != 0u;
    else return chg_bit(bits, j);
  };
  const int lane = threadIdx.x & 63;
  const int g = lane >> 4, k = lane & 15;
  const int64_t wave = (blockIdx.x * (int64_t)BT + threadIdx.x) >> 6;
  const int64_t nwaves = ((int64_t)gridDim.x * BT) >> 6;
  unsigned long long scanned = 0;
  constexpr int kFirst = 4;  // entries a lane checks for its own vertex
  constexpr int kRows = WORDS > 0 ? 4 : 2;  // unresolved rows per lane group and round
  // one vertex per lane for its last kFirst entries (most rows find a
  // changed neighbour there); the rows left unresolved are then scanned by 16
  // lanes each, kRows x 4 rows at a time with their loads in flight together:
  // 16 entries, then 64 a step.  Rows are read from their end: with the
  // internal order's rows sorted by target, the last entries are the
  // lowest-degree neighbours, which are the ones that still change late in a
  // run (from the start: 0.58 -> 0.89 ms per launch on R-MAT 26)
  const int per = pull_rows<WORDS>(n);
  for (int64_t base = wave * per; base < n; base += nwaves * per) {
    const int64_t v = base + lane;
    OffT o = 0;
    int32_t d = 0;  // a hub's row is scanned by k_pull_hubs
    if (lane < per && v < n && cls[v] != kClassHub) {
      o = off[v];
      d = (int32_t)(off[v + 1] - o);
    }
    int4 j = make_int4(0, 0, 0, 0);
    if (d > 0) j = load_four(tgt, (int64_t)o + d - kFirst, (int64_t)o);
    const int32_t e[kFirst] = {j.w, j.z, j.y, j.x};
    bool found = false;
#pragma unroll
    for (int u = 0; u < kFirst; ++u) {
      if (u < d && !found) {
        ++scanned;
        found = changed(e[u]);
      }
    }
    if (found) F[v] = 1;
    unsigned long long pend = __ballot(!found && d > kFirst);
    while (pend) {
      // the next kRows x 4 pending rows, dealt out over the lane groups
      int src[kRows];
#pragma unroll
      for (int r = 0; r < kRows; ++r) src[r] = -1;
#pragma unroll
      for (int q = 0; q < kRows * 4; ++q) {
        const int sq = pend ? __ffsll((long long)pend) - 1 : -1;
        pend &= pend - 1;
        if (g == (q & 3)) src[q >> 2] = sq;
      }
      OffT po[kRows];
      int32_t left[kRows];  // entries of the row not scanned; 0: row done
      bool hit[kRows];
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        const int sl = src[r] < 0 ? 0 : src[r];
        po[r] = __shfl(o, sl);
        const int32_t pd = __shfl(d, sl);  // by all lanes, as it reads any
        left[r] = src[r] < 0 ? 0 : pd - kFirst;
      }
      int32_t j[kRows];
#pragma unroll
      for (int r = 0; r < kRows; ++r)
        j[r] = k < left[r] ? tgt[(int64_t)po[r] + left[r] - 1 - k] : -1;
      bool more = false;
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        bool h = false;
        if (j[r] >= 0) {
          h = changed(j[r]);
          ++scanned;
        }
        hit[r] = group_any16(h, g);
        left[r] = hit[r] || left[r] <= 16 ? 0 : left[r] - 16;
        more |= left[r] != 0;
      }
      while (__any(more)) {
        int4 f[kRows];
#pragma unroll
        for (int r = 0; r < kRows; ++r)
          if (4 * k < left[r])
            f[r] = load_four(tgt, (int64_t)po[r] + left[r] - 4 * k - 4, (int64_t)po[r]);
        more = false;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
          bool h = false;
          const int32_t in = left[r] - 4 * k;  // entries of the row in f[r]
          if (in > 0) {
            h = changed(f[r].w);
            if (in > 1) h |= changed(f[r].z);
            if (in > 2) h |= changed(f[r].y);
            if (in > 3) h |= changed(f[r].x);
            scanned += in < 4 ? in : 4;
          }
          h = group_any16(h, g);
          hit[r] |= h;
          left[r] = h || left[r] <= 64 ? 0 : left[r] - 64;
          more |= left[r] != 0;
        }
      }
#pragma unroll
      for (int r = 0; r < kRows; ++r)
        if (hit[r] && k == 0) F[base + src[r]] = 1;
    }
  }
  // one atomic per workgroup
  __shared__ unsigned long long ws[BT / 64];
  for (int ofs = 32; ofs > 0; ofs >>= 1) scanned += __shfl_xor(scanned, ofs);
  if (lane == 0) ws[threadIdx.x >> 6] = scanned;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int q = 0; q < BT / 64; ++q) t += ws[q];
    if (t) atomicAdd(&stat_slot(st)[kStatPullScanned], t);
  }
}

template <typename OffT>
__global__ __launch_bounds__(kBT) void k_pull_hubs(const OffT* off, const int32_t* tgt,
                                                   const int32_t* hub_vid, int32_t H,
                                                   const uint32_t* chg, uint8_t* F,
                                                   DevStats* st) {
  constexpr int U = 8;  // entries per thread and step, all in flight at once
  __shared__ unsigned long long ws[kBT / 64];
  if (st->stop || st->pull_mode != 1u) return;
  unsigned long long scanned = 0;
  for (int32_t h = blockIdx.x; h < H; h += gridDim.x) {
    const int32_t v = hub_vid[h];
    const int64_t o = (int64_t)off[v];
    const int64_t d = (int64_t)off[v + 1] - o;
    bool found = false;
    for (int64_t t = 0; t < d && !found; t += (int64_t)kBT * U) {
      int32_t j[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t e = t + (int64_t)u * kBT + threadIdx.x;
        j[u] = e < d ? tgt[o + e] : -1;
      }
      int hit = 0;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (j[u] >= 0) {
          ++scanned;
          hit |= chg_bit(chg, j[u]) ? 1 : 0;
        }
      found = __syncthreads_or(hit) != 0;  // uniform over the workgroup
    }
    if (threadIdx.x == 0 && found) F[v] = 1;
  }
  // one atomic per workgroup
  for (int ofs = 32; ofs > 0; ofs >>= 1) scanned += __shfl_xor(scanned, ofs);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = scanned;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int q = 0; q < kBT / 64; ++q) t += ws[q];
    if (t) atomicAdd(&stat_slot(st)[kStatPullScanned], t);
  }
}

// Where the bits go: graphs of up to 2^18 vertices keep them in 32 KB of LDS,
// four workgroups and more to a CU; of up to 1.2 M in 152 KB, one workgroup
// of 16 waves to a CU; larger graphs read them from memory.
template <typename OffT, bool DECIDE>
static void pull_flags(const void* off, const int32_t* tgt, int64_t n, const uint8_t* cls,
                       const uint32_t* bits, uint8_t* F, DevStats* st, const PushArgs& pa,
                       hipStream_t s) {
  const OffT* o = (const OffT*)off;
  const int64_t words = (n + 31) / 32;
  if (words <= kPullSmallWords)
    hipLaunchKernelGGL((k_pull_flags<OffT, 256, kPullSmallWords, DECIDE>),
                       dim3(grid_for(n, 4 * pull_rows<kPullSmallWords>(n), 1024)), dim3(256), 0, s, o,
                       tgt, n, cls, bits, F, st, pa);
  else if (words <= kPullBigWords)
    hipLaunchKernelGGL((k_pull_flags<OffT, 1024, kPullBigWords, DECIDE>),
                       dim3(grid_for(n, 1024, 256)), dim3(1024), 0, s, o, tgt, n, cls, bits, F, st,
                       pa);
  else if constexpr (!DECIDE)
    hipLaunchKernelGGL((k_pull_flags<OffT, 256, 0, false>), dim3(grid_for(n, 256, 2048)),
                       dim3(256), 0, s, o, tgt, n, cls, bits, F, st, pa);
}

hipError_t launch_pull_flags(bool off64, const void* off, const int32_t* tgt, int64_t n,
                             const uint8_t* cls, const uint32_t* chg_bits, uint8_t* F,
                             DevStats* st, hipStream_t s) {
  if (off64) pull_flags<int64_t, false>(off, tgt, n, cls, chg_bits, F, st, PushArgs{}, s);
  else pull_flags<int32_t, false>(off, tgt, n, cls, chg_bits, F, st, PushArgs{}, s);
  return hipGetLastError();
}

bool flags_in_one_launch(int64_t n) { return (n + 31) / 32 <= kPullBigWords; }

hipError_t launch_flags(bool off64, const void* off, const int32_t* tgt, int64_t n,
                        const uint8_t* cls, const uint32_t* chg_bits, uint8_t* F, DevStats* st,
                        int32_t* const* lists, const uint8_t* chg, const FlagRule& rule,
                        hipStream_t s) {
  PushArgs pa;
  for (int q = 0; q < kNumClasses; ++q) pa.lists.p[q] = lists[q];
  pa.chg = chg;
  pa.rule = rule;
  if (off64) pull_flags<int64_t, true>(off, tgt, n, cls, chg_bits, F, st, pa, s);
  else pull_flags<int32_t, true>(off, tgt, n, cls, chg_bits, F, st, pa, s);
  return hipGetLastError();
}

// chg_bits: the packed change bits that launch_publish wrote just before
hipError_t launch_pull_hubs(bool off64, const void* off, const int32_t* tgt,
                            const int32_t* hub_vid, int32_t H, const uint32_t* chg,
                            uint8_t* F, DevStats* st, hipStream_t s) {
  const int g = H < 2048 ? H : 2048;
  if (off64)
    hipLaunchKernelGGL(k_pull_hubs<int64_t>, dim3(g), dim3(kBT), 0, s,
                       (const int64_t*)off, tgt, hub_vid, H, chg, F, st);
  else
    hipLaunchKernelGGL(k_pull_hubs<int32_t>, dim3(g), dim3(kBT), 0, s,
                       (const int32_t*)off, tgt, hub_vid, H, chg, F, st);
  return hipGetLastError();
}

// ---- modularity, Eq. 1 ------------------------------------------------------
// Community form: Q = sigma / 2m - sum_c (Sigma_c / 2m)^2, with Sigma_c the sum
// of the weighted degrees K_v of its vertices.  Edge-parallel: each wave owns a
// contiguous range of CSR entries and takes 256 per step, four consecutive
// ones a lane.  A step inside one row needs only that row's label.  Otherwise
// the rows that start in the step write their labels to LDS at the position
// of their first entry, and each entry takes the label at the last position
// at or before its own (a max scan).  An entry adds its weight to sigma when
// both end labels agree; a row adds K_v to its label once: the row length
// for unit weights, else a segmented sum over the lanes.  The K_v are
// gathered per workgroup in an LDS table of labels (direct-mapped; a row
// whose slot is taken adds to memory), so that a label shared by many rows
// costs one atomic a workgroup on its one address.  It is bound by the lines
// that the targets' labels fetch.  The waves' ranges are short, so that the
// waves at work together read neighbouring rows, whose targets overlap: with
// 8192 ranges instead of up to 65536 4.04 instead of 3.08 ms on R-MAT scale
// 24 (64 entries a step, a search and a segmented sum per entry: 3.78).  On
// 400 000 entries 100 -> 19 us.
namespace {

__device__ __forceinline__ double wave_sum_f64(double x) {
  for (int ofs = 32; ofs > 0; ofs >>= 1) x += __shfl_xor(x, ofs);
  return x;
}

__device__ __forceinline__ double block_sum_f64(double x, double* sh) {
  for (int ofs = 32; ofs > 0; ofs >>= 1) x += __shfl_xor(x, ofs);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = x;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int q = 0; q < (int)(blockDim.x >> 6); ++q) t += sh[q];
  __syncthreads();
  return t;
}

// x's maximum over the lanes up to and including this one.
__device__ __forceinline__ int wave_scan_max(int x) {
#pragma unroll
  for (int ofs = 1; ofs < 64; ofs <<= 1) {
    const int y = __shfl_up(x, ofs);
    if ((int)(threadIdx.x & 63) >= ofs) x = x > y ? x : y;
  }
  return x;
}

}  // namespace

constexpr int kModCache = 1024;  // label slots per workgroup
constexpr int kModStep = 256;    // entries per wave and step
constexpr int kModWaves = 65536;  // ranges at most

template <typename OffT, bool UNIT>
__global__ __launch_bounds__(kBT) void k_mod_edges(const OffT* off, const int32_t* tgt,
                                                   const float* w, int64_t n, int64_t m, int64_t S,
                                                   const int32_t* C, double* sig, DevStats* st) {
  __shared__ double sh[kBT / 64];
  __shared__ int32_t ckey[kModCache];
  __shared__ double cval[kModCache];
  __shared__ __align__(16) int32_t start_all[kBT / 64][kModStep];
  if (st->error & 4u) return;  // a label out of range (k_check_labels)
  for (int x = threadIdx.x; x < kModCache; x += kBT) {
    ckey[x] = -1;
    cval[x] = 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  int32_t* start = start_all[threadIdx.x >> 6];
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t e_begin = wave * S;
  const int64_t e_end = (e_begin + S < m) ? e_begin + S : m;
  double sigma = 0.0, two_m = 0.0;
  uint32_t same = 0;  // unit weights: sigma in whole numbers
  auto add_degree = [&](int32_t c, double K) {
    const int slot = (int)(((uint32_t)c * 0x9E3779B1u) >> 22);
    int k = __hip_atomic_load(&ckey[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (k == -1) {
      int expected = -1;
      __hip_atomic_compare_exchange_strong(&ckey[slot], &expected, c, __ATOMIC_RELAXED,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      k = expected == -1 ? c : expected;
    }
    if (k == c)
      __hip_atomic_fetch_add(&cval[slot], K, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else
      unsafeAtomicAdd(&sig[c], K);  // slot held by another label
  };
  if (e_begin < e_end) {  // uniform over the wave
    // row of e_begin: the largest i with off[i] <= e_begin, 64 probes a round
    int64_t r0 = 0;
    for (int64_t len = n; len > 1;) {
      const int64_t step = (len + 63) / 64;
      const int64_t at = lane * step;
      const bool le = at < len && (int64_t)off[r0 + at] <= e_begin;
      const int64_t below = (int64_t)__popcll(__ballot(le)) - 1;  // >= 0: off[r0] <= e_begin
      r0 += below * step;
      len = len - below * step < step ? len - below * step : step;
    }
    int32_t cl = C[r0];
    if constexpr (UNIT) {
      if (lane == 0 && (int64_t)off[r0] == e_begin)
        add_degree(cl, (double)((int64_t)off[r0 + 1] - e_begin));
    }
    double carry = 0.0, hold = 0.0;  // weights: the current row's sum so far
    auto load_targets = [&](int64_t base) {
      const int64_t e = base + 4 * lane;
      int4 t = make_int4(0, 0, 0, 0);
      if (e + 4 <= e_end) {
        __builtin_memcpy(&t, tgt + e, sizeof(t));
      } else {
        if (e < e_end) t.x = tgt[e];
        if (e + 1 < e_end) t.y = tgt[e + 1];
        if (e + 2 < e_end) t.z = tgt[e + 2];
      }
      return t;
    };
    int4 nxt = load_targets(e_begin);
    for (int64_t base = e_begin; base < e_end; base += kModStep) {
      const int4 t = nxt;
      const int64_t e = base + 4 * lane;
      const int valid = e >= e_end ? 0 : (e_end - e < 4 ? (int)(e_end - e) : 4);
      const int64_t lim = base + kModStep < e_end ? base + kModStep : e_end;
      int32_t lj[4];
      lj[0] = C[t.x];
      lj[1] = C[t.y];
      lj[2] = C[t.z];
      lj[3] = C[t.w];
      float we[4];
      if constexpr (!UNIT) {
#pragma unroll
        for (int i = 0; i < 4; ++i) we[i] = i < valid ? w[e + i] : 0.0f;
      }
      if (base + kModStep < e_end) nxt = load_targets(base + kModStep);
      int32_t la[4];
      if ((int64_t)off[r0 + 1] >= lim) {
        la[0] = la[1] = la[2] = la[3] = cl;
        if constexpr (!UNIT) hold += ((double)we[0] + we[1]) + ((double)we[2] + we[3]);
      } else {
        *reinterpret_cast<int4*>(start + 4 * lane) = make_int4(-1, -1, -1, -1);
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        int64_t rn = r0;
        for (int64_t rb = r0 + 1;; rb += 64) {
          const int64_t i = rb + lane;
          const int64_t v = i < n ? (int64_t)off[i] : INT64_MAX;
          const bool in = v < lim;
          bool starts = false;
          if (in) {
            const int64_t v1 = (int64_t)off[i + 1];
            if (v1 > v) {
              starts = true;
              const int32_t c = C[i];
              start[v - base] = c;
              if constexpr (UNIT) add_degree(c, (double)(v1 - v));
            }
          }
          const unsigned long long b = __ballot(starts);
          if (b) rn = rb + 63 - __clzll((long long)b);
          if (!__all(in)) break;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        const int4 l4 = *reinterpret_cast<const int4*>(start + 4 * lane);
        const int32_t l[4] = {l4.x, l4.y, l4.z, l4.w};
        int p = -1;  // the lane's last row start
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (l[i] >= 0) p = 4 * lane + i;
        int before = __shfl_up(wave_scan_max(p), 1);
        if (lane == 0) before = -1;
        const int32_t prev = before >= 0 ? start[before] : cl;
        la[0] = l[0] >= 0 ? l[0] : prev;
#pragma unroll
        for (int i = 1; i < 4; ++i) la[i] = l[i] >= 0 ? l[i] : la[i - 1];
        if constexpr (!UNIT) {
          carry += wave_sum_f64(hold);
          hold = 0.0;
          // the sum of the row open at the lane's end, over the lanes
          double open = 0.0;
#pragma unroll
          for (int i = 0; i < 4; ++i) open = (l[i] >= 0 ? 0.0 : open) + we[i];
          if (lane == 0 && p < 0) open += carry;
          int f = p >= 0 ? 1 : 0;
#pragma unroll
          for (int ofs = 1; ofs < 64; ofs <<= 1) {
            const double ys = __shfl_up(open, ofs);
            const int yf = __shfl_up(f, ofs);
            if (lane >= ofs && !f) {
              open += ys;
              f |= yf;
            }
          }
          double run = __shfl_up(open, 1);
          if (lane == 0) run = carry;
          // the rows that end in the lane
          int32_t c = prev;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (l[i] >= 0) {
              if (run != 0.0) add_degree(c, run);
              run = 0.0;
              c = l[i];
            }
            run += we[i];
          }
          carry = __shfl(open, 63);
        }
        cl = __builtin_amdgcn_readlane(la[3], 63);
        r0 = rn;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool eq = i < valid && lj[i] == la[i];
        if constexpr (UNIT) {
          same += eq ? 1u : 0u;
        } else {
          sigma += eq ? (double)we[i] : 0.0;
          two_m += (double)we[i];
        }
      }
    }
    if constexpr (!UNIT) {
      carry += wave_sum_f64(hold);
      if (lane == 0 && carry != 0.0) add_degree(cl, carry);
    }
  }
  if constexpr (UNIT) sigma = (double)same;
  const double s1 = block_sum_f64(sigma, sh);
  const double s2 = UNIT ? 0.0 : block_sum_f64(two_m, sh);
  __syncthreads();
  for (int x = threadIdx.x; x < kModCache; x += kBT)
    if (ckey[x] >= 0 && cval[x] != 0.0) unsafeAtomicAdd(&sig[ckey[x]], cval[x]);
  if (threadIdx.x == 0) {
    double* slot = reinterpret_cast<double*>(stat_slot(st)) + kStatMod;
    unsafeAtomicAdd(&slot[0], s1);
    if (UNIT && blockIdx.x == 0) unsafeAtomicAdd(&slot[1], (double)m);
    if (!UNIT) unsafeAtomicAdd(&slot[1], s2);
  }
}

__global__ __launch_bounds__(kBT) void k_mod_sq(const double* sig, int64_t n, DevStats* st) {
  __shared__ double sh[kBT / 64];
  double s = 0.0;
  for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
       c += (int64_t)gridDim.x * blockDim.x)
    s += sig[c] * sig[c];
  const double t = block_sum_f64(s, sh);
  if (threadIdx.x == 0)
    unsafeAtomicAdd(reinterpret_cast<double*>(stat_slot(st)) + kStatMod + 2, t);
}

// The copies of the three sums added to acc and cleared; one wave.
__global__ void k_mod_fold(DevStats* st, double* acc) {
  const int lane = threadIdx.x & 63;
  for (int k = 0; k < 3; ++k) {
    double x = 0.0;
    if (lane < kStatSlots) {
      double* p = reinterpret_cast<double*>(reinterpret_cast<DevState*>(st)->slot[lane]) + kStatMod + k;
      x = *p;
      *p = 0.0;
    }
    const double t = wave_sum_f64(x);
    if (lane == 0) acc[k] = t;
  }
}

// ---- modularity scratch for callers that cannot allocate ----------------------
// Sigma_c (one double per vertex) of lpa_modularity_noalloc lives in this
// file-scope array: one copy per GPU, 32 MiB, held until the process ends.  Host code never takes the array's
// name as an address (it is a host-side stand-in); the device address comes
// from hipGetSymbolAddress, once per device, with that device current.
static __device__ __align__(256) double scratch[kModScratchVertices];

hipError_t modularity_scratch(double** sig) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static double* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = static_cast<double*>(p);
  }
  *sig = addr[dev];
  return hipSuccess;
}

hipError_t launch_modularity(bool off64, const void* off, const int32_t* tgt, const float* w,
                             int64_t n, int64_t m, const int32_t* C, double* sig,
                             double* acc, DevStats* st, hipStream_t s) {
  hipError_t e = launch_fill_f64(sig, 0.0, n, s);
  if (e != hipSuccess) return e;
  if (m > 0) {
    const int64_t S = std::max<int64_t>((m + kModWaves - 1) / kModWaves + kModStep - 1, kModStep) /
                      kModStep * kModStep;
    const int g = (int)(((m + S - 1) / S + kBT / 64 - 1) / (kBT / 64));
    auto go = [&](auto kernel, auto* o) {
      hipLaunchKernelGGL(kernel, dim3(g), dim3(kBT), 0, s, o, tgt, w, n, m, S, C, sig, st);
    };
    if (off64 && w) go(k_mod_edges<int64_t, false>, (const int64_t*)off);
    else if (off64) go(k_mod_edges<int64_t, true>, (const int64_t*)off);
    else if (w) go(k_mod_edges<int32_t, false>, (const int32_t*)off);
    else go(k_mod_edges<int32_t, true>, (const int32_t*)off);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_mod_sq, dim3(grid_for(n, kBT, 2048)), dim3(kBT), 0, s, sig, n, st);
  hipLaunchKernelGGL(k_mod_fold, dim3(1), dim3(64), 0, s, st, acc);
  return hipGetLastError();
}

}  // namespace lpa
