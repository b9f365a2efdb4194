// queue.hip -- batched label propagation (Algorithm 1 run on many independent
// graphs packed into one CSR) as a persistent work queue.
//
// An item is a chunk of up to 2^chunk_log2 consecutive vertices of one graph.
// Per iteration:
//   k_queue_iter_begin  resets the iteration's counters (one thread);
//   k_queue_sweep       a resident grid (every workgroup the GPU holds at
//                       once) pops items from the queue until it is drained.
//                       For each item the workgroup reads and clears the
//                       chunk's flags, sorts the flagged vertices by row
//                       length into LDS lists and processes them: rows of
//                       up to group_max entries with 16 lanes each (16 rows
//                       at a time), longer ones (up to 512 entries) with the
//                       whole workgroup and a 1023-slot table in LDS.  The
//                       first sweep
//                       from the ids over strictly increasing rows needs no
//                       table (each label occurs once per row).
//                       Each vertex takes the label of maximum summed weight
//                       (Eq. 3; smallest label on ties), moves under the
//                       Pick-Less rule (Sec. 4.1) and, when it moves, flags
//                       every neighbour for the next iteration (Sec. 4 item
//                       4);
//   k_queue_step        one workgroup per graph applies Algorithm 1's stop
//                       test with the graph's own vertex count and queues
//                       the graph's chunks that hold flags or changes for the
//                       next iteration;
//   k_iter_end          (graph.hip) records the iteration and ends the run
//                       when every graph has stopped.
// The iteration boundary is the only barrier: a graph's next iteration reads
// what the previous kernels wrote, and graphs never share a vertex, so no
// ordering is needed inside the sweep beyond the relaxed atomics of the
// queue counters.  The queue has two halves by iteration parity, and each
// half one part per XCD: all chunks of graph g go to part g mod 8, so a
// graph's labels, flags and rows are cached in the L2 of the XCD that works
// on it.  A workgroup pops from its own XCD's part first and takes items
// from the other parts once that is drained.
//
// Deterministic mode keeps two label arrays by iteration parity.  A visited
// chunk writes the next label of every vertex (processed ones their result,
// the others a copy); a chunk in which a label changed is visited again in
// the next iteration, so that the copy catches up.  A chunk left unvisited
// had no change in the previous iteration and therefore holds the same
// labels in both arrays.  A graph's final labels (and its flags for a next
// iteration) are in the arrays of its iteration-count parity;
// k_queue_finish moves the odd ones.
#include <type_traits>

#include "lpa_device.h"

namespace lpa {

namespace {

constexpr int kQBT = 256;                 // threads per sweep workgroup
constexpr int kQGroups = kQBT / 16;       // 16-lane groups per workgroup
constexpr int kQWaves = kQBT / 64;
constexpr int kQPool = kQGroups * kMatchSlots;  // LDS table slots per workgroup
constexpr uint32_t kNoItem = 0xFFFFFFFFu;
static_assert(2 * kQueueMaxDegree - 1 <= kQPool, "the pool holds a 512-entry row's table");

__device__ __forceinline__ unsigned int* qhead(unsigned int* ctr, int par, uint32_t x) {
  return ctr + (size_t)((par * kXcds + (int)x) * 2) * kQueueCtrStride;
}
__device__ __forceinline__ unsigned int* qtail(unsigned int* ctr, int par, uint32_t x) {
  return ctr + (size_t)((par * kXcds + (int)x) * 2 + 1) * kQueueCtrStride;
}

// Next item of queue half par for a workgroup, trying part `from` first (its
// own XCD's, later the part it last took an item from), then the others;
// kNoItem once every part is drained.  The tails were written by earlier
// kernels and do not change during the sweep; heads may run past them.
__device__ uint32_t queue_pop(const QueueArgs& q, int par, uint32_t& from) {
  for (int k = 0; k < kXcds; ++k) {
    const uint32_t p = (from + (uint32_t)k) & (uint32_t)(kXcds - 1);
    const unsigned int tail = *qtail(q.qctr, par, p);
    unsigned int* head = qhead(q.qctr, par, p);
    if (__hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= tail) continue;
    const unsigned int pos = atomicAdd(head, 1u);
    if (pos < tail) {
      from = p;
      return q.items[(size_t)par * (size_t)q.nchunks + (size_t)q.qbase[p] + pos];
    }
  }
  return kNoItem;
}

// Words of the bit flags that hold the vertices gv0 .. gv1 - 1.
__device__ __forceinline__ int64_t graph_bits(int64_t gv0, int64_t gv1) {
  return ((gv1 - 1) >> 5) - (gv0 >> 5) + 1;
}

// Bits of flag word x that stand for the vertices v0 .. v1 - 1.
__device__ __forceinline__ uint32_t word_mask(int64_t x, int64_t v0, int64_t v1) {
  const int64_t b0 = x << 5;
  const uint32_t lo = v0 > b0 ? ~0u << (v0 - b0) : ~0u;
  const uint32_t hi = v1 < b0 + 32 ? ~(~0u << (v1 - b0)) : ~0u;
  return lo & hi;
}

}  // namespace

// Dynamic LDS of k_queue_sweep, per vertex of a chunk: its row's header
// (offset from the chunk's first entry << 10 | length), its label, two list
// words.
constexpr size_t kQChunkBytes = 4 + 4 + 2 + 2;
constexpr uint32_t kQMaxRel = 1u << 22;   // header offsets are below this
static_assert((int64_t)kQueueMaxDegree << kQueueMaxChunkLog2 <= (int64_t)kQMaxRel, "header");
static_assert(kQueueMaxDegree < 1024, "header");

// What bounds it: the labels of a graph lie in its XCD's L2, so the sweep is
// bound by instruction issue and by the address unit, which spends up to a
// cycle per lane on a load or store of scattered addresses.  The rows'
// offsets and own labels are therefore read once per chunk, coalesced, into
// LDS, with the flags; a wave takes the headers of up to 64 listed rows from
// there, one per lane, and hands them to the 16 lanes of each row by DPP, so
// that a step loads only targets and labels (the next step's targets while
// the current step's labels are in flight).  The lists are by row length, so
// that the four rows of a wave step take the same number of 16-entry
// slices: up to 16 entries (sums by rotations, where they are exact), up to 32
// and up to 64 (sums by match_sums).  New flags are gathered as bits in LDS and added to the
// graph's words once per chunk, where a byte store per entry took as many
// address cycles as reading the entry's label; a graph whose bits LDS does
// not hold keeps flag bytes (atomic bits per entry were twice as slow there).
// Measured on 2,048 planted partitions (24 M vertices, 490 M entries): a
// full table sweep 5.9 -> 1.8 ms, the first sweep 1.99 -> 1.14 ms, a
// deterministic run 35.8 -> 13.7 ms, an asynchronous one 21.4 -> 12.1 ms; of
// the gain 16 ms came with the chunk headers and match_sums, 6 ms with the
// 32-bit keys (row16_label) and one kernel per mode.
template <typename OffT, bool UNIT, bool DET>
__global__ __launch_bounds__(kQBT, 5) void k_queue_sweep(QueueArgs q) {
  // match slots of the 16 lane groups, or one 1023-slot table for the
  // workgroup path
  __shared__ uint32_t tags[kQPool];
  __shared__ float vals[kQPool];
  extern __shared__ uint32_t chunk_lds[];
  __shared__ unsigned long long wbest[kQWaves];
  __shared__ uint32_t nlist[4], ichg, item_sh;
  __shared__ int moved_sh;
  DevStats* st = q.st;
  if (st->stop) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, k = tid & 15;
  const int l = st->iter;
  const int par = l & 1;
  const int pl = st->pl;                       // fixed for the whole sweep
  const bool id0 = l == 0 && st->ident;        // labels are still the ids
  // first sweep from the ids over rows with strictly increasing targets:
  // every neighbour label occurs once, so a row's Eq. 3 maximum is its
  // largest (weight, smallest id) entry and no sums are needed
  const bool direct = id0 && q.strict_rows;
  int32_t* Cc = par ? q.C1 : q.C0;             // labels at the iteration start
  int32_t* Cw = par ? q.C0 : q.C1;             // deterministic: labels after it
  uint32_t* Bc = par ? q.B1 : q.B0;            // flags of this iteration: bits
  uint32_t* Bn = par ? q.B0 : q.B1;            // (and of the next one), or
  uint8_t* Fc = par ? q.F1 : q.F0;             // bytes for the graphs whose
  uint8_t* Fn = par ? q.F0 : q.F1;             // bits LDS does not hold
  // a neighbour's label.  Asynchronous mode reads past the CU's cache: a graph
  // whose labels fit there would otherwise not see the other CUs' updates until
  // the sweep ends
  auto label = [&](uint32_t v) {
    if constexpr (DET) return (uint32_t)Cc[v];
    else return (uint32_t)__hip_atomic_load(&Cc[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  const OffT* off = reinterpret_cast<const OffT*>(q.off);
  const int64_t CH = (int64_t)1 << q.chunk_log2;
  uint32_t* hdr = chunk_lds;
  int32_t* lab_sh = reinterpret_cast<int32_t*>(chunk_lds + CH);
  uint16_t* lst_a = reinterpret_cast<uint16_t*>(chunk_lds + 2 * CH);
  uint16_t* lst_b = lst_a + CH;
  uint32_t* fb = chunk_lds + 3 * CH;           // the graph's new flags, bits
  const int64_t gm = q.group_max;
  const bool exact = UNIT || q.exact_sums != 0;
  for (int s = tid; s < kQPool; s += kQBT) vals[s] = 0.0f;
  for (int s = tid; s < q.fb_words; s += kQBT) fb[s] = 0u;
  uint32_t* tag = tags + (tid >> 4) * kMatchSlots;
  float* val = vals + (tid >> 4) * kMatchSlots;
  uint32_t from = xcc_id();
  unsigned long long my_edges = 0, my_proc = 0;
  uint32_t my_changed = 0;
  if (tid < 4) nlist[tid] = 0;
  if (tid == 0) {
    ichg = 0;
    item_sh = queue_pop(q, par, from);
  }
  __syncthreads();
  while (true) {
    const uint32_t it = item_sh;
    if (it == kNoItem) break;
    const int32_t g = q.cgraph[it];
    const int64_t gv0 = q.b.v_off[g], gv1 = q.b.v_off[g + 1];
    const int64_t c0 = q.cbase[g], c1 = q.cbase[g + 1];
    const int64_t v0 = gv0 + (((int64_t)it - c0) << q.chunk_log2);
    const int64_t v1 = (v0 + CH < gv1) ? v0 + CH : gv1;
    // the graph's words of the bit flags
    const int64_t w0 = gv0 >> 5;
    const bool bits = graph_bits(gv0, gv1) <= q.fb_words;
    const uint32_t fbw = bits ? (uint32_t)graph_bits(gv0, gv1) : 0u;
    auto flag = [&](int32_t j) {
      if (bits) {
        const uint32_t r = (uint32_t)j - (uint32_t)(w0 << 5);
        if ((r >> 5) < fbw)
          __hip_atomic_fetch_or(&fb[r >> 5], 1u << (j & 31), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_WORKGROUP);
      } else {
        Fn[j] = 1;
        const int64_t cj = c0 + (((int64_t)j - gv0) >> q.chunk_log2);
        if (cj >= c0 && cj < c1) q.cmark[cj] = 1;
      }
    };
    const int64_t e0 = (int64_t)off[v0];
    const int32_t* tgt = q.tgt + e0;
    const float* w = UNIT ? nullptr : q.w + e0;
    // 1. the chunk's labels, row headers and flags; flagged vertices into the
    //    lists by row length, each array filled from both ends
    for (int64_t base = v0; base < v1; base += kQBT) {
      const int64_t v = base + tid;
      int kind = -1;
      if (v < v1) {
        const int64_t o = (int64_t)off[v], d = (int64_t)off[v + 1] - o;
        const bool f = bits ? (Bc[v >> 5] >> (v & 31)) & 1u : Fc[v] != 0;
        if (f && !bits) Fc[v] = 0;
        lab_sh[v - v0] = Cc[v];
        if (f) {
          ++my_proc;
          // a row longer than the tables (the CSR changed after create):
          // left alone, reported through the error bits
          const bool fits = d <= kQueueMaxDegree && o - e0 < (int64_t)kQMaxRel;
          if (!fits) atomicOr(&st->error, 32u);
          if (d >= 1 && fits) {
            hdr[v - v0] = (uint32_t)(o - e0) << 10 | (uint32_t)d;
            // by slices in deterministic mode; one list in asynchronous mode,
            // whose result would change with the order (taken shortest rows
            // first, batches of 256-4,000 vertices ended 0.01-0.02 of
            // modularity lower)
            kind = d > gm ? 3 : (!DET || d > 32 ? 2 : (d > 16 ? 1 : 0));
          }
        }
      }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const unsigned long long m = __ballot(kind == b);
        if (m == 0ull) continue;
        uint32_t pos = 0;
        if (lane == 0) pos = atomicAdd(&nlist[b], (uint32_t)__popcll(m));
        pos = (uint32_t)__shfl((int)pos, 0) + lane_rank(m);
        if (kind == b) {
          uint16_t* lst = b < 2 ? lst_a : lst_b;
          lst[(b & 1) ? (uint32_t)CH - 1u - pos : pos] = (uint16_t)(v - v0);
        }
      }
    }
    __syncthreads();
    // the chunk's flags are taken (its first and last word it may share)
    if (bits)
      for (int64_t x = (v0 >> 5) + tid; x <= (v1 - 1) >> 5; x += kQBT)
        atomicAnd(&Bc[x], ~word_mask(x, v0, v1));
    uint32_t item_changed = 0;
    // 2. rows of up to group_max (<= 64) entries: 16 lanes each, U entries a
    //    lane, R rows of a lane group in flight; FIRST: the first sweep from
    //    the ids over strictly increasing rows
    const bool small = st->ident ? gv1 - gv0 <= kSmallLabels : q.b.v_off[q.b.G] <= kSmallLabels;
    const uint32_t lbase = st->ident ? (uint32_t)gv0 : 0u;  // no label lies below
    auto rows = [&](auto uc, auto rc, auto fc, uint32_t cnt, const uint16_t* lst, int dir) {
      constexpr int U = decltype(uc)::value, R = decltype(rc)::value;
      constexpr bool FIRST = decltype(fc)::value;
      // rows per lane group and batch, so that every group has some
      const uint32_t per = (cnt + kQGroups - 1) / kQGroups;
      const uint32_t T = per < 16u ? per : 16u;
      for (uint32_t b0 = 0; b0 < cnt; b0 += kQGroups * T) {
        // step t takes listed rows 16 t .. 16 t + 15 of the batch
        const uint32_t idx = b0 + (uint32_t)k * kQGroups + (uint32_t)(tid >> 4);
        const bool ok = (uint32_t)k < T && idx < cnt;
        const uint32_t li = ok ? lst[dir * (int)idx] : 0u;
        // headers being handed out: the next row's is in lane 0 of its DPP row
        uint32_t rh = ok ? hdr[li] : 0u, rl = li, rcur = ok ? (uint32_t)lab_sh[li] : 0u;
        const uint32_t dl = rh & 1023u;
        const int32_t old = (int32_t)rcur;
        uint32_t res = rcur;
        int32_t j[R][U];
        uint32_t vs[R], cur[R], d[R];
        float wt[R][U];
        auto targets = [&]() {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const uint32_t h = row_bcast<0>(rh);
            d[r] = h & 1023u;
            vs[r] = (uint32_t)v0 + row_bcast<0>(rl);
            cur[r] = row_bcast<0>(rcur);
            rh = row_left<1>(rh);
            rl = row_left<1>(rl);
            rcur = row_left<1>(rcur);
            const uint32_t last = d[r] ? d[r] - 1u : 0u;
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const uint32_t e = (uint32_t)(u * 16 + k);
              const uint32_t at = (h >> 10) + (e < last ? e : last);
              j[r][u] = __builtin_nontemporal_load(&tgt[at]);
              if constexpr (!UNIT) wt[r][u] = __builtin_nontemporal_load(&w[at]);
            }
          }
        };
        targets();
        for (uint32_t t = 0; t < T; t += R) {
          uint32_t got[R][U], ids[R][U], dc[R], vc[R], cc[R];
          float wc[R][U];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            dc[r] = d[r];
            vc[r] = vs[r];
            cc[r] = cur[r];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              ids[r][u] = (uint32_t)j[r][u];
              wc[r][u] = UNIT ? 1.0f : wt[r][u];
              if constexpr (FIRST) got[r][u] = ids[r][u];
              else got[r][u] = label(ids[r][u]);
            }
          }
          targets();
#pragma unroll
          for (int r = 0; r < R; ++r) {
            uint32_t lab[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              if constexpr (!DET && !FIRST)
                if (id0) got[r][u] = ids[r][u];
              lab[u] = (uint32_t)(u * 16 + k) < dc[r] && ids[r][u] != vc[r] ? got[r][u] : kEmpty;
            }
            typename RowSum<UNIT>::type sum[U];
            if constexpr (FIRST) {
#pragma unroll
              for (int u = 0; u < U; ++u) sum[u] = wc[r][u];
            } else if (U == 1 && exact) {
              sum[0] = rotate_sum<UNIT>(lab[0], wc[r][0]);
            } else {
              if (!exact) {
#pragma unroll
                for (int u = 0; u < U; ++u) merge_lead16(lab[u], wc[r][u]);
              }
              match_sums<U, UNIT, false>(lab, wc[r], tag, val, sum, nullptr);
            }
            const uint32_t c = row16_label<U, UNIT>(lab, sum, small, lbase, cc[r]);
            if ((uint32_t)k == t + r) res = c;
            if (moves(c, (int32_t)cc[r], pl)) {
              // in place at once, so that the steps that follow read it
              if (!DET && k == 0) Cc[vc[r]] = (int32_t)c;
#pragma unroll
              for (int u = 0; u < U; ++u)
                if ((uint32_t)(u * 16 + k) < dc[r]) flag((int32_t)ids[r][u]);
            }
          }
        }
        if (ok) {
          my_edges += dl;
          if (moves(res, old, pl)) {
            ++my_changed;
            ++item_changed;
            if (DET) lab_sh[li] = (int32_t)res;
          }
        }
      }
    };
    auto lists = [&](auto fc) {
      using std::integral_constant;
      rows(integral_constant<int, 1>{}, integral_constant<int, 2>{}, fc, nlist[0], lst_a, 1);
      rows(integral_constant<int, 2>{}, integral_constant<int, 1>{}, fc, nlist[1],
           lst_a + CH - 1, -1);
      rows(integral_constant<int, 4>{}, integral_constant<int, 1>{}, fc, nlist[2], lst_b, 1);
    };
    if (direct) lists(std::true_type{});
    else lists(std::false_type{});
    // 3. rows of group_max + 1 .. 512 entries: the whole workgroup, one row
    //    at a time, in a 1023-slot table over the match slots' LDS
    const uint32_t nl = nlist[3];
    if (nl) {
      __syncthreads();  // the groups' slots are free
      for (int s = tid; s < 2 * kQueueMaxDegree - 1; s += kQBT) tags[s] = kEmpty;
    }
    for (uint32_t idx = 0; idx < nl; ++idx) {
      __syncthreads();  // the previous row's table is clear
      const uint32_t li = lst_b[CH - 1 - idx];
      const int32_t v = (int32_t)v0 + (int32_t)li;
      const uint32_t o = hdr[li] >> 10, d = hdr[li] & 1023u;
      const int32_t cur = lab_sh[li];
      const uint32_t p1 = table_p1(d);
      unsigned long long best = 0;
      for (uint32_t b = 0; b < d; b += kQBT) {
        const uint32_t e = b + tid;
        const bool has = e < d;
        const int32_t j = has ? __builtin_nontemporal_load(&tgt[o + e]) : v;
        float wt = 0.0f;
        if constexpr (UNIT) wt = has ? 1.0f : 0.0f;
        else wt = has ? __builtin_nontemporal_load(&w[o + e]) : 0.0f;
        if (direct) {
          if (j != v) best = umax64(best, pack_key(wt, (uint32_t)j));
        } else {
          uint32_t lab = (j != v) ? (id0 ? (uint32_t)j : label((uint32_t)j)) : kEmpty;
          merge_lead(lab, wt, UNIT);
          if (lab != kEmpty) lds_accumulate(tags, vals, p1, lab, wt, q.probe);
        }
      }
      if (!direct) {
        __syncthreads();
        for (uint32_t s = (uint32_t)tid; s < p1; s += kQBT) {
          const uint32_t kk = tags[s];
          if (kk != kEmpty) {
            best = umax64(best, pack_key(vals[s], kk));
            tags[s] = kEmpty;
            vals[s] = 0.0f;
          }
        }
      }
      best = wave_max_u64(best);
      if (lane == 0) wbest[wv] = best;
      __syncthreads();
      if (tid == 0) {
        unsigned long long b = 0;
        for (int x = 0; x < kQWaves; ++x) b = umax64(b, wbest[x]);
        uint32_t cstar = 0;
        const bool moved = decide(b, cur, pl, &cstar);
        my_edges += d;
        if (moved) {
          if (DET) lab_sh[li] = (int32_t)cstar;
          else Cc[v] = (int32_t)cstar;
          ++my_changed;
          ++item_changed;
        }
        moved_sh = moved ? 1 : 0;
      }
      __syncthreads();
      if (moved_sh) {
        for (uint32_t e = tid; e < d; e += kQBT) flag(tgt[o + e]);
      }
    }
    // 4. the item's changes go to the graph's count; a chunk with a change
    //    is visited again next iteration (deterministic copy, see above)
    const uint32_t c = wave_sum_u32(item_changed);
    if (lane == 0 && c) atomicAdd(&ichg, c);
    __syncthreads();
    if (DET)
      for (int64_t v = v0 + tid; v < v1; v += kQBT) Cw[v] = lab_sh[v - v0];
    if (ichg)
      for (uint32_t x = tid; x < fbw; x += kQBT)
        if (const uint32_t b = fb[x]) {
          atomicOr(&Bn[w0 + x], b);
          fb[x] = 0u;
        }
    __syncthreads();
    if (tid < 4) nlist[tid] = 0;
    if (tid == 0) {
      if (ichg) {
        atomicAdd(&q.gchanged[g], ichg);
        q.cmark[it] = 1;
      }
      ichg = 0;
      item_sh = queue_pop(q, par, from);
    }
    __syncthreads();
  }
  // one device atomic per counter and workgroup
  flush_stats(my_edges, my_changed, 0ull, st, 0);
  __shared__ unsigned long long wp[kQWaves];
  const unsigned long long p = wave_sum_u64(my_proc);
  if (lane == 0) wp[wv] = p;
  __syncthreads();
  if (tid == 0) {
    unsigned long long t = 0;
    for (int x = 0; x < kQWaves; ++x) t += wp[x];
    if (t) atomicAdd(&stat_slot(st)[kStatProcessed], t);
  }
}

// Counters of the iteration; the other queue half is emptied for the step
// kernel to refill.
__global__ void k_queue_iter_begin(QueueArgs q) {
  DevStats* st = q.st;
  if (st->stop) return;
  begin_iteration(st);
  const int np = (st->iter + 1) & 1, tid = threadIdx.x;
  if (tid < 2 * kXcds) q.qctr[(size_t)(np * 2 * kXcds + tid) * kQueueCtrStride] = 0u;
}

// Per graph still running: Algorithm 1's stop test on its own counts, then
// its marked chunks into the next queue half (one tail atomic per round of
// 256 chunks).
__global__ __launch_bounds__(kQBT) void k_queue_step(QueueArgs q) {
  __shared__ uint32_t wcnt[kQWaves];
  __shared__ uint32_t base_sh;
  __shared__ int state_sh;
  DevStats* st = q.st;
  if (st->stop) return;
  const int l = st->iter;
  const int np = (l + 1) & 1;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int32_t g = blockIdx.x; g < q.b.G; g += gridDim.x) {
    if (tid == 0) {
      int state = 0;  // 0: stopped earlier, 1: stops now, 2: runs on
      if (!q.b.done[g]) {
        const unsigned int t = q.gchanged[g];
        q.gchanged[g] = 0u;
        const int64_t ng = q.b.v_off[g + 1] - q.b.v_off[g];
        q.b.changed_last[g] = (long long)t;
        const bool f = (!st->pl && (double)t < st->tol * (double)ng) || l + 1 >= st->cap;
        if (f) {
          q.b.done[g] = 1;
          q.b.iters[g] = l + 1;
          state = 1;
        } else {
          atomicAdd(&st->graphs_left, 1u);
          state = 2;
        }
      }
      state_sh = state;
    }
    __syncthreads();
    if (state_sh == 2) {
      const int64_t c0 = q.cbase[g], c1 = q.cbase[g + 1];
      const int64_t gv0 = q.b.v_off[g], gv1 = q.b.v_off[g + 1];
      const uint32_t* Bn = np ? q.B1 : q.B0;
      const uint32_t x = (uint32_t)g & (uint32_t)(kXcds - 1);
      const int64_t CH = (int64_t)1 << q.chunk_log2;
      uint32_t* out = q.items + (size_t)np * (size_t)q.nchunks + (size_t)q.qbase[x];
      for (int64_t cb = c0; cb < c1; cb += kQBT) {
        const int64_t c = cb + tid;
        bool vis = false;
        if (c < c1) {
          if (q.cmark[c]) {
            q.cmark[c] = 0;
            vis = true;
          } else if (graph_bits(gv0, gv1) <= q.fb_words) {
            const int64_t v0 = gv0 + ((c - c0) << q.chunk_log2);
            const int64_t v1 = v0 + CH < gv1 ? v0 + CH : gv1;
            uint32_t any = 0;
            for (int64_t x = v0 >> 5; x <= (v1 - 1) >> 5 && !any; ++x) any = Bn[x] & word_mask(x, v0, v1);
            vis = any != 0u;
          }
        }
        const unsigned long long m = __ballot(vis);
        if (lane == 0) wcnt[wv] = (uint32_t)__popcll(m);
        __syncthreads();
        if (tid == 0) {
          uint32_t tot = 0;
          for (int w = 0; w < kQWaves; ++w) tot += wcnt[w];
          base_sh = tot ? atomicAdd(qtail(q.qctr, np, x), tot) : 0u;
        }
        __syncthreads();
        uint32_t pos = base_sh;
        for (int w = 0; w < wv; ++w) pos += wcnt[w];
        if (vis) out[pos + lane_rank(m)] = (uint32_t)c;
        __syncthreads();
      }
    }
    __syncthreads();
  }
}

// After the run, by chunk: each vertex's flag for a next iteration, held in
// the array of its graph's iteration-count parity, to the handle's flag bytes
// F0; in deterministic mode the labels of the graphs with an odd count move
// from C1 to C0, the handle's.
__global__ __launch_bounds__(kQBT) void k_queue_finish(QueueArgs q) {
  const bool det = q.C1 != q.C0;
  const int64_t CH = (int64_t)1 << q.chunk_log2;
  for (int64_t c = blockIdx.x; c < q.nchunks; c += gridDim.x) {
    const int32_t g = q.cgraph[c];
    const bool odd = q.b.iters[g] & 1;
    const int64_t gv0 = q.b.v_off[g], gv1 = q.b.v_off[g + 1];
    const bool bits = graph_bits(gv0, gv1) <= q.fb_words;
    if (!bits && !odd) continue;
    const uint32_t* B = odd ? q.B1 : q.B0;
    const int64_t v0 = gv0 + ((c - q.cbase[g]) << q.chunk_log2);
    const int64_t v1 = v0 + CH < gv1 ? v0 + CH : gv1;
    for (int64_t v = v0 + threadIdx.x; v < v1; v += kQBT) {
      q.F0[v] = bits ? (uint8_t)((B[v >> 5] >> (v & 31)) & 1u) : q.F1[v];
      if (det && odd) q.C0[v] = q.C1[v];
    }
  }
}

template <typename OffT>
__global__ void k_max_degree(const OffT* off, int64_t n, unsigned long long* dmax) {
  unsigned long long m = 0;
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < n;
       v += (int64_t)gridDim.x * blockDim.x) {
    const unsigned long long d = (unsigned long long)((int64_t)off[v + 1] - (int64_t)off[v]);
    m = d > m ? d : m;
  }
  for (int ofs = 32; ofs > 0; ofs >>= 1) {
    const unsigned long long o = __shfl_xor(m, ofs);
    m = o > m ? o : m;
  }
  if ((threadIdx.x & 63) == 0 && m) atomicMax(dmax, m);
}

// The initial queue (every chunk of every non-empty graph, in XCD parts)
// and its counters are built once by the host and copied in; every vertex is
// flagged for iteration 0, the odd flags, the chunk marks and the graphs'
// counts start at zero; deterministic mode starts both label arrays equal.
hipError_t launch_queue_begin(const QueueArgs& q, int64_t n, hipStream_t s) {
  hipError_t e = launch_fill_u32(q.B0, ~0u, (n + 31) / 32, s);
  if (e == hipSuccess) e = launch_fill_u32(q.B1, 0u, (n + 31) / 32, s);
  if (e == hipSuccess && q.F1) e = launch_fill_u8(q.F1, 0, n, s);
  if (e == hipSuccess) e = launch_fill_u8(q.cmark, 0, q.nchunks, s);
  if (e == hipSuccess) e = launch_fill_u32(q.gchanged, 0u, q.b.G, s);
  if (e == hipSuccess && q.C1 != q.C0)
    e = hipMemcpyAsync(q.C1, q.C0, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToDevice, s);
  return e;
}

hipError_t launch_queue_iter_begin(const QueueArgs& q, hipStream_t s) {
  hipLaunchKernelGGL(k_queue_iter_begin, dim3(1), dim3(64), 0, s, q);
  return hipGetLastError();
}

hipError_t launch_queue_sweep(bool off64, const QueueArgs& q, int grid, hipStream_t s) {
  if (q.chunk_log2 < 0 || q.chunk_log2 > kQueueMaxChunkLog2 || q.group_max < 1 ||
      q.group_max > 64 || q.fb_words < 0 || q.fb_words > kQueueFlagWords)
    return hipErrorInvalidValue;
  const size_t lds = (kQChunkBytes << q.chunk_log2) + sizeof(uint32_t) * (size_t)q.fb_words;
  auto launch = [&](auto oc, auto uc, auto dc) {
    hipLaunchKernelGGL((k_queue_sweep<decltype(oc), decltype(uc)::value, decltype(dc)::value>),
                       dim3(grid), dim3(kQBT), lds, s, q);
  };
  auto by_mode = [&](auto oc, auto uc) {
    if (q.async_mode) launch(oc, uc, std::false_type{});
    else launch(oc, uc, std::true_type{});
  };
  auto by_weight = [&](auto oc) {
    if (q.w) by_mode(oc, std::false_type{});
    else by_mode(oc, std::true_type{});
  };
  if (off64) by_weight(int64_t{});
  else by_weight(int32_t{});
  return hipGetLastError();
}

hipError_t launch_queue_step(const QueueArgs& q, hipStream_t s) {
  const int g = q.b.G < 8192 ? (q.b.G > 0 ? q.b.G : 1) : 8192;
  hipLaunchKernelGGL(k_queue_step, dim3(g), dim3(kQBT), 0, s, q);
  return hipGetLastError();
}

hipError_t launch_queue_finish(const QueueArgs& q, hipStream_t s) {
  const int64_t want = q.nchunks < 1 ? 1 : q.nchunks;
  hipLaunchKernelGGL(k_queue_finish, dim3((unsigned)(want < 8192 ? want : 8192)), dim3(kQBT), 0,
                     s, q);
  return hipGetLastError();
}

// Five workgroups per CU: 96 VGPRs; 22 KB of LDS at the default chunk and up to
// 8 KB of flag bits each.  (Those that start later find the queue drained.)
int queue_sweep_resident() { return 256 * 6; }

hipError_t launch_max_degree(bool off64, const void* off, int64_t n, unsigned long long* dmax,
                             hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t want = (n + 255) / 256;
  const int g = (int)(want < 2048 ? want : 2048);
  if (off64)
    hipLaunchKernelGGL(k_max_degree<int64_t>, dim3(g), dim3(256), 0, s,
                       static_cast<const int64_t*>(off), n, dmax);
  else
    hipLaunchKernelGGL(k_max_degree<int32_t>, dim3(g), dim3(256), 0, s,
                       static_cast<const int32_t*>(off), n, dmax);
  return hipGetLastError();
}

}  // namespace lpa
