// bpida_batch.hip -- batched, persistent Block-Parallel IDA* for gfx950.
//
// One launch searches every instance of a batch through all of its f-limits.
// Work lives in a device queue of chunks (up to 64 stack entries of one
// instance at one limit).  A workgroup (one wave64) pops a chunk into its LDS
// stack and runs BPDFS rounds (Alg. 1) on it; it gives the 64 oldest entries
// of its stack back to the queue when its stack would overflow LDS, or when
// other workgroups are idle and the queue holds fewer chunks than there are
// workgroups waiting for work (donation; the paper's BPIDA* balances statically, its
// intra-block donation idea for PFullLB is applied here across workgroups).
//
// Per instance, `outstanding` counts its chunks that are queued or held by a
// workgroup at the current limit.  The workgroup whose decrement brings it to
// zero completes the limit on the device: it adds the split tree's interior
// nodes, writes the node count of the limit, stops on a goal (all optimal
// solutions: the limit has been searched to completion), and otherwise
// advances the limit by 2 and seeds the instance's subtree roots again.
#include <limits.h>
#include <stddef.h>

#include "bpida_board.h"
#include "bpida_internal.h"
#include "bpida_ring.h"
#include "bpida_ring5.h"
#include "bpida_round.h"

namespace bpida {

#define AGENT __HIP_MEMORY_SCOPE_AGENT

// The split kernels' level sizes, built at compile time.
__device__ WalkTable g_walk_table = make_walk_table();

hipError_t walk_table_device(const int32_t** out) {
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_walk_table));
  *out = static_cast<const int32_t*>(p);
  return e;
}

// The search kernel's arguments, read where they lie.  The functions below
// that run once a chunk or a limit take a fresh view of them: values that the
// compiler may assume loaded already it keeps across the search loop, in
// scalar registers that it then spills around every round.
using Args = const __attribute__((address_space(4))) BatchArgs;
__device__ __forceinline__ Args& fresh() {
  Args* p = (Args*)__builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(p));
  return *p;
}
// (where BatchArgs::server is set only)
using Srv = const __attribute__((address_space(4))) ServerArgs;
__device__ __forceinline__ Srv& fresh_server() {
  using All = const __attribute__((address_space(4))) ServerBatchArgs;
  All* p = (All*)__builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(p));
  return p->srv;
}

__device__ __forceinline__ uint64_t ld_relaxed(uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, AGENT);
}
__device__ __forceinline__ int32_t ld_relaxed(int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, AGENT);
}
// The value lane 0 loads, in every lane: a branch on it is uniform (a
// per-lane load, even of one address, makes the compiler treat the branch
// as divergent).
__device__ __forceinline__ int32_t ld_wave(int32_t* p) {
  return __builtin_amdgcn_readfirstlane(ld_relaxed(p));
}

// ---------------------------------------------------------------------------
// Ticket queue of chunks.  Producers and consumers take tickets with a
// fetch-and-add on tail / head (no compare-and-swap loops on those two
// counters, which collapse under thousands of contending workgroups).  Slot
// k of the ring carries the state of ticket t = the next ticket to use it:
// 4t free for producer t, 4t + 1 claimed by producer t (being written),
// 4t + 2 holds the chunk of ticket t.  An idle wave takes one consumer ticket
// and then polls only its own slot, so waiting waves do not contend on a
// shared line; head - tail = waiting waves - queued chunks, which is what a
// busy wave reads to decide whether to donate.  Every operation is done by a
// whole wave: lane 0 handles tickets, all lanes move the 64 entries.
//
// A producer whose slot is still occupied after A.push_spin polls gives its
// ticket up and raises the slot's `abandoned` mark to at least t + 1.  A
// consumer holding ticket t whose slot is free for t while the mark is past
// t hands the slot on to ticket t + capacity with a compare-and-swap (the
// producer claims it with one too, so exactly one of them wins; a late
// producer that loses gives up as well).  A lost ticket therefore never
// strands a consumer and the ring keeps working; the lost chunk's work is
// gone, its instance is marked lost and the call reports BPIDA_ENOMEM.
// ---------------------------------------------------------------------------
constexpr uint64_t kNoTicket = ~0ull;

__device__ __forceinline__ uint64_t bcast64(uint64_t v) {
  const uint32_t lo = (uint32_t)wave_bcast((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)wave_bcast((int)(uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ bool cas64(uint64_t* p, uint64_t expect, uint64_t want) {
  return __hip_atomic_compare_exchange_strong(p, &expect, want, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                              AGENT);
}

// Payload and bookkeeping that pass between waves go through relaxed
// agent-scope accesses (which read and write past the caches that other
// compute units do not see) in an order kept by waiting for the earlier ones:
// a release would write back this XCD's whole L2 and an acquire drop its
// lines, on every hand-over.
__device__ __forceinline__ void performed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
template <class T>
__device__ __forceinline__ void st_relaxed(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, AGENT);
}
template <class T>
__device__ __forceinline__ T ld_agent(const T* p) {
  return __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, AGENT);
}

// One chunk in a wave's registers: lane k holds entry k; the rest is uniform.
struct Unit {
  uint64_t tile = 0, hi = 0;  // hi: 5x5 only
  uint16_t meta = 0;
  int count = 0, inst = 0, kind = 0, limit = 0, width = 0;
};

// Work of instance i that had been added to its outstanding units could not be
// queued: takes `units` of them back and marks the instance's counts void.
__device__ __forceinline__ void drop_units(int i, int units, int err) {
  Args& A = fresh();
  if (lane_id() == 0) {
    st_relaxed(&A.is[i].lost, 1);
    atomicOr(&A.q->err, err);
    performed();
    __hip_atomic_fetch_add(&A.is[i].outstanding, -units, __ATOMIC_RELAXED, AGENT);
  }
}

// lane / parts for parts 1, 3 and 7 (lane below 64, and the counts up to 70
// that q_push rounds up).
__device__ __forceinline__ uint32_t lane_over(uint32_t lane, int parts) {
  return parts == 1 ? lane : (lane * (parts == 3 ? 21846u : 9363u)) >> 16;
}
constexpr bool check_lane_over() {
  for (uint32_t l = 0; l <= 70; ++l)
    if (((l * 21846u) >> 16) != l / 3 || ((l * 9363u) >> 16) != l / 7) return false;
  return true;
}
static_assert(check_lane_over(), "lane division");

// Pushes the unit's entries as `parts` (1, 3 or 7) chunks, entry j to chunk j
// modulo parts.  One part: returns false if the ring stayed full for the whole
// bounded wait (the entries were not queued).  Several parts cost what one
// does; a part that a full ring refuses is dropped, its instance's counts void.
// `pos`: the first ticket.
__device__ __forceinline__ bool q_push(const Unit& u, RunStats& wc, uint64_t& pos, int parts) {
  Args& A = fresh();
  const int lane = lane_id();
  QueueCtl* q = A.q;
  const uint64_t mask = A.qmask;
  uint64_t depth = 0;
  if (lane == 0) {
    pos = __hip_atomic_fetch_add(&q->tail, (uint64_t)parts, __ATOMIC_RELAXED, AGENT);
    if ((pos & 7) == 0) {  // (the line of `head` is busy with takes)
      const uint64_t h = ld_relaxed(&q->head);
      if (pos + 1 > h) depth = pos + 1 - h;
    }
  }
  pos = bcast64(pos);
  const bool head = lane < parts;  // lane c looks after chunk c
  const uint64_t my = pos + (uint64_t)(head ? lane : 0);
  SlotCtl* sc = A.seq + (my & mask);
  bool ok = false, open = head;
  for (int k = 0; k < A.push_spin; ++k) {
    if (open) {
      const uint64_t v = ld_relaxed(&sc->seq);
      if (v == 4 * my) {
        ok = cas64(&sc->seq, 4 * my, 4 * my + 1);
        open = false;
      } else if (v > 4 * my) {
        open = false;  // handed on past this ticket by its consumer
      }
    }
    if (!__builtin_amdgcn_ballot_w64(open)) break;
    __builtin_amdgcn_s_sleep(1);
  }
  if (head && !ok) {
    __hip_atomic_fetch_max(&sc->abandoned, my + 1, __ATOMIC_RELAXED, AGENT);
    atomicOr(&q->err, 16);  // ticket lost: the call reports BPIDA_ENOMEM
  }
  const uint64_t okm = __builtin_amdgcn_ballot_w64(ok);
  wc.qmax = max(wc.qmax, bcast64(depth));
  if (parts == 1 && okm == 0) return false;
  const uint32_t row = lane_over((uint32_t)lane, parts), part = (uint32_t)lane - row * (uint32_t)parts;
  if (lane < u.count && ((okm >> part) & 1ull)) {
    const uint64_t slot = (pos + part) & mask;
    st_relaxed(&A.slots[slot].tiles[row], u.tile);
    if (u.kind & kChunkWide) st_relaxed(&A.hi[slot * kQChunk + row], u.hi);
    st_relaxed(&A.slots[slot].meta[row], u.meta);
  }
  if (ok) {
    QChunk* c = A.slots + (my & mask);
    const int count = (int)lane_over((uint32_t)(u.count - lane + parts - 1), parts);
    st_relaxed(&c->inst, (int32_t)u.inst);
    st_relaxed(&c->info, (int32_t)(count | (u.kind << 8) | (u.width << 16)));
    st_relaxed(&c->limit, (int32_t)u.limit);
  }
  performed();  // the payload, and the atomics on the instance before it, come first
  if (ok) st_relaxed(&sc->seq, 4 * my + 2);
  const int lost = parts - (int)__popcll(okm);
  if (lost) drop_units(u.inst, lost, 2);
  return true;
}

__device__ __forceinline__ bool q_push(const Unit& u, RunStats& wc, int parts = 1) {
  uint64_t pos = 0;
  return q_push(u, wc, pos, parts);
}

// Takes a consumer ticket if `ticket` holds none, then checks whether that
// ticket's chunk has arrived: 1 with the chunk; 0 not yet (the ticket is kept
// for the next call, or dropped if its producer gave up); -1 the search is
// over.
__device__ __forceinline__ int q_take(uint64_t& ticket, Unit& u, RunStats& wc) {
  Args& A = fresh();
  const int lane = lane_id();
  QueueCtl* q = A.q;
  const uint64_t mask = A.qmask;
  int ready = 0;
  if (lane == 0) {
    const bool fresh = ticket == kNoTicket;
    if (fresh) {
      ticket = __hip_atomic_fetch_add(&q->head, (uint64_t)1, __ATOMIC_RELAXED, AGENT);
      performed();  // a ticket that end_search did not see sees `remaining` below
    }
    SlotCtl* sc = A.seq + (ticket & mask);
    const uint64_t v = ld_relaxed(&sc->seq);
    ready = v == 4 * ticket + 2 ? 1 : v == kSeqEnd ? -1 : 0;
    if (!ready && fresh && ld_relaxed(&q->remaining) <= 0) ready = -1;
    if (!ready && v == 4 * ticket && ld_relaxed(&sc->abandoned) > ticket &&
        cas64(&sc->seq, 4 * ticket, 4 * (ticket + mask + 1))) {
      // a producer of this slot gave up at or after this ticket: hand the
      // slot on and take a new ticket next time
      ticket = kNoTicket;
    }
  }
  ticket = bcast64(ticket);
  ready = wave_bcast(ready);
  if (ready <= 0) return ready;
  asm volatile("" ::: "memory");  // the payload is read after the slot's state
  const QChunk* c = A.slots + (ticket & mask);
  u.tile = ld_agent(&c->tiles[lane]);
  u.meta = ld_agent(&c->meta[lane]);
  const int inst = ld_agent(&c->inst), info = ld_agent(&c->info), limit = ld_agent(&c->limit);
  u.inst = wave_bcast(inst);
  u.limit = wave_bcast(limit);
  u.count = wave_bcast(info) & 255;
  u.kind = (wave_bcast(info) >> 8) & 255;
  u.width = wave_bcast(info) >> 16;
  // the high words only for a 5x5 chunk: a 4x4 chunk reads 6 lines, not 10
  const bool wide = (u.kind & kChunkWide) != 0;
  u.hi = wide ? ld_agent(&A.hi[(ticket & mask) * kQChunk + lane]) : 0ull;
  wc.chunks_read_wide += wide ? 1 : 0;
  performed();  // all lanes have read the slot before it is handed back
  if (lane == 0) st_relaxed(&A.seq[ticket & mask].seq, 4 * (ticket + mask + 1));
  ticket = kNoTicket;
  return 1;
}

// Called by the wave that brought `remaining` to zero: no chunk is queued or
// held any more (the caller has waited for that decrement).  Tells every wave
// that waits on a ticket; one that takes its ticket after the fetch_add below
// sees `remaining` itself.
__device__ __forceinline__ void end_search() {
  Args& A = fresh();
  const int lane = lane_id();
  uint64_t h = 0, t = 0;
  if (lane == 0) {
    h = __hip_atomic_fetch_add(&A.q->head, (uint64_t)0, __ATOMIC_RELAXED, AGENT);
    t = ld_relaxed(&A.q->tail);
  }
  h = bcast64(h);
  t = bcast64(t);
  if (h > t + A.qmask + 1) t = h - A.qmask - 1;
  for (uint64_t k = t + (uint64_t)lane; k < h; k += 64) st_relaxed(&A.seq[k & A.qmask].seq, kSeqEnd);
}

// ---------------------------------------------------------------------------
// Limit bookkeeping, executed by one wave.
// ---------------------------------------------------------------------------

// Whether the queue has A.deal slots free beyond producer ticket t (the slot
// that far ahead is ready for its next ticket; slots fill in order).
__device__ __forceinline__ bool queue_has_room(uint64_t t) {
  Args& A = fresh();
  const uint64_t ahead = t + (uint64_t)A.deal;
  int room = 0;
  if (lane_id() == 0) room = ld_relaxed(&A.seq[ahead & A.qmask].seq) >= 4 * ahead;
  return wave_bcast(room) != 0;
}

// Most roots of a limit that is dealt out.  Chunks of 64 of more of them are
// enough for the waves there are, and more but smaller ones cost their
// hand-overs: dealt, split depth 12 took 5.3 ms for 2 hard 4x4 states against
// 3.3 and 28.9 for 4 5x5 states against 19.2, depth 8 (1383 roots on average)
// 5.8 ms for 30 5x5 states against 5.0; but 30 hard 4x4 states at depth 8 (635
// roots) 13.6 against 14.6.
constexpr int kDealRoots = 768;

// Hands the roots of instance i with f <= L out as chunks: the last one stays
// with the caller (`mine`: it is searched next, or pushed), the others go to
// the queue.  A guard unit keeps the limit from completing meanwhile; it
// becomes mine's unit.  Returns true if there is no chunk and the guard's
// release brought the instance's outstanding count to zero, i.e. the caller
// must complete the limit itself.
// `stage` (128 u64) and `stage_m` (64 u16) are LDS the caller does not use
// while seeding (its LDS stack is empty whenever a limit is seeded).
// `nodes`: what the limit before it expanded (0: the first).  A limit that
// will keep one wave busy for long (the next one expands some four times the
// nodes) is dealt out at once to the waves that wait: every 64 roots go to 2,
// 4 or 8 of them (this wave among them for the last), 8192 nodes' worth each
// at least, whether they go on waiting or not, as long as the queue keeps room
// for all chunks of 64 roots and for spills (BatchArgs::deal): a queue that
// dealt chunks fill stops every wave that has to push, and the call can end in
// BPIDA_ENOMEM.  (Dealing no more chunks than waves wait at each 64 roots costs
// 4096 easy states 11 %: many small chunks even their ends out.)  Against one
// wave that donates from its 32nd round on: one hard state 1.25 -> 1.14 ms, 64
// easy ones 562 -> 525 us; at half these counts the easy ones take 3 % longer.
template <int W>
__device__ __forceinline__ bool seed_limit(int i, int L, uint64_t nodes, uint64_t* stage, uint16_t* stage_m,
                                           Unit& mine, RunStats& wc) {
  Args& A = fresh();
  const int lane = lane_id();
  InstState* S = A.is + i;
  const int width = W ? W : S->width;
  const bool wide = width == 5;
  if (lane == 0) st_relaxed(&S->outstanding, 1);
  const NodeW* roots = A.tree + S->root_off;
  // first-solution mode: a goal inside the split tree ends the search at
  // this limit without searching any subtree
  const int nroots = (A.first_solution && A.goal_g[i] <= L) ? 0 : S->nroots;
  int fm = INT_MAX;
  bool full = false;
  int parts = 0;  // chunks dealt out beside this wave's own
  uint64_t pushed = kNoTicket;  // ticket of the last push
  if (nodes >= 4096 && nroots <= kDealRoots && A.deal) {
    int64_t ht = 0;
    if (lane == 0) ht = (int64_t)(ld_relaxed(&A.q->head) - ld_relaxed(&A.q->tail));
    const int wait = wave_bcast((int)ht);
    parts = wait >= 7 && nodes >= 16384 ? 7 : wait >= 3 && nodes >= 8192 ? 3 : wait >= 1 ? 1 : 0;
  }
  mine.count = 0;
  mine.inst = i;
  mine.limit = L;
  mine.width = width;
  mine.kind = wide ? kChunkWide : kChunkNodes;
  for (int base = 0; base < nroots && !full; base += 64) {
    const int r = base + lane;
    NodeW R;
    R.lo = 0;
    R.hi = 0;
    R.meta = 0;
    R.f = 0;
    bool keep = false;
    if (r < nroots) {
      R = roots[r];
      keep = (int)R.f <= L;
      if (!keep) fm = min(fm, (int)R.f);
    }
    const uint64_t km = __ballot(keep);
    const int cnt = __popcll(km);
    if (cnt == 0) continue;
    // compact the kept roots into lanes 0..cnt-1 through LDS
    const int off = __builtin_amdgcn_mbcnt_hi((uint32_t)(km >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
    if (keep) {
      stage[off] = R.lo;
      stage[64 + off] = R.hi;
      stage_m[off] = stack_meta((int)(R.meta & 31u), (int)((R.meta >> 5) & 7u), L - (int)R.f);
    }
    WAVE_SYNC();
    // chunks of seed_chunk roots: smaller seeds when a batch has few roots
    // per workgroup, so the whole grid has work from the start
    const int sc = A.seed_chunk > 0 ? A.seed_chunk : kQChunk;
    for (int p0 = 0; p0 < cnt && !full; p0 += sc) {
      const int n = min(sc, cnt - p0);
      if (parts && pushed != kNoTicket && !queue_has_room(pushed)) parts = 0;
      const bool deal = n > parts && parts > 0;
      // entry e of the chunk stays if e is a multiple of parts + 1
      const int stride = deal ? parts + 1 : 1;
      const int keep = deal ? (int)((uint32_t)(n + parts) / (uint32_t)stride) : n;
      auto from_stage = [&](int e, int count) {
        const bool on = lane < count;
        mine.count = count;
        mine.tile = on ? stage[p0 + e] : 0ull;
        mine.hi = on ? stage[64 + p0 + e] : 0ull;
        mine.meta = on ? stage_m[p0 + e] : (uint16_t)0;
      };
      // first the chunk kept so far, then what this one deals out
#pragma unroll 1
      for (int turn = mine.count ? 0 : 1; turn < (deal ? 2 : 1) && !full; ++turn) {
        const int k = turn ? parts : 1;
        if (turn) {
          const uint32_t row = lane_over((uint32_t)lane, parts);
          from_stage((int)(row * (uint32_t)stride + 1 + ((uint32_t)lane - row * (uint32_t)parts)), n - keep);
        }
        if (lane == 0) __hip_atomic_fetch_add(&S->outstanding, k, __ATOMIC_RELAXED, AGENT);
        full = !q_push(mine, wc, pushed, k);
      }
      if (!full) from_stage(lane * stride, keep);
    }
    WAVE_SYNC();
  }
  if (full) drop_units(i, 1, 1);  // the remaining roots are dropped; the call reports BPIDA_ENOMEM
  fm = wave_min(fm);
  if (lane == 0 && fm != INT_MAX) __hip_atomic_fetch_min(&S->fmin, fm, __ATOMIC_RELAXED, AGENT);
  wc.roots_read += (uint64_t)nroots;
  if (mine.count) return false;
  performed();
  int last = 0;
  if (lane == 0) last = __hip_atomic_fetch_add(&S->outstanding, -1, __ATOMIC_RELAXED, AGENT) == 1;
  return wave_bcast(last) != 0;
}

// Server mode: copy slot i's answer into the pinned result ring, publish it,
// and free the slot.  Executed by one wave after the slot's outputs are final.
__device__ __forceinline__ void emit_result(int i, int status) {
  Args& A = fresh();
  const int lane = lane_id();
  Srv& V = fresh_server();
  WAVE_SYNC_MEM();  // the slot's output row, written by lane 0, is visible
  const uint64_t t = V.ticket[i];
  ServerRes* r = V.res + (t & V.ring_mask);
  // (columns of earlier limits may come from other waves)
  r->nodes[lane] = ld_agent(&A.out_nodes[(size_t)i * 64 + lane]);
  if (lane == 0) {
    r->len = ld_agent(&A.out_len[i]);
    r->status = status;
  }
  WAVE_SYNC_MEM();
  if (lane == 0) {
    __hip_atomic_store(&r->seq, t + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&V.busy[i], 0, __ATOMIC_RELEASE, AGENT);
    __hip_atomic_fetch_add(V.in_flight, -1, __ATOMIC_RELEASE, AGENT);
  }
}

// Completes limit L of instance i (its outstanding count is zero and this
// wave observed it), then advances it.  Loops while a new limit has no work;
// the new limit's last chunk is left in `mine` (count 0: the instance is
// done).
template <int W>
__device__ __forceinline__ void complete_limit(int i, int L, uint64_t* stage, uint16_t* stage_m, Unit& mine,
                           RunStats& wc) {
  Args& A = fresh();
  const int lane = lane_id();
  InstState* S = A.is + i;
  mine.count = 0;
  // the server's split trees and histograms are written while the kernel runs
  if (A.server) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  for (;;) {
    const int col = ld_relaxed(&S->col), goals = ld_relaxed(&S->goals), lost = ld_relaxed(&S->lost);
    const uint64_t searched = ld_relaxed(&S->nodes);
    const int fsearch = ld_relaxed(&S->fmin);
    const int goal_g = A.goal_g[i];
    // interior nodes of the split tree (depth < D) expanded at this limit
    const uint32_t* h = A.hist + (size_t)i * kHistBins;
    uint32_t interior = 0;
    int fm = INT_MAX;
    uint32_t c[kHistBins / 64];
    for (int k = 0; k < kHistBins / 64; ++k) c[k] = h[64 * k + lane];
    for (int k = 0; k < kHistBins / 64; ++k) {
      const int f = 64 * k + lane;
      if (f <= L) interior += c[k];
      else if (c[k]) fm = min(fm, f);
    }
    for (int o = 32; o > 0; o >>= 1) interior += __shfl_xor(interior, o, 64);
    fm = wave_min(fm);
    int state = 0;  // 0: advance, 1: solved, <0: error code
    int left = 1;
    const uint64_t total = searched + interior;
    if (lane == 0) {
      st_relaxed(&A.out_nodes[(size_t)i * 64 + col], total);
      const int fnext = min(fm, fsearch);
      if (lost) {
        state = -4;  // BPIDA_ENOMEM: work of this limit was dropped, its counts are void
      } else if (goals > 0 || goal_g <= L) {
        st_relaxed(&A.out_len[i], L);
        state = 1;
      } else if (fnext != L + 2) {
        state = -6;  // BPIDA_EINTERNAL
      } else if (A.exact_limit) {
        state = 2;  // one limit only, and no goal within it
      } else if (col + 1 >= 64 || L + 2 > A.max_limit) {
        state = -3;  // BPIDA_ELIMIT
      }
      if (state != 0) {
        st_relaxed(&S->done, state);
        if (!A.server) left = __hip_atomic_fetch_add(&A.q->remaining, -1, __ATOMIC_RELAXED, AGENT) - 1;
      } else {
        st_relaxed(&S->limit, L + 2);
        st_relaxed(&S->col, col + 1);
        st_relaxed(&S->nodes, (uint64_t)0);
        st_relaxed(&S->fmin, INT_MAX);
        st_relaxed(&S->goals, 0);
      }
    }
    state = wave_bcast(state);
    if (state != 0) {
      performed();
      if (A.server) emit_result(i, state);
      else if (wave_bcast(left) == 0) end_search();
      return;
    }
    L += 2;
    if (!seed_limit<W>(i, L, total, stage, stage_m, mine, wc)) return;
  }
}

// ---------------------------------------------------------------------------
// Server admission, executed by the one workgroup holding the admitter role.
// ---------------------------------------------------------------------------

// Validate and pack a state of 16 bytes (in pinned host memory) with one wave.
__device__ __forceinline__ Inst wave_ingest4(const uint8_t* src) {
  const int lane = lane_id();
  const uint32_t v = lane < 16 ? (uint32_t)src[lane] : 0u;
  // permutation: every value 0..15 exactly once
  uint32_t seen = lane < 16 && v < 16 ? (1u << v) : 0u;
  for (int o = 32; o > 0; o >>= 1) seen |= __shfl_xor(seen, o, 64);
  const uint64_t valid = __builtin_amdgcn_ballot_w64(lane < 16 && v < 16);
  const uint64_t blank_m = __builtin_amdgcn_ballot_w64(lane < 16 && v == 0);
  // inversions: lane p counts q > p with v[q] < v[p]
  uint32_t inv = 0;
  for (int q = 0; q < 16; ++q) {
    const uint32_t vq = (uint32_t)__shfl((int)v, q, 64);
    inv += (lane < 16 && q > lane && vq < v) ? 1u : 0u;
  }
  int h = 0;
  if (lane < 16 && v != 0) {
    const int dr = (lane >> 2) - (int)(v >> 2), dc = (lane & 3) - (int)(v & 3);
    h = (dr < 0 ? -dr : dr) + (dc < 0 ? -dc : dc);
  }
  uint64_t word = lane < 16 ? (uint64_t)(v & 15u) << (4 * lane) : 0ull;
  for (int o = 32; o > 0; o >>= 1) {
    inv += (uint32_t)__shfl_xor((int)inv, o, 64);
    h += __shfl_xor(h, o, 64);
    word |= (uint64_t)__shfl_xor((long long)word, o, 64);
  }
  Inst I;
  I.tiles = word;
  I.blank = blank_m ? (int)__builtin_ctzll(blank_m) : 0;
  I.h0 = h;
  I.pad = 0;
  if (seen != 0xFFFFu || valid != 0xFFFFull) I.status = -1;  // BPIDA_EINVAL
  else {
    const uint32_t bpar = (uint32_t)((I.blank >> 2) + (I.blank & 3)) & 1u;
    I.status = ((inv & 1u) == bpar) ? 0 : -2;  // BPIDA_EUNSOLVABLE
  }
  return I;
}

// The root split of one instance with one wave (CreateRootSet; same tree as
// split4_kernel): levels 0..depth of the parent-pruned tree are written to
// base[], interior nodes binned by f in hist_lds (256 entries of LDS).
// Returns the first root's index inside base; the root count is
// walks[blank][depth].
__device__ __forceinline__ int64_t wave_split4(const Inst& I, int depth, const int32_t* walks, NodeW* base,
                               uint32_t* hist_lds, uint32_t* hist_out, int32_t* goal_g_out) {
  const int lane = lane_id();
  for (int k = lane; k < kHistBins; k += 64) hist_lds[k] = 0;
  if (lane == 0) {
    NodeW r;
    r.lo = I.tiles;
    r.hi = 0;
    r.meta = node_meta(I.blank, 4, 0, I.h0);
    r.f = (uint32_t)I.h0;
    base[0] = r;
  }
  WAVE_SYNC_MEM();
  const int32_t* lc = walks + walk_row(I.blank, 4);
  int gmin = INT_MAX;
  int64_t lvl = 0;
  for (int d = 0; d < depth; ++d) {
    const int cnt = lc[d];
    const int64_t next = lvl + cnt;
    int64_t fill = next;
    for (int k0 = 0; k0 < cnt; k0 += 64) {
      const int k = k0 + lane;
      NodeW nd;
      nd.lo = 0;
      nd.hi = 0;
      nd.meta = 0;
      nd.f = 0;
      if (k < cnt) nd = base[lvl + k];
      const int b = (int)(nd.meta & 31u), fb = (int)((nd.meta >> 5) & 7u);
      const int g = (int)((nd.meta >> 8) & 255u), h = (int)((nd.meta >> 16) & 255u);
      if (k < cnt) {
        atomicAdd(&hist_lds[min(g + h, kHistBins - 1)], 1u);
        if (nd.lo == kGoal4) gmin = min(gmin, g);
      }
      for (int a = 0; a < 4; ++a) {
        const bool ok = k < cnt && ((kMoveMask4 >> (4 * b + a)) & 1ull) && a != fb;
        const int nn = (b + (a == 0 ? -4 : a == 1 ? -1 : a == 2 ? 1 : 4)) & 15;
        const uint32_t t = (uint32_t)(nd.lo >> (4 * nn)) & 15u;
        const int sh = (a == 0 || a == 3) ? 2 : 0;
        const uint32_t idx = (((t >> sh) & 3u) << 2) | (((uint32_t)nn >> sh) & 3u);
        const int h2 = h + (((kDhTable4 >> (16 * a + idx)) & 1ull) ? 1 : -1);
        const uint64_t km = __builtin_amdgcn_ballot_w64(ok);
        const int off = __builtin_amdgcn_mbcnt_hi((uint32_t)(km >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
        if (ok && fill + off < next + lc[d + 1]) {  // the level's exact size bounds it
          NodeW c;
          c.lo = nd.lo + ((uint64_t)t << (4 * b)) - ((uint64_t)t << (4 * nn));
          c.hi = 0;
          c.meta = node_meta(nn, 3 - a, g + 1, h2);
          c.f = (uint32_t)(g + 1 + h2);
          base[fill + off] = c;
        }
        fill += __popcll(km);
      }
    }
    WAVE_SYNC_MEM();  // this level's children are visible to the whole wave
    lvl = next;
  }
  gmin = wave_min(gmin);
  for (int k = lane; k < kHistBins; k += 64) hist_out[k] = hist_lds[k];
  if (lane == 0) *goal_g_out = gmin;
  WAVE_SYNC_MEM();
  return lvl;
}

// Seeds a request's first limit with every chunk in the queue: the admitter
// searches nothing itself.
__device__ __forceinline__ void admit_limit(int i, int L, uint64_t* st, uint16_t* sm) {
  Args& A = fresh();
  Unit mine;
  RunStats wc = {};  // (the admitter's own counts are not reported)
  if (seed_limit<4>(i, L, 0, st, sm, mine, wc)) complete_limit<4>(i, L, st, sm, mine, wc);
  while (mine.count && !q_push(mine, wc)) {
    // lost: this was the instance's last unit unless other chunks are out
    int last = 0;
    if (lane_id() == 0) {
      st_relaxed(&A.is[i].lost, 1);
      atomicOr(&A.q->err, 1);
      performed();
      last = __hip_atomic_fetch_add(&A.is[i].outstanding, -1, __ATOMIC_RELAXED, AGENT) == 1;
    }
    L = mine.limit;
    mine.count = 0;
    if (wave_bcast(last)) complete_limit<4>(i, L, st, sm, mine, wc);
  }
}

// Admits requests until the host asks to stop and nothing is in flight.
__device__ __forceinline__ void admitter_loop(uint64_t* st, uint16_t* sm, uint64_t deadline) {
  Args& A = fresh();
  const int lane = lane_id();
  Srv& V = fresh_server();
  QueueCtl* q = A.q;
  uint32_t* hist_lds = (uint32_t*)st;  // the stack is unused by the admitter
  uint64_t head = 0;
  int cursor = 0;
  for (;;) {
    if (wall_clock64() > deadline) {
      if (lane == 0) {
        atomicOr(&q->err, 8);
        __hip_atomic_store(&q->remaining, 0, __ATOMIC_RELEASE, AGENT);
      }
      return;
    }
    uint64_t tail = 0;
    int stop = 0, busy_all = 0;
    if (lane == 0) {
      tail = __hip_atomic_load(&V.host->req_tail, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
      stop = __hip_atomic_load(&V.host->stop, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    tail = bcast64(tail);
    stop = wave_bcast(stop);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");  // request bytes published before req_tail
    if (tail == head) {
      if (stop) {
        int inflight = 0;
        if (lane == 0) inflight = __hip_atomic_load(V.in_flight, __ATOMIC_ACQUIRE, AGENT);
        if (wave_bcast(inflight) == 0) {
          if (lane == 0) st_relaxed(&q->remaining, 0);
          performed();
          end_search();
          return;
        }
      }
      __builtin_amdgcn_s_sleep(32);
      continue;
    }
    // the HBM frontier budget: while more chunks wait in the work queue than
    // the budget allows, the searching workgroups are behind, and a new
    // request's seeds (and later spills) could overflow it; wait
    if (V.backlog_max > 0) {
      int64_t backlog = 0;
      if (lane == 0) backlog = (int64_t)(ld_relaxed(&q->tail) - ld_relaxed(&q->head));
      backlog = (int64_t)bcast64((uint64_t)backlog);
      if (backlog > V.backlog_max) {
        __builtin_amdgcn_s_sleep(32);
        continue;
      }
    }
    // a free instance slot (the in-flight budget); wait if none
    int slot = -1;
    for (int k0 = 0; k0 < V.slots && slot < 0; k0 += 64) {
      const int j = (cursor + k0 + lane) % V.slots;
      const bool fr = k0 + lane < V.slots &&
                      __hip_atomic_load(&V.busy[j], __ATOMIC_ACQUIRE, AGENT) == 0;
      const uint64_t fm = __builtin_amdgcn_ballot_w64(fr);
      if (fm) slot = (cursor + k0 + (int)__builtin_ctzll(fm)) % V.slots;
    }
    if (slot < 0) {
      busy_all = 1;
      __builtin_amdgcn_s_sleep(32);
      continue;
    }
    (void)busy_all;
    cursor = (slot + 1) % V.slots;
    const Inst I = wave_ingest4(V.req[head & V.ring_mask].state);
    if (lane == 0) {
      __hip_atomic_store(&V.host->req_admitted, head + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
      V.busy[slot] = 1;
      V.ticket[slot] = head;
      __hip_atomic_fetch_add(V.in_flight, 1, __ATOMIC_RELAXED, AGENT);
    }
    A.out_nodes[(size_t)slot * 64 + lane] = 0;
    if (lane == 0) A.out_len[slot] = -1;
    InstState S;
    S.limit = first_limit(I.h0, A.start_limit);
    S.col = (S.limit - I.h0) / 2;
    S.done = I.status;
    S.outstanding = 0;
    S.nodes = 0;
    S.fmin = INT_MAX;
    S.goals = 0;
    S.stop = 0;
    S.lost = 0;
    S.root_off = (int64_t)slot * V.stride;
    S.nroots = 0;
    S.width = 4;
    if (I.status == 0) {
      NodeW* base = const_cast<NodeW*>(A.tree) + (int64_t)slot * V.stride;
      const int64_t r0 = wave_split4(I, V.depth, V.walks, base, hist_lds,
                                     const_cast<uint32_t*>(A.hist) + (size_t)slot * kHistBins,
                                     const_cast<int32_t*>(A.goal_g) + slot);
      S.root_off += r0;
      S.nroots = V.walks[walk_row(I.blank, 4) + V.depth];
      // a first limit past the cap or past the 64 output columns
      if (S.limit > A.max_limit || S.col >= 64) S.done = -3;  // BPIDA_ELIMIT
    }
    if (lane == 0) A.is[slot] = S;
    WAVE_SYNC_MEM();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (S.done != 0) emit_result(slot, S.done);
    else admit_limit(slot, S.limit, st, sm);
    ++head;
  }
}

// Adds this wave's counts for the unit of instance i it held at limit L and
// releases the unit; completes the limit if it was the last unit, which may
// leave the next limit's chunk in `mine`.
template <int W>
__device__ __forceinline__ void release_unit(int i, int L, uint64_t expanded, int goals, int fmin,
                             uint64_t* stage, uint16_t* stage_m, Unit& mine,
                           RunStats& wc) {
  Args& A = fresh();
  const int lane = lane_id();
  InstState* S = A.is + i;
  mine.count = 0;
  fmin = wave_min(fmin);
  if (lane == 0) {
    if (expanded) __hip_atomic_fetch_add(&S->nodes, expanded, __ATOMIC_RELAXED, AGENT);
    if (goals) __hip_atomic_fetch_add(&S->goals, goals, __ATOMIC_RELAXED, AGENT);
    if (fmin != INT_MAX) __hip_atomic_fetch_min(&S->fmin, fmin, __ATOMIC_RELAXED, AGENT);
  }
  performed();  // the counts are in before the unit is gone
  int last = 0;
  if (lane == 0) last = __hip_atomic_fetch_add(&S->outstanding, -1, __ATOMIC_RELAXED, AGENT) == 1;
  if (wave_bcast(last)) complete_limit<W>(i, L, stage, stage_m, mine, wc);
}

// ---------------------------------------------------------------------------
// The persistent kernel.
// ---------------------------------------------------------------------------
// A wave's clock in rounds, over all its units.
struct RoundClock {
  uint32_t tick = 0;       // rounds started
  uint32_t next_look = 0;  // the tick of the next look for waiting waves
  bool fed = false;        // nobody waited at the last look
};

// The LDS stack of one wave while it searches a unit: entries [0, top), the
// oldest at 0.  NodeStack holds 4x4 nodes to expand (16-node rounds: Alg. 1's
// map, lane l expands node l/4 with move l%4), RingStack expanded nodes with
// the moves they have left (one move per lane and round; bpida_ring.h, 5x5:
// bpida_ring5.h).
constexpr int kCounterBytes = (sizeof(RunStats) + 15) / 16 * 16;
// The wave's counters take the last bytes of its 10 * CAP, except behind a
// 16-node stack too small to miss them, which is not bound by LDS either.
template <int CAP, int NPL>
constexpr bool counters_inside() {
  return NPL == 64 || CAP >= 1024;
}

template <int CAP>
struct NodeStack {
  static_assert((CAP & (CAP - 1)) == 0 && CAP >= 128, "stack");
  static constexpr int kCap = CAP - (counters_inside<CAP, 16>() ? kCounterBytes / 2 : 0), kNpl = 16;
  // largest growth of one round: a node has at most 3 children (its parent's
  // cell is excluded).  Only a root of the split (depth 0) has no parent and
  // may have 4, and a root is expanded in the unit's first round, which
  // starts from one chunk (at most 64 entries) and so cannot overflow.
  static constexpr int kGrow = 32;
  struct Entry {
    uint64_t s;
    uint16_t m;
  };
  uint64_t* st;
  uint16_t* sm;
  LaneMap M;
  int limit;

  __device__ __forceinline__ NodeStack(uint64_t* lds, int lim)
      : st(lds), sm((uint16_t*)(lds + CAP)), M(make_lane_map(lane_id())), limit(lim) {}
  __device__ __forceinline__ Entry get(uint32_t i) const { return {st[i], sm[i]}; }
  __device__ __forceinline__ void put(uint32_t i, Entry e) {
    st[i] = e.s;
    sm[i] = e.m;
  }
  // (u: the unit's instance and limit)
  __device__ __forceinline__ bool push(Unit u, Entry e, int count, RunStats& wc, int parts = 1) const {
    u.tile = e.s;
    u.meta = e.m;
    u.kind = kChunkNodes;
    u.count = count;
    return q_push(u, wc, parts);
  }
  __device__ __forceinline__ uint32_t round(uint32_t top, int kp, int& goals, int& fmin) {
    return bp_round<CAP>(st, sm, top, kp, limit, M, goals, fmin);
  }
  __device__ __forceinline__ uint32_t full_round(uint32_t top, uint64_t& gm, int& fmin) {
    int goals = 0;
    top = bp_round<CAP>(st, sm, top, kNpl, limit, M, goals, fmin);
    gm |= (uint64_t)goals;
    return top;
  }
  __device__ __forceinline__ uint32_t load(const Unit& u, uint64_t&, int&) {
    if (lane_id() < u.count) put((uint32_t)lane_id(), {u.tile, u.meta});
    WAVE_SYNC();
    return (uint32_t)u.count;
  }
};

// Bit of the moves that undo the move a node forbids (4: none).
template <uint32_t U, uint32_t L, uint32_t R, uint32_t D>
__device__ __forceinline__ uint32_t forbidden_bit(uint32_t fb) {
  return fb == 0 ? U : fb == 1 ? L : fb == 2 ? R : fb == 3 ? D : 0u;
}

template <int W, int CAP>
struct RingStack {
  static constexpr int kCap = CAP, kNpl = 64;
  static constexpr int kGrow = 64;  // an entry and its child replace an entry
  static constexpr uint32_t kTable = kRingEntry * CAP;
  struct Entry {
    uint32_t r, c, m;
  };
  Entry* st;
  RingConsts k;

  __device__ __forceinline__ RingStack(uint64_t* lds)
      : st((Entry*)lds), k(make_ring_consts<W>((char*)lds, kTable)) {}
  __device__ __forceinline__ Entry get(uint32_t i) const { return st[i]; }
  __device__ __forceinline__ void put(uint32_t i, Entry e) { st[i] = e; }
  __device__ __forceinline__ bool push(Unit u, Entry e, int count, RunStats& wc, int parts = 1) const {
    u.tile = (uint64_t)e.r | ((uint64_t)e.c << 32);
    u.meta = (uint16_t)ring_pack(e.m);
    u.kind = kChunkRing;
    u.count = count;
    return q_push(u, wc, parts);
  }
  __device__ __forceinline__ uint32_t round(uint32_t top, int kp, int& goals, int&) {
    uint64_t gm = 0;
    top = ring_round<W, kTable, false>(top, kp, gm, k);
    goals += __popcll(gm);
    return top;
  }
  __device__ __forceinline__ uint32_t full_round(uint32_t top, uint64_t& gm, int&) {
    return ring_round<W, kTable, true>(top, 64, gm, k);
  }

  // Loads a chunk: entries that are under way as they are; nodes are expanded
  // here (counted, tested for the goal, and stored if they keep a move).
  __device__ __forceinline__ uint32_t load(const Unit& u, uint64_t& expanded, int& goals) {
    const uint32_t lane = (uint32_t)lane_id();
    const uint64_t t = u.tile;
    const uint32_t meta = u.meta;
    uint32_t top = (uint32_t)u.count;
    if (u.kind == kChunkRing) {
      if (lane < top) put(lane, {(uint32_t)t, (uint32_t)(t >> 32), ring_unpack(meta)});
    } else {
      uint32_t r, c, b;
      ring_planes<W>(t, meta & 15u, &r, &c, &b);
      const uint32_t undo = forbidden_bit<kRingU, kRingL, kRingR, kRingD>((meta >> 5) & 7u);
      const uint32_t base = (b << 3) | ((meta >> 9) * kRingSlack1);
      const uint32_t near = ring_nearer(r, c, ring_compare<W>(b));
      const uint32_t m = ring_meta(base, near, ring_legal<W>(b), undo);
      expanded += (uint64_t)top;
      goals += __popcll(__builtin_amdgcn_ballot_w64(lane < top && t == (uint64_t)Board<W>::goal()));
      const uint64_t km = __builtin_amdgcn_ballot_w64(lane < top && m > kRingBase);
      const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(km >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
      if (lane < top && m > kRingBase) put(at, {r, c, m});
      top = (uint32_t)__popcll(km);
    }
    WAVE_SYNC();
    return top;
  }
};

template <int CAP>
struct RingStack<5, CAP> {
  static constexpr int kCap = CAP, kNpl = 64;
  static constexpr int kGrow = 64;
  static constexpr uint32_t kTable = (kR5Entry * CAP + 15u) & ~15u;
  struct Entry {
    R5Planes s;
    uint32_t m;
  };
  static_assert(sizeof(Entry) == kR5Entry, "entry");
  Entry* st;
  R5Consts k;

  __device__ __forceinline__ RingStack(uint64_t* lds) : st((Entry*)lds), k(make_r5_consts((char*)lds, kTable)) {}
  __device__ __forceinline__ Entry get(uint32_t i) const { return st[i]; }
  __device__ __forceinline__ void put(uint32_t i, Entry e) { st[i] = e; }
  __device__ __forceinline__ bool push(Unit u, Entry e, int count, RunStats& wc, int parts = 1) const {
    const unsigned __int128 s = r5_board(e.s, (e.m >> 4) & 31u);
    u.tile = (uint64_t)s;
    u.hi = (uint64_t)(s >> 64);
    u.meta = (uint16_t)r5_pack(e.m);
    u.kind = kChunkRing | kChunkWide;
    u.count = count;
    return q_push(u, wc, parts);
  }
  __device__ __forceinline__ uint32_t round(uint32_t top, int kp, int& goals, int&) {
    uint64_t gm = 0;
    top = r5_round<kTable, false>(top, kp, gm, k);
    goals += __popcll(gm);
    return top;
  }
  __device__ __forceinline__ uint32_t full_round(uint32_t top, uint64_t& gm, int&) {
    return r5_round<kTable, true>(top, 64, gm, k);
  }
  // As RingStack::load.
  __device__ __forceinline__ uint32_t load(const Unit& u, uint64_t& expanded, int& goals) {
    const uint32_t lane = (uint32_t)lane_id();
    const unsigned __int128 t = (unsigned __int128)u.tile | ((unsigned __int128)u.hi << 64);
    const uint32_t meta = u.meta;
    const bool ring = (u.kind & kChunkRing) != 0;
    uint32_t top = (uint32_t)u.count;
    // the blank's board cell: in the meta word, as a ring cell if under way
    const uint32_t c = meta & 31u, b = ring ? c - c / 6u : c;
    const R5Planes s = r5_planes(t, b);
    uint32_t m;
    if (ring) {
      m = r5_unpack(meta);
      if (lane < top) put(lane, {s, m});
    } else {
      const uint32_t rb = r5_cell(b);
      const uint32_t undo = forbidden_bit<kR5U, kR5L, kR5R, kR5D>((meta >> 5) & 7u);
      const uint32_t base = (rb << 4) | ((meta >> 9) * kR5Slack1);
      m = r5_meta(base, r5_nearer(s, r5_compare(rb, 0), r5_compare(rb, 1), r5_compare(rb, 2)), r5_legal(rb), undo);
      expanded += (uint64_t)top;
      goals += __popcll(__builtin_amdgcn_ballot_w64(lane < top && t == Board<5>::goal()));
      const uint64_t km = __builtin_amdgcn_ballot_w64(lane < top && m > kR5Base);
      const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(km >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
      if (lane < top && m > kR5Base) put(at, {s, m});
      top = (uint32_t)__popcll(km);
    }
    WAVE_SYNC();
    return top;
  }
};

// Moves stack entries [src, src + n) down to [dst, dst + n), dst < src, 64 at
// a time in ascending order: every entry is read before anything is written
// over it.
template <class ST>
__device__ __forceinline__ void stack_down(ST& S, uint32_t dst, uint32_t src, uint32_t n) {
  for (uint32_t i = 0; i < n; i += 64u) {
    const uint32_t k = i + (uint32_t)lane_id();
    if (k < n) S.put(dst + k, S.get(src + k));
  }
  WAVE_SYNC();
}

// The oldest entries of a stack of `avail` that a donation to `parts` (1 or 3)
// waves splits, and how many of them stay: every chunk takes at most the
// donated chunk's entries (half the two-way window), all together 64, a lane
// each.
__host__ __device__ constexpr int donation_window(int avail, int parts, int window) {
  const int most = parts == 1 ? window : (parts + 1) * (window / 2), lanes = 64 + 64 / parts;
  const int w = most < lanes ? most : lanes;
  return avail < w ? avail : w;
}
__host__ __device__ constexpr int donation_kept(int w, int parts) { return (w + parts) / (parts + 1); }
constexpr bool check_donation() {
  for (int chunk = 16; chunk <= 64; chunk *= 2)
    for (int parts = 1; parts <= 3; parts += 2)
      for (int avail = parts == 1 ? 2 : 64; avail <= 256; ++avail) {
        const int w = donation_window(avail, parts, 2 * chunk), keep = donation_kept(w, parts), give = w - keep;
        if (w > avail || give < parts || give > 64 || keep < 1 || keep > 64) return false;
        if (keep > chunk || (give + parts - 1) / parts > chunk) return false;
      }
  return true;
}
static_assert(check_donation(), "donated chunks");

// Searches one unit (the entries [0, top) of stack S) of an instance until
// its stack is empty: BPDFS rounds, with spills to the queue when LDS would
// overflow and donations to waiting workgroups.  Returns false if the time
// budget ran out (abandoned).
template <class ST, bool FS>
__device__ __forceinline__ bool run_unit(const Unit& u, ST& S, uint32_t top, RunStats& wc, RoundClock& clk,
                         uint64_t deadline, uint64_t& expanded, int& goals, int& fmin) {
  Args& A = fresh();
  using Entry = typename ST::Entry;
  constexpr int kCap = ST::kCap, kNpl = ST::kNpl, kGrow = ST::kGrow;
  const int lane = lane_id(), inst = u.inst;
  QueueCtl* q = A.q;
  constexpr uint32_t kLookMin = 32;  // rounds
  const int waves = (int)(gridDim.x * (blockDim.x >> 6));
  const float look_share = 4.0f * (float)(A.donate_mask + 1u) / (float)waves;
  const int dhigh = A.donate_min > 0 ? A.donate_min : min(4 * kNpl, kCap / 2);
  const int dlow = min(dhigh, A.donate_min > 0 ? A.donate_min : 2 * kNpl);
  uint32_t tick = clk.tick;
  // Entries taken from the bottom (spills, donations) make the rest move
  // down, so a position never wraps and a round addresses the stack without
  // a mask.
  if (FS) {
    if (goals > 0 && lane == 0) __hip_atomic_store(&A.is[inst].stop, 1, __ATOMIC_RELAXED, AGENT);
    if (goals > 0 || wave_bcast(lane == 0 ? ld_relaxed(&A.is[inst].stop) : 0)) top = 0;
  }
  while (top != 0) {
    int avail = (int)top;
    ++tick;
    const bool poll = (tick & 63u) == 0;
    if ((tick & 1023u) == 0) {
      // the time budget is spent, or work was dropped somewhere (every
      // count is void and the call reports BPIDA_ENOMEM): stop instead of
      // searching on
      const bool late = wall_clock64() > deadline;
      if (late || (!A.server && (ld_wave(&q->err) & kErrFatal))) {
        if (late && lane == 0) atomicOr(&q->err, 8);
        return false;
      }
    }
    if ((int32_t)(tick - clk.next_look) >= 0 && avail + kGrow <= kCap) {
      // Donation when workgroups wait on tickets no queued chunk covers: the
      // oldest min(window, avail) entries (the shallowest, largest subtrees)
      // are split alternately, so donor and receiver each keep about half.
      //
      // A look reads head and tail, which every push and take advances (or,
      // after one that found nobody waiting, `fed`, which changes seldom: 256
      // 5x5 states, which spill 17 chunks a microsecond, 63 -> 53 ms): all
      // waves together can afford a few dozen of those a microsecond.  So the
      // period is 4 * donate_every rounds while every wave searches (100 hard
      // 4x4 states: 25.5 ms with 512 rounds, 28.7 ms with 128, 44 ms with
      // 64), and shrinks with the share of waves that search, down to 32
      // rounds when few do (one hard 4x4 state: 3.1 ms at a fixed 512, 1.4 ms).
      // Donating from a shallow stack hands over pieces too small to pay for
      // the transfer, and a threshold the stack seldom reaches leaves subtrees
      // on one workgroup: four rounds' worth of pops, at most half the stack,
      // but two while more waves wait than search (64 easy states: 1.37 ms
      // with four throughout, 0.78 ms with two, 0.97 ms with one).
      if (avail < dlow) {
        clk.next_look = tick + kLookMin;
      } else {
        int64_t ht = 0;
        if (lane == 0 && !(clk.fed && ld_relaxed(&q->fed))) {
          ht = (int64_t)(ld_relaxed(&q->head) - ld_relaxed(&q->tail));
          if (ht <= 0 && !clk.fed) st_relaxed(&q->fed, 1);
        }
        const int wait = min(max(wave_bcast((int)ht), 0), waves);
        clk.fed = wait == 0;
        clk.next_look = tick + (uint32_t)max((int)kLookMin, (int)((float)(waves - wait) * look_share));
        const int dmin = wait > waves - wait ? dlow : dhigh;
        if (wait > 0 && avail >= dmin) {
          const int parts = avail >= 64 && wait >= 15 * (waves - wait) ? 3 : 1;
          const int w = donation_window(avail, parts, A.donate_window);
          const int keep_n = donation_kept(w, parts), h = w - keep_n;
          // (positions up to 127: inside the stack's storage, read for every lane)
          const uint32_t row = lane_over((uint32_t)lane, parts);
          const Entry give = S.get(row * (uint32_t)(parts + 1) + 1 + ((uint32_t)lane - row * (uint32_t)parts));
          const Entry keep = S.get(min((uint32_t)lane * (uint32_t)(parts + 1), 127u));
          WAVE_SYNC();
          if (lane == 0) __hip_atomic_fetch_add(&A.is[inst].outstanding, parts, __ATOMIC_RELAXED, AGENT);
          if (S.push(u, give, h, wc, parts)) {
            wc.pushes += (uint64_t)parts;
            wc.voluntary += 1;
            // the kept entries become the bottom, those above the window
            // close up behind them
            if (lane < keep_n) S.put(lane, keep);
            WAVE_SYNC();
            stack_down(S, (uint32_t)keep_n, (uint32_t)w, top - (uint32_t)w);
            top -= (uint32_t)h;
            avail -= h;
          } else if (lane == 0) {
            __hip_atomic_fetch_add(&A.is[inst].outstanding, -1, __ATOMIC_RELAXED, AGENT);
          }
        }
      }
    }
    if (avail + kGrow > kCap) {
      // LDS could overflow: move the oldest entries to the queue, 64 at a
      // time, until the largest round fits.
      do {
        const Entry e = S.get(lane);
        WAVE_SYNC();
        if (lane == 0) __hip_atomic_fetch_add(&A.is[inst].outstanding, 1, __ATOMIC_RELAXED, AGENT);
        if (S.push(u, e, 64, wc)) {
          wc.pushes += 1;
        } else if (lane == 0) {
          __hip_atomic_fetch_add(&A.is[inst].outstanding, -1, __ATOMIC_RELAXED, AGENT);
          __hip_atomic_store(&A.is[inst].lost, 1, __ATOMIC_RELAXED, AGENT);
          atomicOr(&q->err, 2);  // entries dropped: the call reports BPIDA_ENOMEM
        }
        stack_down(S, 0u, 64u, top - 64u);
        top -= 64u;
        avail -= 64;
      } while (avail + kGrow > kCap);
    }
    // uniform as the compiler may not know it to be: a stack top it takes for a
    // per-lane value moves the inner loop's bookkeeping to vector registers
    // (13 more vector instructions a round, 15 % of a 4x4 search)
    top = (uint32_t)wave_bcast((int)top);
    const int kp = min((int)top, kNpl);
    top = S.round(top, kp, goals, fmin);
    // the spill above keeps every round inside the stack; a round that ended
    // past it would have overwritten entries (reported, never silent)
    if (top > (uint32_t)kCap) atomicOr(&q->err, 32);  // every lane: a uniform branch
    expanded += (uint64_t)kp;
    if constexpr (FS) {
      // first-solution mode (Alg. 1 returns at its first goal): the unit that
      // expands a goal stops its instance; the others see the flag within 64
      // rounds and drop their stacks
      if (goals > 0) {
        if (lane == 0) __hip_atomic_store(&A.is[inst].stop, 1, __ATOMIC_RELAXED, AGENT);
        break;
      }
      if (poll && wave_bcast(lane == 0 ? ld_relaxed(&A.is[inst].stop) : 0))
        break;
    }
    {
      // Full rounds with nothing else to test: while the stack holds a round's
      // entries and has room for what they leave (the condition under which
      // the round above needs no spill) and no poll is due, full rounds
      // run back to back; their counts are added once at the end.  The
      // first-solution search also leaves after a round that expanded a goal
      // (a test of the wave's goal mask, uniform), and stops its instance
      // outside the loop.  (16-node rounds one at a time: 4096 uneven states
      // 5.2 s, back to back 3.0 s.)
      const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane(max(min((int)(63u - (tick & 63u)), (int)(clk.next_look - tick) - 1), 0));
      uint32_t r = 0;
      uint64_t gm = 0;  // nonzero: a round expanded a goal
      for (;;) {
        if (r >= n) break;
        if (top - (uint32_t)kNpl > (uint32_t)(kCap - kGrow - kNpl)) break;
        top = S.full_round(top, gm, fmin);
        ++r;
        if constexpr (FS) {
          if (gm != 0) break;
        }
      }
      if (gm != 0) goals += 1;
      tick += r;
      expanded += (uint64_t)kNpl * r;
      if constexpr (FS) {
        if (goals > 0) {
          if (lane == 0) __hip_atomic_store(&A.is[inst].stop, 1, __ATOMIC_RELAXED, AGENT);
          break;
        }
      }
    }
  }
  // 64-node rounds: a pruned child always has f = limit + 2,
  // and every limit below the optimum prunes one: below the optimum, a path
  // of approaching moves from a slack-0 node cannot reach the goal, so it
  // ends at a node whose remaining moves all go away and are pruned
  if (kNpl == 64) fmin = u.limit + 2;
  // (one round a tick: counted here, not in LDS every round; an abandoned
  // unit's are left out, its call fails)
  wc.rounds += tick - clk.tick;
  clk.tick = tick;
  return true;
}

// The persistent kernel.  A workgroup holds WPG independent waves (Sec. 5's
// block = one warp, WPG times over): each wave has its own stack and takes
// its own work, and no wave ever waits for another.  LDS per wave: 10 * CAP
// bytes, i.e. CAP nodes of a 16-node round (56 fewer from 1024 on), about 4/5
// CAP entries of the 3x3 and 4x4 64-node round, or a third of CAP of the 5x5
// one; a chunk carries its width.
//
// Waves per SIMD a one-wave workgroup's stack allows (LDS: 160 KB per compute
// unit).  The launch bound keeps the vector registers within that occupancy,
// capped at 6, for 16-node rounds at 5.  Those left alone take 135 to 151
// registers, 3 waves (4096 uneven states 6.4 s at 3 waves, 5.2 s at 5).  256 and
// 512 entries have room for 8 waves, but at 64 registers a wave spills 37 to
// 118 of them: at 8 against 6 waves 512 entries take 785 against 670 us for 64
// easy states (a quarter of the grid, as tuned: 405 against 389), 540 against
// 480 for 2048 3x3, 2.5 against 2.3 ms for 1000 easy, 33.9 against 32.9 for 100
// hard; only batches that keep every wave busy gain (777 uneven: 89.7 against
// 95.7 ms).
template <int CAP, int NPL>
constexpr int batch_waves_per_simd() {
  constexpr int w = (int)(163840u / (10u * CAP)) / 4, most = NPL == 64 ? 6 : 5;
  return w > most ? most : w < 1 ? 1 : w;
}
template <int CAP>
constexpr int ring_cap() {
  return (CAP * 10 - (int)kRingTable - kCounterBytes) / 12 / 16 * 16;
}
template <int CAP>
constexpr int ring5_cap() {
  return (CAP * 10 - (int)kR5Table - kCounterBytes) / 28 / 16 * 16;
}

template <int CAP, int NPL, int WPG, bool FS, int W>
__global__ __launch_bounds__(64 * WPG, (batch_waves_per_simd<CAP, NPL>()))
void batch4_kernel(std::conditional_t<W == 0, ServerBatchArgs, BatchArgs>) {
  Args& A = fresh();
  static_assert(CAP % 16 == 0 && (NPL == 64 || (CAP & (CAP - 1)) == 0), "stack size");
  static_assert(NPL == 16 || NPL == 64, "nodes per round");
  static_assert(NPL == 16 || CAP >= 256, "stack too small for 64-node rounds");
  static_assert(WPG == 1 || WPG == 2 || WPG == 4, "waves per workgroup");
  // u64 words of one wave's stack and counters: in registers these cost 22
  // scalar registers the search loop has better uses for (it spilled 40 to 190
  // vector registers around them)
  constexpr int kWords = 10 * CAP / 8 + (counters_inside<CAP, NPL>() ? 0 : kCounterBytes / 8);
  __shared__ __attribute__((aligned(16))) uint64_t lds[WPG * kWords];
  uint64_t* st = lds + (WPG == 1 ? 0 : (int)(threadIdx.x >> 6) * kWords);
  uint16_t* sm = (uint16_t*)(st + CAP);  // staging of the seeds' meta words
  const int lane = lane_id();
  QueueCtl* q = A.q;

  if (W == 0 && A.server) {
    int role = 0;
    if (lane == 0) role = atomicCAS(fresh_server().admitter, 0, 1) == 0;
    if (wave_bcast(role)) {
      admitter_loop(st, sm, wall_clock64() + A.budget_ticks);
      RunStats none = {};
      none.t_first = ~0ull;
      if (lane == 0) A.wave_stats[blockIdx.x * WPG + (WPG == 1 ? 0 : threadIdx.x >> 6)] = none;
      return;
    }
  }

  Unit u;  // the chunk to search next (count 0: none)
  // (every lane writes the same values to the same words)
  RunStats& wc = *(RunStats*)(st + kWords - kCounterBytes / 8);
  wc = RunStats{};
  wc.t_first = wall_clock64();

  // Seed the first limit of every instance through a shared cursor: all
  // instances are seeded by workgroups that are running, whatever part of
  // the grid is resident.  A wave searches the last chunk it seeded itself.
  // The cursor is read before it is advanced: thousands of waves that
  // advance it past the end hold up the few that search.
  for (;;) {
    int i = A.n;
    if (lane == 0 && ld_relaxed(&q->seed_next) < A.n)
      i = __hip_atomic_fetch_add(&q->seed_next, 1, __ATOMIC_RELAXED, AGENT);
    i = wave_bcast(i);
    if (i >= A.n) break;
    if (ld_wave(&q->err) & kErrFatal) break;  // work already lost: stop seeding
    if (A.is[i].done != 0) {  // nothing to search
      int left = 1;
      if (lane == 0) left = __hip_atomic_fetch_add(&q->remaining, -1, __ATOMIC_RELAXED, AGENT) - 1;
      if (wave_bcast(left) == 0) end_search();
      continue;
    }
    if (u.count && !q_push(u, wc)) drop_units(u.inst, 1, 1);
    const int L = A.is[i].limit;
    if (seed_limit<W>(i, L, 0, st, sm, u, wc)) complete_limit<W>(i, L, st, sm, u, wc);
  }

  uint64_t t_mark = wall_clock64();
  bool idle = false;
  uint64_t idle_since = 0, idle_act = 0;
  RoundClock clk;
  uint32_t polls = 0;
  uint64_t ticket = kNoTicket;  // consumer ticket held while idle
  const uint64_t deadline = wall_clock64() + A.budget_ticks;

  for (;;) {
    if (u.count == 0) {
      const int got = q_take(ticket, u, wc);
      if (got < 0) break;
      if (got == 0) {
        // Wait.  The ticket's own slot is all that is polled, with longer
        // sleeps up to 2048 clocks; the shared words (end of the search,
        // lost work, queue activity) are read every 32nd time only: thousands
        // of waiting waves that read them on every poll held up the searching
        // waves' looks at head and tail by some 25 us each.
        if (!idle) {
          idle = true;
          polls = 0;
          idle_since = 0;
        }
        ++polls;
        if ((polls == 8 || (polls & 31u) == 0) && lane == 0 && ld_relaxed(&q->fed)) st_relaxed(&q->fed, 0);
        if ((polls & 31u) == 0) {
          if (ld_wave(&q->remaining) <= 0) break;
          if (!A.server && (ld_wave(&q->err) & kErrFatal)) break;
          const uint64_t now = wall_clock64();
          // queue activity seen by this idle workgroup (lane 0's view)
          uint64_t act = 0;
          if (lane == 0) act = ld_relaxed(&q->head) + ld_relaxed(&q->tail);
          act = (uint64_t)(uint32_t)wave_bcast((int)(uint32_t)act);
          if (idle_since == 0 || act != idle_act) {
            idle_since = now;  // the queue moved: work is being shared
            idle_act = act;
          } else if (now - idle_since > A.idle_ticks || now > deadline) {
            // no queue activity for the whole watchdog period although
            // instances remain, or the run's time budget is spent
            if (lane == 0) atomicOr(&q->err, now > deadline ? 8 : 4);
            break;
          }
          wc.t_idle += now - t_mark;
          t_mark = now;
        }
        if (polls < 8) __builtin_amdgcn_s_sleep(4);
        else __builtin_amdgcn_s_sleep(32);
        continue;
      }
      wc.pops += 1;
    }
    idle = false;
    {
      const uint64_t now = wall_clock64();
      wc.t_queue += now - t_mark;
      t_mark = now;
    }
    uint64_t expanded = 0;
    int goals = 0, fmin = INT_MAX;
    bool ok = true;
    if (W ? W == 5 : u.width == 5) {
      // (smaller stacks take no 5x5 batch: the host refuses it)
      if constexpr (CAP / 2 >= 512 && (W == 0 || W == 5)) {
        RingStack<5, ring5_cap<CAP>()> S(st);
        const uint32_t top = S.load(u, expanded, goals);
        ok = run_unit<RingStack<5, ring5_cap<CAP>()>, FS>(u, S, top, wc, clk, deadline, expanded, goals, fmin);
      }
    } else if (W ? W == 3 : u.width == 3) {
      if constexpr (CAP >= 256 && (W == 0 || W == 3)) {
        RingStack<3, ring_cap<CAP>()> S(st);
        const uint32_t top = S.load(u, expanded, goals);
        ok = run_unit<RingStack<3, ring_cap<CAP>()>, FS>(u, S, top, wc, clk, deadline, expanded, goals,
                                                         fmin);
      }
    } else if constexpr (W == 3 || W == 5) {
    } else if constexpr (NPL == 64) {
      RingStack<4, ring_cap<CAP>()> S(st);
      const uint32_t top = S.load(u, expanded, goals);
      ok = run_unit<RingStack<4, ring_cap<CAP>()>, FS>(u, S, top, wc, clk, deadline, expanded, goals,
                                                       fmin);
    } else {
      NodeStack<CAP> S(st, u.limit);
      const uint32_t top = S.load(u, expanded, goals);
      ok = run_unit<NodeStack<CAP>, FS>(u, S, top, wc, clk, deadline, expanded, goals, fmin);
    }
    if (!ok) break;
    const uint64_t now = wall_clock64();
    wc.t_work += now - t_mark;
    t_mark = now;
    wc.searched += expanded;
    release_unit<W>(u.inst, u.limit, expanded, goals, fmin, st, sm, u, wc);
  }
  wc.t_last = wall_clock64();
  if (lane == 0 && A.wave_stats) A.wave_stats[blockIdx.x * WPG + (WPG == 1 ? 0 : threadIdx.x >> 6)] = wc;
}

// ---------------------------------------------------------------------------
// After the search, in one launch.  Workgroup 0 (with F.out) sums the waves'
// counters.  The others: per-instance status, 1 solved, < 0 a bpida_status (a
// queue that overflowed marks every instance: its dropped work invalidates
// every count; a watchdog or deadline stop marks the unfinished ones), and the
// outputs' copies for the host.  A call that waits reads statuses, counters
// and, for small batches, outputs from pinned memory that this kernel wrote:
// each copy by the runtime instead took 25 to 50 us.
// ---------------------------------------------------------------------------
constexpr int kFinishThreads = 512;
__device__ __forceinline__ uint64_t stat_join(int k, uint64_t a, uint64_t b) {
  if (k == offsetof(RunStats, t_first) / 8) return min(a, b);
  if (k == offsetof(RunStats, qmax) / 8 || k == offsetof(RunStats, t_last) / 8) return max(a, b);
  return a + b;
}
__global__ __launch_bounds__(kFinishThreads) void batch_finish_kernel(FinishArgs F) {
  const int tid = threadIdx.x;
  int block = (int)blockIdx.x;
  if (F.out && block-- == 0) {
    __shared__ uint64_t part[kFinishThreads / 64][kRunStats];
    uint64_t sum[kRunStats] = {};
    sum[offsetof(RunStats, t_first) / 8] = ~0ull;
    for (int i = tid; i < F.waves; i += kFinishThreads) {
      uint64_t v[kRunStats];
      for (int k = 0; k < kRunStats; ++k) v[k] = ((const uint64_t*)(F.wave_stats + i))[k];
      for (int k = 0; k < kRunStats; ++k) sum[k] = stat_join(k, sum[k], v[k]);
    }
    for (int k = 0; k < kRunStats; ++k) {
      for (int o = 32; o > 0; o >>= 1) sum[k] = stat_join(k, sum[k], __shfl_xor(sum[k], o, 64));
      if ((tid & 63) == 0) part[tid >> 6][k] = sum[k];
    }
    __syncthreads();
    if (tid < kRunStats) {
      uint64_t s = part[0][tid];
      for (int j = 1; j < kFinishThreads / 64; ++j) s = stat_join(tid, s, part[j][tid]);
      ((uint64_t*)&F.out->sum)[tid] = s;
    }
    if (tid == 0) F.out->err = F.q->err;
    return;
  }
  const int64_t at = (int64_t)block * kFinishThreads + tid;
  if (at < F.n) {
    const int32_t done = F.is[at].done;
    int32_t v = done;
    if (F.q->err & kErrFatal) v = -4;  // BPIDA_ENOMEM
    else if (F.q->err & 32) v = -6;    // LDS stack overrun: BPIDA_EINTERNAL
    else if (done == 0) v = -6;        // stopped by the watchdog or the deadline
    F.status[at] = v;
    if (F.host_len) F.host_len[at] = F.len[at];
  }
  if (F.host_nodes && at < (int64_t)F.n * 64) F.host_nodes[at] = F.nodes[at];
}

hipError_t launch_batch_finish(const FinishArgs& F, hipStream_t s) {
  const int64_t work = !F.is ? 0 : F.host_nodes ? (int64_t)F.n * 64 : F.n;
  const int64_t blocks = (F.out ? 1 : 0) + (work + kFinishThreads - 1) / kFinishThreads;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(batch_finish_kernel, dim3((unsigned)blocks), dim3(kFinishThreads), 0, s, F);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Before the search, in one launch: ingest, root split and state of every
// instance, its output row, the queue's slots and control block.
// ---------------------------------------------------------------------------

// Validates (a permutation of 0..w*w-1 whose parity matches the blank's
// distance from cell 0), packs and measures the state at s with one wave:
// lane p takes cell p.
__device__ __forceinline__ InstW wave_ingest(const uint8_t* __restrict__ s, int w) {
  const int lane = lane_id();
  const int nn = w * w, bits = w == 5 ? 5 : 4;
  const bool on = lane < nn;
  const uint32_t v = on ? (uint32_t)s[lane] : 0xFFu;
  const bool fits = on && v < (uint32_t)nn;
  uint32_t seen = fits ? 1u << v : 0u, inv = 0;
  for (int p = 0; p < 25; ++p) inv += (p > lane && p < nn && (uint32_t)__builtin_amdgcn_readlane((int)v, p) < v) ? 1u : 0u;
  if (!on) inv = 0;
  int h = 0;
  if (fits && v != 0) {
    const int dr = lane / w - (int)v / w, dc = lane % w - (int)v % w;
    h = (dr < 0 ? -dr : dr) + (dc < 0 ? -dc : dc);
  }
  const unsigned __int128 word = on ? (unsigned __int128)(v & 31u) << (bits * lane) : 0;
  uint64_t lo = (uint64_t)word, hi = (uint64_t)(word >> 64);
  for (int o = 32; o > 0; o >>= 1) {
    seen |= (uint32_t)__shfl_xor((int)seen, o, 64);
    inv += (uint32_t)__shfl_xor((int)inv, o, 64);
    h += __shfl_xor(h, o, 64);
    lo |= __shfl_xor(lo, o, 64);
    hi |= __shfl_xor(hi, o, 64);
  }
  const uint64_t blank_m = __builtin_amdgcn_ballot_w64(on && v == 0);
  InstW r;
  r.lo = 0;
  r.hi = 0;
  r.blank = 0;
  r.h0 = 0;
  r.status = -1;  // BPIDA_EINVAL
  r.width = w;
  if (seen == (1u << nn) - 1u) {  // nn cells with nn different tiles
    r.blank = (int)__builtin_ctzll(blank_m);
    const uint32_t bpar = (uint32_t)(r.blank / w + r.blank % w) & 1u;
    r.status = (inv & 1u) == bpar ? 0 : -2;  // BPIDA_EUNSOLVABLE
    r.lo = lo;
    r.hi = hi;
    r.h0 = h;
  }
  return r;
}

constexpr int kSplitThreadsW = 256;

// The parent-pruned tree of one instance to depth D, level after level
// (CreateRootSet, no duplicate elimination); the workgroup's instance has
// width W and its start may not make move fb0 first (4: any move).  Level
// sizes come from the walk-count table of that width.
template <int W>
__device__ void split_impl(const InstW& I, int fb0, int depth, const int32_t* walks, NodeW* base,
                           uint32_t* h_lds, int32_t* fill, int32_t* gmin, int32_t* bad,
                           int64_t* lvl_out) {
  using B = Board<W>;
  using S = typename B::S;
  const int32_t* lc = walks + walk_row(I.blank, fb0);
  if (threadIdx.x == 0) {
    NodeW r;
    r.lo = I.lo;
    r.hi = I.hi;
    r.meta = node_meta(I.blank, fb0, 0, I.h0);
    r.f = (uint32_t)I.h0;
    base[0] = r;
  }
  __syncthreads();
  int64_t lvl = 0;
  for (int d = 0; d < depth; ++d) {
    const int cnt = lc[d];
    const int64_t next = lvl + cnt;
    for (int k = threadIdx.x; k < cnt; k += kSplitThreadsW) {
      const NodeW nd = base[lvl + k];
      S s = (S)nd.lo;
      if constexpr (W == 5) s |= (S)nd.hi << 64;
      const uint32_t b = nd.meta & 31u, fb = (nd.meta >> 5) & 7u;
      const int g = (int)((nd.meta >> 8) & 255u), h = (int)((nd.meta >> 16) & 255u);
      atomicAdd(&h_lds[min(g + h, kHistBins - 1)], 1u);
      if (s == B::goal()) atomicMin(gmin, g);
      const uint32_t lm = B::legal(b) & ~(1u << fb);
      for (int a = 0; a < 4; ++a) {
        if (!((lm >> a) & 1u)) continue;
        const int delta = a == 0 ? -W : a == 1 ? -1 : a == 2 ? 1 : W;
        const uint32_t nn = b + (uint32_t)delta;
        const uint32_t t = (uint32_t)(s >> (B::BITS * nn)) & B::MASK;
        const bool vert = a == 0 || a == 3;
        const uint32_t ct = vert ? t / W : t % W, cn = vert ? nn / W : nn % W;
        const int up = (int)((B::table(a) >> (ct * W + cn)) & 1u);
        const int h2 = h + (up ? 1 : -1);
        const S cs = s + ((S)t << (B::BITS * b)) - ((S)t << (B::BITS * nn));
        NodeW c;
        c.lo = (uint64_t)cs;
        c.hi = W == 5 ? (uint64_t)((unsigned __int128)cs >> 64) : 0ull;
        c.meta = node_meta((int)nn, 3 - a, g + 1, h2);
        c.f = (uint32_t)(g + 1 + h2);
        const int slot = atomicAdd(fill, 1);
        if (slot < lc[d + 1]) base[next + slot] = c;
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      if (*fill != lc[d + 1]) *bad = 1;
      *fill = 0;
    }
    lvl = next;
    __syncthreads();
  }
  *lvl_out = lvl;
}

// Workgroups 0..n-1 take an instance each, the others the queue (kPrepSlots
// slots a thread).  The instance's split-tree region is tree_off[i] (or
// i * stride); `forbid` (null: none) = per instance the move its start may
// not make first (4: any).
constexpr int kPrepSlots = 4;
__global__ __launch_bounds__(kSplitThreadsW) void batch_prep_kernel(BatchArgs A, PrepArgs P) {
  const int i = blockIdx.x;
  const int tid = threadIdx.x;
  if (i >= A.n) {
    const int64_t k0 = ((int64_t)(i - A.n) * kSplitThreadsW + tid) * kPrepSlots;
    for (int64_t k = k0; k < k0 + kPrepSlots && k <= (int64_t)A.qmask; ++k) {
      A.seq[k].seq = 4 * (uint64_t)k;
      A.seq[k].abandoned = 0;
    }
    if (i == A.n) {
      for (int k = tid; k < (int)(sizeof(QueueCtl) / 4); k += kSplitThreadsW) ((uint32_t*)A.q)[k] = 0;
      __syncthreads();
      if (tid == 0) A.q->remaining = A.n;
    }
    return;
  }
  __shared__ InstW I;
  __shared__ uint32_t h_lds[kHistBins];
  __shared__ int32_t fill, gmin, bad;
  if (tid < 64) {
    const int w = P.widths ? P.widths[i] : P.width;
    const InstW v = wave_ingest(P.states + (P.byte_off ? P.byte_off[i] : (int64_t)i * w * w), w);
    if (tid == 0) {
      I = v;
      gmin = INT_MAX;
      fill = 0;
      bad = 0;
      A.out_len[i] = -1;
    }
    A.out_nodes[(size_t)i * 64 + tid] = 0;
  }
  for (int k = tid; k < kHistBins; k += kSplitThreadsW) h_lds[k] = 0;
  __syncthreads();
  const int fb0 = P.forbid ? min((int)P.forbid[i], 4) : 4;
  const int64_t region = P.tree_off ? P.tree_off[i] : (int64_t)i * P.stride;
  NodeW* base = const_cast<NodeW*>(A.tree) + region;
  const int32_t* wk = P.walks + (size_t)(I.width - 3) * kWalkStride;
  int64_t lvl = 0;
  if (I.status == 0) {
    if (I.width == 3) split_impl<3>(I, fb0, P.depth, wk, base, h_lds, &fill, &gmin, &bad, &lvl);
    else if (I.width == 4) split_impl<4>(I, fb0, P.depth, wk, base, h_lds, &fill, &gmin, &bad, &lvl);
    else split_impl<5>(I, fb0, P.depth, wk, base, h_lds, &fill, &gmin, &bad, &lvl);
  }
  for (int k = tid; k < kHistBins; k += kSplitThreadsW)
    const_cast<uint32_t*>(A.hist)[(size_t)i * kHistBins + k] = h_lds[k];
  if (tid == 0) {
    const_cast<int32_t*>(A.goal_g)[i] = gmin;
    InstState S;
    S.limit = first_limit(I.h0, A.start_limit);
    S.col = (S.limit - I.h0) / 2;
    S.done = I.status;  // 0 = to search
    if (A.exact_limit) {
      // one limit only: a limit below h0 or of the other parity has no path
      // of exactly that length
      S.limit = A.exact_limit[i];
      S.col = 0;
      if (S.done == 0 && (S.limit < I.h0 || ((S.limit - I.h0) & 1))) S.done = 2;
    }
    S.outstanding = 0;
    S.nodes = 0;
    S.fmin = INT_MAX;
    S.goals = 0;
    S.stop = 0;
    S.lost = 0;
    S.root_off = region + lvl;
    S.nroots = I.status == 0 ? wk[walk_row(I.blank, fb0) + P.depth] : 0;
    S.width = I.width;
    if (S.done == 0 && (S.limit > A.max_limit || S.col >= 64)) S.done = -3;  // BPIDA_ELIMIT
    if (bad) S.done = -6;                                                    // BPIDA_EINTERNAL
    A.is[i] = S;
  }
}

hipError_t launch_batch_prep(const BatchArgs& A, const PrepArgs& P, hipStream_t s) {
  const int64_t per = (int64_t)kSplitThreadsW * kPrepSlots;
  const int64_t blocks = A.n + ((int64_t)A.qmask + per) / per;
  hipLaunchKernelGGL(batch_prep_kernel, dim3((unsigned)blocks), dim3(kSplitThreadsW), 0, s, A, P);
  return hipGetLastError();
}

// Server set-up: queue sequence numbers, free instance slots, one sentinel in
// `remaining` (cleared by the admitter when the server shuts down).
__global__ void server_setup_kernel(BatchArgs A, ServerArgs V) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k <= (int64_t)A.qmask) {
    A.seq[k].seq = 4 * (uint64_t)k;
    A.seq[k].abandoned = 0;
  }
  if (k < V.slots) V.busy[k] = 0;
  if (k == 0) {
    A.q->remaining = 1;
    *V.admitter = 0;
    *V.in_flight = 0;
  }
}

hipError_t launch_server_setup(const BatchArgs& A, const ServerArgs& V, hipStream_t s) {
  const int64_t work = std::max<int64_t>((int64_t)A.qmask + 1, V.slots);
  hipLaunchKernelGGL(server_setup_kernel, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, s, A, V);
  return hipGetLastError();
}

// The first-solution search is a kernel of its own: with both unit loops in
// one kernel the register allocation of each suffers.  So is, for 64-node
// rounds of single-wave workgroups, the search of a batch of one width (W; 0:
// any, by chunk, and the server): with the rounds of all three widths and the
// admitter in one kernel it is 56 KB of code against 25, and a 640-entry
// 4x4 stack's wave spills 136 bytes against 52 (batch of 100 hard states 25.8
// -> 24.0 ms, 3x3 batch of 2048 367 -> 351 us).  The
// server's arguments go to the general kernel alone: with them 256 bytes
// long (and 256 hidden ones), the others' made an easy state from host
// buffers take 252 us on average against 241, and 264 bytes 5 to 10 us more.
template <int CAP, int NPL, int WPG, int W>
static hipError_t launch_batch_t(int grid, const BatchArgs& A, hipStream_t s, const ServerArgs* srv = nullptr) {
  std::conditional_t<W == 0, ServerBatchArgs, BatchArgs> K;
  if constexpr (W == 0) K = ServerBatchArgs{A, srv ? *srv : ServerArgs{}};
  else K = A;
  if (A.first_solution)
    hipLaunchKernelGGL((batch4_kernel<CAP, NPL, WPG, true, W>), dim3(grid), dim3(64 * WPG), 0, s, K);
  else
    hipLaunchKernelGGL((batch4_kernel<CAP, NPL, WPG, false, W>), dim3(grid), dim3(64 * WPG), 0, s, K);
  return hipGetLastError();
}

template <int CAP, int NPL, int WPG>
static hipError_t launch_batch_w(int width, int grid, const BatchArgs& A, hipStream_t s, const ServerArgs* srv) {
  if constexpr (NPL == 64 && WPG == 1) {
    // (smaller stacks take no batch of that width: the host refuses it)
    if (width == 3) return launch_batch_t<CAP, NPL, WPG, 3>(grid, A, s);
    if constexpr (CAP >= 512)
      if (width == 4) return launch_batch_t<CAP, NPL, WPG, 4>(grid, A, s);
    if constexpr (CAP >= 1024)
      if (width == 5) return launch_batch_t<CAP, NPL, WPG, 5>(grid, A, s);
  }
  return launch_batch_t<CAP, NPL, WPG, 0>(grid, A, s, srv);
}

template <int CAP, int NPL, int WPG>
static int occupancy_t() {
  // (asked once: it does not change, every call needs it, and each of the two
  // queries takes some 5 us; the callers hold the library's lock)
  static int known = -1;
  if (known >= 0) return known;
  int nb = 0, nf = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, batch4_kernel<CAP, NPL, WPG, false, 0>, 64 * WPG, 0) !=
          hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&nf, batch4_kernel<CAP, NPL, WPG, true, 0>, 64 * WPG, 0) !=
          hipSuccess)
    return 0;
  known = nb < nf ? nb : nf;  // the grid suits either kernel
  return known;
}

// Supported (stack capacity, nodes per round, waves per workgroup) triples.
#define BATCH_CONFIGS(X)                                                                         \
  X(128, 16, 1) X(256, 16, 1) X(512, 16, 1) X(1024, 16, 1) X(2048, 16, 1) X(256, 64, 1)          \
  X(512, 64, 1) X(640, 64, 1) X(672, 64, 1) X(768, 64, 1) X(1024, 64, 1) X(2048, 64, 1)    \
  X(512, 64, 2) X(1024, 64, 2) X(2048, 64, 2)                                                     \
  X(512, 64, 4) X(1024, 64, 4) X(2048, 64, 4)

hipError_t launch_batch4(int lds_cap, int npl, int wpg, int width, int grid, const BatchArgs& A, hipStream_t s,
                         const ServerArgs* srv) {
  if (grid <= 0) return hipSuccess;
#define X(C, N, G) \
  if (lds_cap == C && npl == N && wpg == G) return launch_batch_w<C, N, G>(width, grid, A, s, srv);
  BATCH_CONFIGS(X)
#undef X
  return hipErrorInvalidValue;
}

int batch4_max_blocks_per_cu(int lds_cap, int npl, int wpg) {
#define X(C, N, G) \
  if (lds_cap == C && npl == N && wpg == G) return occupancy_t<C, N, G>();
  BATCH_CONFIGS(X)
#undef X
  return 0;
}

}  // namespace bpida
