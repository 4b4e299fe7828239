// gpuos_kernels.hip -- device side of the GPUOS hot path for gfx950 (CDNA4).
//
//  * gpuos_worker_kernel: the persistent kernel (paper Section 4.1 "Persistent
//    Kernel Executor", device loop of Section 4.2).  Workgroup 0 is the
//    dispatcher: it is the single reader of the host ring (one PCIe poller
//    instead of hundreds), mirrors new records into device memory, resolves
//    each task's operator-table slot and version once ("claim time"), expands
//    tasks into work units (chunks) and publishes each with one 8-byte store
//    whose stamp makes it claimable (a lone new record takes the first
//    wavefront's short cut past the batch pass).  Every other workgroup is a
//    worker (run_worker in gpuos_device.h): its first wavefront claims work
//    units with an atomic fetch-add and holds up to eight descriptors, running
//    whichever is ready; the 4 wavefronts of the workgroup execute a chunk
//    together, and the last finisher of a task publishes its completion
//    (device-side done word for dependants, one 8-byte completion word to host
//    memory).
//  * gpuos_single_task_kernel: the same chunk executor as an ordinary kernel,
//    one launch per task (the per-op-launch comparison of the paper's Section 6).
//
// Wavefronts are 64 lanes; a workgroup is 256 threads.  Nothing here is a dense
// contraction, so there is no MFMA: the paths are bandwidth- or latency-bound
// and use 16-byte-per-lane global accesses, LDS for descriptor broadcast and
// cross-wave combines, and DPP / permute wave reductions.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "../../include/gpuos.h"
#include "gpuos_internal.h"
#include "gpuos_device.h"

namespace gpuos {

// ---------------------------------------------------------------------------
// dispatcher (workgroup 0)
//
// Besides mirroring the host ring it is the scheduler of dependent work.  Units are claimed in
// publication order; a workgroup holds a few units at a time and runs whichever of them is ready, and
// when none is it can only wait.  Two rules keep that from hurting:
//  * A task with more than kSmallTaskChunks chunks whose dependencies are incomplete when it is
//    dequeued is HELD on a pending list and published when the done words say so (otherwise hundreds
//    of descriptor slots would be taken by it while ready work of other chains sits behind it).  Small
//    dependent tasks are published at once and wait, in the workgroups that claimed their units, on the
//    done word: the shortest hand-off for sequential chains of small operations.
//  * Publication order respects dependency order: a task that names a task which is itself not yet
//    published (it is on the pending list, or held earlier in the same pass) is held too, whatever its
//    size.  So whatever a waiting worker waits for lies BEFORE its own unit in the unit ring, its units
//    were claimed earlier by resident workgroups, and by induction over the ring position the wait
//    ends.  (Without this rule a held large task followed by more small dependants than the workgroups
//    can hold parks every workgroup behind units that come after theirs.)
// Held tasks are flagged RF_DEPS_RESOLVED: they are published only after their dependencies
// completed, so their workers never wait.
// ---------------------------------------------------------------------------
constexpr uint32_t kPendMax = 128;         // tasks held back at a time
constexpr uint64_t kLookaheadUnits = 8192; // work units kept published ahead of the claim counter
constexpr uint32_t kPrefetch = 4;          // records read together with every doorbell poll (4 x 16 lanes)
constexpr uint32_t kStageRetries = 4096;   // re-reads of a record that fails its check word (~ms) before it is failed

struct PubEntry {                          // what it takes to publish a task's work units
  uint32_t slot;
  uint32_t nchunks;
  uint32_t opinfo;                         // op id | table slot << 8 | valid << 9 | lap of the ticket (10 bits) << 16
  uint32_t route;                          // 0: main unit ring; 1: the second ring, served by the run-time kernel
};
struct PendEntry {
  uint64_t ticket;
  PubEntry pub;
  uint16_t dep[3];
  uint16_t run;                            // tickets it stands for: this one and the links that run with it (>= 1)
};

// A staged record with a pitch of 68 words instead of 64: when the 64 lanes of a wavefront read the
// same field of 64 different records (the resolve and split steps do little else), a pitch of 64
// words puts all of them on one LDS bank; with 68 they spread over 16.
struct alignas(16) StagedRecord : Record {
  uint32_t pitch_pad[4];
};
static_assert(sizeof(StagedRecord) == 272, "staging pitch");

struct DispShared {
  StagedRecord rec[kDispatchBatch];        // 17 KB staging of the batch being mirrored
  uint64_t entry[GPUOS_MAX_OPS];           // shadow of the device table: current {impl, version}
  PubEntry pub[kDispatchBatch];            // tasks whose units are published in this pass (<= 64)
  uint32_t ubeg[kDispatchBatch + 1];       // exclusive prefix of their nchunks
  PendEntry pend[kPendMax];
  uint32_t ok[kDispatchBatch];             // staging: record passed its check on this read
  uint32_t pre[kPrefetch];                 // prefetched with the poll and valid
  uint32_t preok[kDispatchBatch];          // requested while the previous batch was written out: arrived whole
  uint32_t opcnt[GPUOS_MAX_OPS];           // tracing: tasks dispatched per operator since the last flush
  uint32_t ready[kPendMax];                // per pending entry: dependencies complete
  uint32_t native[GPUOS_MAX_PROGRAMS];     // per operator program: 1 = its tasks go to the second ring (native code is being served there)
  uint64_t tail, epoch_word;
  uint32_t npend, npub, npub_second;
  uint64_t claimed;                        // last value read from the claim counter
  uint64_t lane_tickets, lane_units;       // what the first wavefront's short cut for lone tasks has dispatched / published
  uint32_t lane_counted;                   // ... and whether it counted an operator (tracing)
};


DEV void dispatcher_refresh_native(const WorkerArgs& a, DispShared* s) {
  // which programs a run-time kernel serves natively, and which generation of it is wanted
  // (the host changes both only between two epoch bumps, and waits in between)
  const uint32_t tid = threadIdx.x;
  if (tid < GPUOS_MAX_PROGRAMS)
    s->native[tid] = (a.units_j != nullptr && a.progs != nullptr)
                         ? __hip_atomic_load(&a.progs[tid].native, __ATOMIC_RELAXED, SC_SYSTEM) : 0u;
  if (tid == GPUOS_MAX_PROGRAMS) {
    const uint32_t g = __hip_atomic_load(&a.bell->jit_gen, __ATOMIC_RELAXED, SC_SYSTEM);
    __hip_atomic_store(&a.d->jit_gen, g, __ATOMIC_RELAXED, SC_SYSTEM);
  }
}

DEV void dispatcher_refresh_table(const WorkerArgs& a, DispShared* s, uint32_t only_op) {
  // copy entries host table -> device table with the dual-slot protocol: the
  // inactive slot is written first, then the version is published.
  for (uint32_t op = threadIdx.x; op < GPUOS_MAX_OPS; op += kThreads) {
    if (only_op != 0xffu && op != only_op) continue;
    const uint32_t ver = __hip_atomic_load(&a.htable[op].version, __ATOMIC_RELAXED, SC_SYSTEM);
    if (ver == 0) continue;
    order_loads();
    const uint64_t e = __hip_atomic_load(&a.htable[op].slot[ver & 1u], __ATOMIC_RELAXED, SC_SYSTEM);
    if (e == s->entry[op]) continue;
    const uint32_t ev = (uint32_t)(e >> 32);
    __hip_atomic_store(&a.dtable[op].slot[ev & 1u], e, __ATOMIC_RELAXED, SC_SYSTEM);
    drain_stores();
    __hip_atomic_store(&a.dtable[op].version, ev, __ATOMIC_RELAXED, SC_SYSTEM);
    s->entry[op] = e;
  }
}

DEV bool deps_complete(const WorkerArgs& a, uint64_t ticket, const uint16_t* dep) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t back = dep[k];
    if (back != 0 && back <= ticket) {
      const uint64_t want = done_target(ticket - back, a.cap_shift);
      ok = ok && __hip_atomic_load(&a.st[(ticket - back) & a.cap_mask].done_seq, __ATOMIC_RELAXED, SC_SYSTEM) >= want;
    }
  }
  return ok;
}

// Does the task name a ticket that sits on the pending list (published later than everything the
// dispatcher has published so far)?  The list is in ticket order: two compares reject most
// candidates, a binary search decides the rest.
DEV bool names_pending(const DispShared* s, uint64_t ticket, const uint16_t* dep) {
  const uint32_t np = s->npend;
  if (np == 0) return false;
  const uint64_t first = s->pend[0].ticket, last = s->pend[np - 1].ticket + s->pend[np - 1].run - 1u;
  bool hit = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t back = dep[k];
    if (back == 0 || back > ticket) continue;
    const uint64_t d = ticket - back;
    if (d < first || d > last) continue;
    uint32_t lo = 0, hi = np;                      // entries [0, lo) begin at or before d
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (s->pend[mid].ticket <= d) lo = mid + 1; else hi = mid;
    }
    hit = hit || (lo > 0 && d - s->pend[lo - 1].ticket < s->pend[lo - 1].run);
  }
  return hit;
}

// Inclusive sum over the wavefront with DPP: shifts by 1, 2, 4, 8 inside each row of 16 lanes
// (lanes the shift runs out of the row for add 0), then lane 15 of a row to the whole next row
// (rows 1 and 3), then lane 31 to rows 2 and 3.  Six shuffles through the LDS crossbar before.
DEV int wave_prefix_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}
// First wavefront: the units of s->pub[0 .. npub) that go to ring `route`, numbered: entries of the other ring
// count as zero units (they keep their place in the list, so both rings see their tasks in list order).
DEV void dispatcher_number_units(DispShared* s, uint32_t npub, uint32_t route) {
  const uint32_t tid = threadIdx.x;
  const int v = wave_prefix_sum((int)((tid < npub && s->pub[tid].route == route) ? s->pub[tid].nchunks : 0u));
  s->ubeg[tid + 1] = (uint32_t)v;                // (entries past npub hold the total: the search below counts them out)
  if (tid == 0) s->ubeg[0] = 0;
}
// Write those units and make them claimable (by the whole workgroup); returns how many there are.
DEV uint32_t dispatcher_store_units(const WorkerArgs& a, DispShared* s, uint32_t npub, uint64_t units_w, uint32_t route) {
  const uint32_t tid = threadIdx.x;
  uint64_t* const ring = route == 0 ? a.units : a.units_j;
  const uint32_t total = s->ubeg[npub];
  // (no wait for the mirror stores of this pass: a worker checks the record it fetches, see mirror_record_valid)
  for (uint32_t u = tid; u < total; u += kThreads) {
    // The task of unit u is the number of prefix entries 1..64 that are <= u (they only grow).  Counted
    // in two levels of seven independent reads each, two LDS latencies, where a binary search takes six.
    static_assert(kDispatchBatch == 64, "two levels of eight");
    uint32_t oct = 0;
#pragma unroll
    for (uint32_t k = 1; k < 8; ++k) oct += s->ubeg[8u * k] <= u ? 1u : 0u;
    uint32_t lo = 8u * oct;
#pragma unroll
    for (uint32_t j = 1; j < 8; ++j) lo += s->ubeg[8u * oct + j] <= u ? 1u : 0u;
    const PubEntry pe = s->pub[lo];
    const uint64_t g = units_w + u;
    // one 8-byte store publishes the unit: the stamp makes it claimable
    __hip_atomic_store(&ring[g & a.unit_mask],
                       pack_unit(u - s->ubeg[lo], pe.opinfo >> 16, pe.slot, pe.opinfo & 0xffu, (pe.opinfo >> 8) & 1u, (pe.opinfo >> 9) & 1u,
                                 unit_stamp(g, a.unit_shift)),
                       __ATOMIC_RELAXED, SC_SYSTEM);
  }
  return total;
}
// Both, between barriers.
DEV uint32_t dispatcher_publish(const WorkerArgs& a, DispShared* s, uint32_t npub, uint64_t units_w, uint32_t route = 0) {
  if (threadIdx.x < 64) dispatcher_number_units(s, npub, route);
  __syncthreads();
  const uint32_t total = dispatcher_store_units(a, s, npub, units_w, route);
  __syncthreads();                                 // s->pub / s->ubeg may be rewritten after this
  return total;
}

struct UnitCursors { uint64_t w[2]; };      // units published so far on the main ring and on the second ring

// Publish s->pub[0 .. npub) on the ring(s) its entries name.  Called by the whole workgroup.
DEV void dispatcher_publish_all(const WorkerArgs& a, DispShared* s, uint32_t npub, UnitCursors& uc, bool any_second) {
  uc.w[0] += dispatcher_publish(a, s, npub, uc.w[0], 0);
  if (any_second) uc.w[1] += dispatcher_publish(a, s, npub, uc.w[1], 1);
}

// Publish the pending tasks whose dependencies have completed.
DEV void dispatcher_service_pending(const WorkerArgs& a, DispShared* s, UnitCursors& uc) {
  const uint32_t tid = threadIdx.x;
  const uint32_t np = s->npend;
  if (np == 0) return;
  static_assert(kPendMax <= 128 && kPendMax <= kThreads, "one pending entry per thread of the first two wavefronts");
  // One entry per thread: is it ready, and where does it go?  The first kDispatchBatch ready entries
  // move to the publish list, everything else closes ranks in the pending list; both keep their order
  // (ticket order).  Positions come from a ballot inside each of the two wavefronts plus the count
  // of the first one.
  const uint32_t lane = tid & 63u, wave = tid >> 6;
  PendEntry e;
  bool ready = false;
  if (tid < np) {
    e = s->pend[tid];
    ready = deps_complete(a, e.ticket, e.dep);
  }
  uint64_t m_ready = 0;
  if (tid < 128u) {
    m_ready = __ballot(ready);
    const uint64_t m_second = __ballot(ready && e.pub.route != 0);
    if (lane == 0) { s->ready[wave] = (uint32_t)__popcll(m_ready); s->ready[2 + wave] = m_second != 0 ? 1u : 0u; }
  }
  __syncthreads();                                 // the counts; and every entry is in its thread's registers
  const uint32_t ready0 = s->ready[0], ready_all = ready0 + s->ready[1];
  const bool any_second = (s->ready[2] | s->ready[3]) != 0;
  if (tid < np) {
    const uint32_t ready_before = (uint32_t)__popcll(m_ready & ((1ull << lane) - 1ull)) + (wave ? ready0 : 0u);
    const uint32_t taken_before = ready_before < kDispatchBatch ? ready_before : kDispatchBatch;
    if (ready && ready_before < kDispatchBatch) s->pub[ready_before] = e.pub;      // the rest waits for the next call
    else s->pend[tid - taken_before] = e;
  }
  const uint32_t npub = ready_all < kDispatchBatch ? ready_all : kDispatchBatch;
  __syncthreads();                                 // the lists are complete (and s->ready may be reused)
  if (tid == 0) s->npend = np - npub;
  if (npub == 0) { __syncthreads(); return; }
  order_loads();
  dispatcher_publish_all(a, s, npub, uc, any_second);   // its barriers also cover the new pending count
}

// First wavefront: plan a batch of n <= 64 staged records, beginning with ticket `mirrored` (m_bad: records that
// never passed their check).  Resolves the operator table ("claim time": slot, version, impl, status) and the
// dependencies in the records themselves, splits the batch into tasks that are published now (s->pub) and tasks
// that are held back (s->pend), and numbers the units of the main ring (s->ubeg).
// A lane reads what it asks of its record in one go, keeps it in registers and writes it back at the end: this is a
// chain of LDS latencies that every pass waits for, a pass of two records as long as one of 64.  (Field by field from
// LDS it took 1.35 us of a pass's 2.5.)
DEV void dispatcher_plan(const WorkerArgs& a, DispShared* s, uint32_t n, uint64_t mirrored, uint64_t m_bad, bool tracing, uint64_t tk0, uint64_t& st_deferred) {
  const uint32_t tid = threadIdx.x;
  const bool mine = tid < n, bad = (m_bad >> tid) & 1u;
  static_assert(offsetof(Record, path) == 2 && offsetof(Record, n_inputs) == 4 && offsetof(Record, rflags) == 9 && offsetof(Record, sel) == 13 &&
                offsetof(Record, impl) == 16 && offsetof(Record, version) == 20 && offsetof(Record, status) == 24 && offsetof(Record, nchunks) == 28 &&
                offsetof(Record, dep) == 48 && offsetof(Record, run) == 54 && offsetof(Record, ticket) == 56, "the words that are read and written as vectors");
  v4i* const words = (v4i*)&s->rec[tid];
  v4i w0 = words[0], w1 = words[1], w3 = words[3];
  const uint32_t npend0 = s->npend;
  if (bad) { w0[0] &= (int)0xff00ffff; w0[2] &= (int)0xffff00ff; w1[3] = 1; w3[0] = 0; w3[1] = 0; }       // (path, rflags, dep): do not trust any field
  static_assert(PATH_NOP == 0, "the path of a record that is not trusted");
  const uint32_t op = (uint32_t)w0[0] & 0xffffu, path = ((uint32_t)w0[0] >> 16) & 0xffu, n_inputs = (uint32_t)w0[1] & 0xffu;
  uint32_t rflags = ((uint32_t)w0[2] >> 8) & 0xffu, nchunks = (uint32_t)w1[3];
  const uint16_t dep[3] = {(uint16_t)((uint32_t)w3[0] & 0xffffu), (uint16_t)((uint32_t)w3[0] >> 16), (uint16_t)((uint32_t)w3[1] & 0xffffu)};
  const bool deps = (dep[0] | dep[1] | dep[2]) != 0;
  const uint64_t ticket = mirrored + tid;
  const uint64_t e = !bad && op < GPUOS_MAX_OPS ? s->entry[op] : 0ull;          // bounds check on the op id; 0: never registered
  const int32_t status = bad ? GPUOS_E_INVAL : (e == 0 ? GPUOS_E_BADOP : GPUOS_OK);
  const uint32_t impl = (uint32_t)e, sel = (uint32_t)(e >> 32) & 1u;
  if (status != GPUOS_OK || nchunks == 0) nchunks = 1;         // one unit reports the task
  if (tracing && mine) {
    s->rec[tid].t_dequeue[0] = (uint32_t)tk0; s->rec[tid].t_dequeue[1] = (uint32_t)(tk0 >> 32);
    if (op < GPUOS_MAX_OPS) atomicAdd(&s->opcnt[op], 1u);
  }
  // A link goes with the record before it: no units of its own, and nothing to wait for but that one (a
  // held head holds it, see below).  Only inside one pass, so that its mirror record is on its way
  // before the units that stand for it are.  Not under tracing, whose records tell of
  // one task at a time.
  const uint64_t m_can = __ballot(mine && status == GPUOS_OK && impl_links(impl, n_inputs, path));
  const uint64_t m_mark = __ballot(!tracing && (rflags & RF_LINK) != 0);
  const uint64_t m_link = m_can & m_mark & (m_can << 1);
  const bool link = (m_link >> tid) & 1u;
  const uint64_t behind = tid < 63u ? ~(m_link >> (tid + 1u)) : ~0ull;
  const uint32_t run = link ? 0u : (uint32_t)__builtin_ctzll(behind) + 1u;
  bool held = false;
  if (mine && !link && deps) {
    if (nchunks > kSmallTaskChunks) {
      // a large dependent task: its workers never wait; it is published once its
      // dependencies are complete (now, or later from the pending list)
      rflags |= RF_DEPS_RESOLVED;
      held = !deps_complete(a, ticket, dep);
    } else {
      // a small one is published at once and its workers wait, unless it names a task that is
      // itself held back: then it joins the pending list behind that task (tasks held in this
      // very pass are found below, in the split)
      held = names_pending(s, ticket, dep);
    }
  }
  // A task that names a task held in this pass is held too (a large one already is: such a
  // dependency cannot be complete).  Dependencies point backwards, so a few rounds of
  // "held if one of my in-pass dependencies is held" reach the fixed point.
  uint64_t m_def = __ballot(held);
  if (m_def != 0) {
    uint64_t dep_mask = 0;                                     // records of this pass the task names
    if (mine && !held) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const uint32_t back = dep[k];
        if (back != 0 && back <= tid) dep_mask |= 1ull << (tid - back);
      }
    }
    while (true) {
      held = held || (dep_mask & m_def) != 0;
      const uint64_t m2 = __ballot(held);
      if (m2 == m_def) break;
      m_def = m2;
    }
  }
  const bool unit = mine && run != 0;                        // (a link has no units)
  const uint64_t m_pub = __ballot(unit && !held), m_pend = __ballot(unit && held);
  const uint64_t below = (1ull << tid) - 1ull;
  const uint32_t pub_before = (uint32_t)__popcll(m_pub & below);
  if (held) rflags |= RF_DEPS_RESOLVED;                      // published only after its dependencies completed
  // tasks of a program that a run-time kernel holds as native code go to that kernel's ring
  const uint32_t prog = impl - GPUOS_IMPL_PROGRAM_BASE;
  PubEntry pe;
  pe.slot = (uint32_t)(ticket & a.cap_mask);
  pe.nchunks = nchunks;
  pe.opinfo = (op & 0xffu) | (sel << 8) | ((status == GPUOS_OK ? 1u : 0u) << 9) | ((uint32_t)((ticket >> a.cap_shift) & 0x3ffu) << 16);
  pe.route = (status == GPUOS_OK && impl >= GPUOS_IMPL_PROGRAM_BASE && prog < GPUOS_MAX_PROGRAMS && s->native[prog] != 0) ? 1u : 0u;
  if (unit) {
    if (held) {
      PendEntry& pd = s->pend[npend0 + (uint32_t)__popcll(m_pend & below)];
      pd.ticket = ticket;
      pd.pub = pe;
      pd.dep[0] = dep[0]; pd.dep[1] = dep[1]; pd.dep[2] = dep[2];
      pd.run = (uint16_t)run;
    } else {
      s->pub[pub_before] = pe;
    }
  }
  if (mine) {
    w0[2] = (int)(((uint32_t)w0[2] & 0xffff00ffu) | (rflags << 8));
    w0[3] = (int)(((uint32_t)w0[3] & 0xffff00ffu) | (sel << 8));
    w1[0] = (int)impl; w1[1] = (int)(uint32_t)(e >> 32); w1[2] = status; w1[3] = (int)nchunks;
    w3[1] = (int)(((uint32_t)w3[1] & 0xffffu) | (run << 16));
    w3[2] = (int)(uint32_t)ticket; w3[3] = (int)(uint32_t)(ticket >> 32);
    words[0] = w0; words[1] = w1; words[3] = w3;
  }
  // the units of the main ring, numbered as dispatcher_number_units does (entries past npub hold the total)
  const bool pub = (m_pub >> tid) & 1u;
  const int sum = wave_prefix_sum(pub && pe.route == 0 ? (int)nchunks : 0), total = __builtin_amdgcn_readlane(sum, 63);
  const uint32_t npub = (uint32_t)__popcll(m_pub);
  s->ubeg[1u + (pub ? pub_before : npub + tid - pub_before)] = (uint32_t)(pub ? sum : total);
  const uint64_t m_second = __ballot(pub && pe.route != 0);  // published now, on the second ring
  if (tid == 0) {
    s->ubeg[0] = 0;
    st_deferred += (uint32_t)__popcll(m_pend);
    s->npend = npend0 + (uint32_t)__popcll(m_pend);
    s->npub = npub;
    s->npub_second = m_second != 0 ? 1u : 0u;
  }
}

DEV void run_dispatcher(const WorkerArgs& a, DispShared* s) {
  const uint32_t tid = threadIdx.x;
  // A context whose worker was stopped and started again continues its ticket and work-unit
  // counts (both are zero on a fresh context); the operator table is read again from the host's
  // copy because the epoch seen starts at zero.
  uint64_t mirrored = a.resume_tickets, seen_epoch = 0;
  UnitCursors uc;
  uc.w[0] = __hip_atomic_load(&a.d->tail_units, __ATOMIC_RELAXED, SC_SYSTEM);
  uc.w[1] = __hip_atomic_load(&a.d->tail_units_j, __ATOMIC_RELAXED, SC_SYSTEM);
  for (uint32_t op = tid; op < GPUOS_MAX_OPS; op += kThreads) { s->entry[op] = 0; s->opcnt[op] = 0; }
  if (tid == 0) { s->npend = 0; s->lane_counted = 0; s->claimed = uc.w[0]; }
  __syncthreads();
  uint64_t idle_since = wall_clock64();
  if (tid == 0) {
    if (!a.resume) __hip_atomic_store(&a.h->clock_origin, idle_since, __ATOMIC_RELAXED, SC_SYSTEM);
    // the first heartbeat leaves together with the clock origin: the host pairs the moment it sees
    // it with device tick `clock_origin` (later heartbeats are poll counts, all above 1)
    __hip_atomic_store(&a.h->heartbeat, 1ull, __ATOMIC_RELAXED, SC_SYSTEM);
  }
  const bool tracing = a.trace != nullptr;
  const bool timing = a.timing != 0;
  uint32_t passes_since_flush = 0;
  bool counts_dirty = false;
  uint64_t polls = 0;
  bool stopping = false;
  uint64_t st_batches = 0, st_records = 0, st_units = 0, st_stage = 0, st_resolve = 0, st_write = 0, st_busy = 0;
  uint64_t st_deferred = 0;
  constexpr uint32_t kStagePieces = kDispatchBatch * 16u / kThreads;      // 16-byte pieces of a batch per thread
  static_assert(kStagePieces * kThreads == kDispatchBatch * 16u, "a batch is staged in whole rounds of the workgroup");
  uint64_t pre_base = ~0ull;               // first ticket of the records requested ahead (they wait in s->rec)
  uint32_t pre_n = 0;                      // how many
  const rsrc_t rh = make_rsrc(a.hring, (a.cap_mask + 1u) * (uint32_t)sizeof(Record));
  const rsrc_t rd = make_rsrc(a.dring, (a.cap_mask + 1u) * (uint32_t)sizeof(Record));
  const rsrc_t rbell = make_rsrc(a.bell, 16u);
  static_assert(offsetof(DoorbellCtl, tail) == 0 && offsetof(DoorbellCtl, epoch_word) == 8, "tail and epoch word are read with one 16-byte load");
  while (true) {
    // ---- poll the host ring (wavefront 0; the only PCIe poller of the kernel) ----
    // Every poll also reads the next kPrefetch records of the ring in the same round trip.  When
    // the doorbell then shows them published and their check words hold, they are already staged:
    // a lone task reaches the workers after one PCIe read latency instead of two.
    if (tid < 64) {
      uint64_t t, e;
      v4i q;
      const uint32_t g = tid >> 4, part = tid & 15u;               // record g of the prefetch window, 16-byte piece
      const bool have_pending = s->npend != 0;
      bool lane_dirty = false;                         // the short cut below counted an operator (tracing) since the last flush
      struct Poll { uint64_t t, e; v4i q; };
      auto request = [&](uint64_t base) {
        Poll p;
        const uint32_t slot = (uint32_t)((base + g) & a.cap_mask);
        const v4i b = Mem<POL_COHERENT>::ld16(rbell, 0u);        // tail and epoch word, one sample of both
        p.t = ((uint64_t)(uint32_t)b[1] << 32) | (uint32_t)b[0];
        p.e = ((uint64_t)(uint32_t)b[3] << 32) | (uint32_t)b[2];
        p.q = Mem<POL_COHERENT>::ld16(rh, slot * (uint32_t)sizeof(Record) + part * 16u);
        return p;
      };
      while (true) {
        const Poll cur = request(mirrored);
        t = cur.t; e = cur.e; q = cur.q;
        ++polls;
        if (tid == 0 && (polls & 63u) == 0) __hip_atomic_store(&a.h->heartbeat, polls, __ATOMIC_RELAXED, SC_SYSTEM);
        if (t == mirrored + 1 && e == seen_epoch && !stopping && !have_pending) {
          // ---- short cut for a lone task ----
          // One new record, whole (its check word holds), no table change, nothing held back: this
          // wavefront resolves, mirrors and publishes it by itself and polls on.  The other three
          // stay at the barrier below; the barriers of a batch pass are not on a lone task's
          // way.  Anything special (a dependency, a fence, many chunks, the second ring, a full
          // lookahead window) takes the ordinary way.
          order_loads();
          const uint32_t x0 = record_piece_sum(q, part);
          const uint64_t claimed0 = uni64(s->claimed);
          bool lone = __builtin_amdgcn_readfirstlane((uint32_t)(x0 == record_check_seed(mirrored))) != 0 &&
                      !(uc.w[0] > claimed0 && uc.w[0] - claimed0 >= kLookaheadUnits);
          if (lone) {
            if (tid < 16) ((v4i*)&s->rec[0])[part] = q;
            lds_wave_sync();
            Record& rc = s->rec[0];
            const uint32_t op = uni(rc.op_id);
            uint32_t nch = uni(rc.nchunks);
            const uint64_t ent = op < GPUOS_MAX_OPS ? s->entry[op] : 0ull;
            const uint32_t impl = uni((uint32_t)ent);
            lone = (rc.rflags & RF_FENCE) == 0 && (rc.dep[0] | rc.dep[1] | rc.dep[2]) == 0 && nch <= 64u &&
                   impl < GPUOS_IMPL_PROGRAM_BASE;
            if (lone) {
              const int32_t status = ent == 0 ? GPUOS_E_BADOP : GPUOS_OK;        // (covers an op id out of range)
              if (status != GPUOS_OK || nch == 0) nch = 1;
              const uint32_t sel = (uint32_t)((ent >> 32) & 1u);
              const uint64_t tk0 = clock_if(tracing);
              lds_wave_sync();                                             // every lane has read what lane 0 overwrites
              if (tid == 0) {
                rc.impl = impl;
                rc.version = (uint32_t)(ent >> 32);
                rc.sel = (uint8_t)sel;
                rc.status = status;
                rc.nchunks = nch;
                rc.ticket = mirrored;
                if (tracing) {
                  rc.t_dequeue[0] = (uint32_t)tk0; rc.t_dequeue[1] = (uint32_t)(tk0 >> 32);
                  if (op < GPUOS_MAX_OPS) { atomicAdd(&s->opcnt[op], 1u); s->lane_counted = 1u; }
                }
              }
              lane_dirty = tracing;
              lds_wave_sync();
              const uint32_t slot0 = (uint32_t)(mirrored & a.cap_mask);
              if (tid < 16) {
                v4i w = ((const v4i*)&s->rec[0])[part];
                if (part == 15u) w[3] = 0;
                const uint32_t xs = record_piece_sum(w, part);
                if (part == 15u) w[3] = (int)(record_check_seed(mirrored) - xs);
                Mem<POL_COHERENT>::st16(rd, slot0 * (uint32_t)sizeof(Record) + part * 16u, w);
              }
              if (tid < nch) {
                const uint64_t gu = uc.w[0] + tid;
                __hip_atomic_store(&a.units[gu & a.unit_mask],
                                   pack_unit(tid, (uint32_t)((mirrored >> a.cap_shift) & 0x3ffu), slot0, op, sel, status == GPUOS_OK ? 1u : 0u,
                                             unit_stamp(gu, a.unit_shift)),
                                   __ATOMIC_RELAXED, SC_SYSTEM);
              }
              mirrored += 1;
              uc.w[0] += nch;
              if (tid == 0) __hip_atomic_store(&a.h->dispatched, mirrored, __ATOMIC_RELAXED, SC_SYSTEM);
              if (timing || a.idle_exit_ticks != 0) idle_since = wall_clock64();
              st_batches += 1; st_records += 1; st_units += nch;
              continue;
            }
          }
        }
        if (t != mirrored || e != seen_epoch || stopping || have_pending) break;
        if (lane_dirty && (polls & 63u) == 0) break;    // idle again: let the whole workgroup publish the per-operator counts
        if ((polls & 63u) == 0 && a.idle_exit_ticks != 0 && wall_clock64() - idle_since > a.idle_exit_ticks) {
          e |= 2u;                                  // behave as if the host had asked to stop
          break;
        }
      }
      order_loads();
      // keep the prefetched records whose check word holds and that the doorbell value read in the
      // same round covers
      const uint32_t x = record_piece_sum(q, part);
      const bool good = mirrored + g < t && x == record_check_seed(mirrored + g);
      if (good) ((v4i*)&s->rec[g])[part] = q;
      if (part == 0) s->pre[g] = good ? 1u : 0u;
      if (e & 3u) {                                 // stop: take the final tail after the flag
        t = __hip_atomic_load(&a.bell->tail, __ATOMIC_RELAXED, SC_SYSTEM);
        order_loads();
      }
      if (tid == 0) {
        s->tail = t;
        s->epoch_word = e;
        s->lane_tickets = mirrored;
        s->lane_units = uc.w[0];
      }
    }
    __syncthreads();
    const uint64_t tail = s->tail, ew = s->epoch_word;
    mirrored = s->lane_tickets;                      // the short cut above may have moved both on
    uc.w[0] = s->lane_units;
    if (tracing && s->lane_counted) counts_dirty = true;
    __syncthreads();
    if (tracing && tid == 0) s->lane_counted = 0;  // (read again only after the next poll's barrier)
    if ((ew >> 12) != (seen_epoch >> 12)) {
      const uint32_t hinted = (uint32_t)((ew >> 4) & 0xffu);
      const bool one = ((ew >> 12) - (seen_epoch >> 12)) == 1 && hinted != 0xffu;
      dispatcher_refresh_table(a, s, one ? hinted : 0xffu);
      dispatcher_refresh_native(a, s);
      if (tid == 0) {
        const uint32_t y = __hip_atomic_load(&a.bell->yield_every, __ATOMIC_RELAXED, SC_SYSTEM);
        __hip_atomic_store(&a.d->yield_every, y, __ATOMIC_RELAXED, SC_SYSTEM);
      }
      __syncthreads();
    }
    seen_epoch = ew & ~3ull;
    if (ew & 3u) stopping = true;

    dispatcher_service_pending(a, s, uc);

    // ---- mirror new records, batch by batch ----
    // A pass has three barriers: every wavefront finds out by itself what the batch is (the same few LDS words) and
    // requests its share of the next one; the first plans the batch, alone and without a barrier; then all
    // write it out.  (As a dozen short steps with a barrier behind each a pass of 64 mixed
    // tasks took 4.3 us, 3.3 so.)
    bool first_batch = true;                       // the prefetched records belong to the first batch after a poll
    while (mirrored < tail) {
      // Dequeue only a bounded distance ahead of execution: the dependency state seen at dequeue
      // time is then close to what the workers will see, and the pending list stays short.
      // The claim counter only grows: it is read again only when the value at hand says "too far ahead".
      if (uc.w[0] > s->claimed && uc.w[0] - s->claimed >= kLookaheadUnits) {
        __syncthreads();
        if (tid == 0) s->claimed = __hip_atomic_load(&a.d->claim, __ATOMIC_RELAXED, SC_SYSTEM);
        __syncthreads();
      }
      const bool throttled = uc.w[0] > s->claimed && uc.w[0] - s->claimed >= kLookaheadUnits;
      const uint32_t room = kPendMax - s->npend, lane = tid & 63u;
      uint32_t n = (uint32_t)((tail - mirrored) < kDispatchBatch ? (tail - mirrored) : kDispatchBatch);
      if (n > room) n = room;
      if (throttled || n == 0) {                                   // let the workers catch up
        __syncthreads();                                           // everyone has read the pending count
        dispatcher_service_pending(a, s, uc);
        if (s->npend == 0) __builtin_amdgcn_s_sleep(8);
        __syncthreads();
        break;                                                     // back to the poll loop (stop, table, heartbeat)
      }
      const uint64_t tk0 = clock_if(timing || tracing);
      // Records requested ahead (with the poll, or while the previous batch was written out) already
      // lie in s->rec and were checked as they arrived.
      static_assert(kDispatchBatch == 64, "a wavefront looks at the whole batch");
      const bool ahead = (pre_base == mirrored && lane < pre_n && s->preok[lane] != 0) || (first_batch && lane < kPrefetch && s->pre[lane] != 0);
      first_batch = false;
      uint64_t m_bad = __ballot(lane < n && !ahead);               // the same in every wavefront
      if (m_bad != 0) {
        // stage: 16 pieces of 16 bytes per record.  System-scope loads: an ordinary load of host
        // memory may hit a line the CU's vector cache kept from the previous lap of the ring.
        // Every record carries a check word (a weighted sum of its 64 words must equal a seed made
        // from its ticket): a record that has not landed completely yet, or is left over from the previous lap,
        // fails the check and is read again; one that never passes is completed with an error
        // instead of being executed.
        for (uint32_t attempt = 0; m_bad != 0 && attempt < kStageRetries; ++attempt) {
          if (attempt != 0) __builtin_amdgcn_s_sleep(16);
          __syncthreads();                                         // everyone has read the last attempt's verdicts
#pragma unroll
          for (uint32_t j = 0; j < kStagePieces; ++j) {
            const uint32_t p = tid + j * kThreads;
            const uint32_t rix = p >> 4, part = p & 15u;
            if ((m_bad >> rix) & 1u) {                             // uniform over the 16 lanes of a record
              const uint32_t slot = (uint32_t)((mirrored + rix) & a.cap_mask);
              const v4i q = Mem<POL_COHERENT>::ld16(rh, slot * (uint32_t)sizeof(Record) + part * 16u);
              ((v4i*)&s->rec[rix])[part] = q;
              const uint32_t x = record_piece_sum(q, part);
              if (part == 0) s->ok[rix] = (x == record_check_seed(mirrored + rix)) ? 1u : 0u;
            }
          }
          __syncthreads();
          m_bad &= ~__ballot(((m_bad >> lane) & 1u) && s->ok[lane]);
        }
      }
      const uint64_t tk1 = clock_if(timing);
      // a FENCE task starts a batch of its own: cut the batch in front of the first one after slot 0
      {
        const uint64_t m = __ballot(lane >= 1 && lane < n && !((m_bad >> lane) & 1u) && (s->rec[lane].rflags & RF_FENCE));
        if (m) n = (uint32_t)__builtin_ctzll(m);
      }
      const bool fence = !(m_bad & 1u) && (uni(s->rec[0].rflags) & RF_FENCE) != 0;
      // Request the next batch now, if the doorbell value already covers it: the loads travel while
      // this batch is planned and written out.  A piece that turns
      // out incomplete fails its record's check word when it arrives and is read again at staging time.
      pre_base = mirrored + n;
      pre_n = tail > pre_base ? (uint32_t)((tail - pre_base) < kDispatchBatch ? (tail - pre_base) : kDispatchBatch) : 0u;
      v4i pre_q[kStagePieces];
#pragma unroll
      for (uint32_t j = 0; j < kStagePieces; ++j) {
        // No branch round the load: a piece that is not wanted gets an offset past the ring, which the
        // buffer hardware answers with zero without touching memory.  (With the load under an `if`
        // the compiler waited for each of the four before it issued the next: four memory round
        // trips in a row, 1.6 of the pass's 4.4 us.)
        const uint32_t p = tid + j * kThreads;
        const uint32_t slot = (uint32_t)((pre_base + (p >> 4)) & a.cap_mask);
        pre_q[j] = Mem<POL_COHERENT>::ld16(rh, p < pre_n * 16u ? slot * (uint32_t)sizeof(Record) + (p & 15u) * 16u : kNoLoad);
      }
      // a leading FENCE: everything earlier must be published and complete first
      if (fence) {
        __syncthreads();
        while (s->npend != 0) { dispatcher_service_pending(a, s, uc); __syncthreads(); }
        if (tid == 0) {
          while (__hip_atomic_load(&a.d->done_count, __ATOMIC_RELAXED, SC_SYSTEM) < mirrored)
            __builtin_amdgcn_s_sleep(4);
          order_loads();
        }
        __syncthreads();
      }
      __syncthreads();                                             // everyone has read what the plan is about to change
      if (tid < 64) dispatcher_plan(a, s, n, mirrored, m_bad, tracing, tk0, st_deferred);
      __syncthreads();
      const uint64_t tk2 = clock_if(timing);
      // Write the records into the device mirror (write-through stores), held-back ones included; each leaves
      // with a check word of its own over what it now holds (resolved fields, ticket).  Then a thread puts the next batch's
      // pieces where it took its own out (checked as they arrive: the next pass finds the verdict in s->preok), and only then
      // the units are stored: the wait for those loads leaves the mirror stores in flight, and the records
      // have a head start (a worker that sees its unit first fetches its record twice).
#pragma unroll
      for (uint32_t j = 0; j < kStagePieces; ++j) {
        if (j * (kThreads / 16u) >= uni(n)) break;                 // (16 records a round: most passes of a few tasks have one)
        const uint32_t p = tid + j * kThreads, rix = p >> 4, part = p & 15u;
        v4i q = ((const v4i*)&s->rec[rix])[part];
        if (part == 15u) q[3] = 0;
        const uint32_t x = record_piece_sum(q, part);              // the 16 lanes of a record share a row
        if (part == 15u) q[3] = (int)(record_check_seed(mirrored + rix) - x);
        const uint32_t slot = (uint32_t)((mirrored + rix) & a.cap_mask);
        Mem<POL_COHERENT>::st16(rd, p < n * 16u ? slot * (uint32_t)sizeof(Record) + part * 16u : kNoLoad, q);
      }
      if (pre_n != 0) {
#pragma unroll
        for (uint32_t j = 0; j < kStagePieces; ++j) {
          const uint32_t p = tid + j * kThreads;
          if (p < pre_n * 16u) {                                   // uniform over the 16 lanes of a record
            ((v4i*)&s->rec[p >> 4])[p & 15u] = pre_q[j];
            const uint32_t x = record_piece_sum(pre_q[j], p & 15u);
            if ((p & 15u) == 0) s->preok[p >> 4] = (x == record_check_seed(pre_base + (p >> 4))) ? 1u : 0u;
          }
        }
      }
      const uint64_t before = uc.w[0] + uc.w[1];
      uc.w[0] += dispatcher_store_units(a, s, s->npub, uc.w[0], 0);        // (no wait for the stores above: see mirror_record_valid)
      if (s->npub_second != 0) {
        __syncthreads();
        uc.w[1] += dispatcher_publish(a, s, s->npub, uc.w[1], 1);
      }
      const uint32_t total = (uint32_t)(uc.w[0] + uc.w[1] - before);
      __syncthreads();
      mirrored += n;
      if (tid == 0) __hip_atomic_store(&a.h->dispatched, mirrored, __ATOMIC_RELAXED, SC_SYSTEM);
      if (timing || a.idle_exit_ticks != 0) idle_since = wall_clock64();
      st_batches += 1; st_records += n; st_units += total;
      if (timing) { st_stage += tk1 - tk0; st_resolve += tk2 - tk1; st_write += idle_since - tk2; st_busy += idle_since - tk0; }
      dispatcher_service_pending(a, s, uc);
      if (tracing) {
        counts_dirty = true;
        if (++passes_since_flush >= 256u) {
          for (uint32_t op = tid; op < GPUOS_MAX_OPS; op += kThreads) {
            const uint32_t add = s->opcnt[op];
            if (add) { s->opcnt[op] = 0; __hip_atomic_fetch_add(&a.opcount[op], (uint64_t)add, __ATOMIC_RELAXED, SC_SYSTEM); }
          }
          passes_since_flush = 0;
          counts_dirty = false;
          __syncthreads();
        }
      }
    }
    if (tracing && counts_dirty && mirrored >= tail) {        // the ring ran empty: publish the per-operator counts
      for (uint32_t op = tid; op < GPUOS_MAX_OPS; op += kThreads) {
        const uint32_t add = s->opcnt[op];
        if (add) { s->opcnt[op] = 0; __hip_atomic_fetch_add(&a.opcount[op], (uint64_t)add, __ATOMIC_RELAXED, SC_SYSTEM); }
      }
      passes_since_flush = 0;
      counts_dirty = false;
      __syncthreads();
    }
    if (stopping && mirrored >= tail) {
      while (s->npend != 0) dispatcher_service_pending(a, s, uc);   // nothing is left behind
      drain_stores();                                  // every unit store of every wave has landed ...
      __syncthreads();                                 // ... before the stop flag can be seen
      if (tid == 0) {
        uint64_t* st = a.d->stat;
        // totals over every run of the context's worker
        st[ST_DISP_BATCHES] += st_batches; st[ST_DISP_RECORDS] += st_records; st[ST_DISP_UNITS] += st_units;
        st[ST_DISP_TICKS_STAGE] += st_stage; st[ST_DISP_TICKS_RESOLVE] += st_resolve; st[ST_DISP_TICKS_WRITE] += st_write;
        st[ST_DISP_TICKS_TOTAL_BUSY] += st_busy; st[ST_DISP_POLLS] += polls; st[ST_DISP_DEFERRED] += st_deferred;
        __hip_atomic_store(&a.d->tail_units, uc.w[0], __ATOMIC_RELAXED, SC_SYSTEM);
        __hip_atomic_store(&a.d->tail_units_j, uc.w[1], __ATOMIC_RELAXED, SC_SYSTEM);
        drain_stores();
        __hip_atomic_store(&a.d->stop_dev, 1u, __ATOMIC_RELAXED, SC_SYSTEM);
        __hip_atomic_store(&a.h->exit_code, (ew & 2u) ? 2u : 1u, __ATOMIC_RELAXED, SC_SYSTEM);
      }
      return;
    }
  }
}

union KernelShared {
  DispShared disp;
  WorkShared work;
};

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) gpuos_worker_kernel(WorkerArgs a) {
  __shared__ KernelShared sh;
  if (blockIdx.x == 0) run_dispatcher(a, &sh.disp);
  else run_worker<0, BuiltinExec>(&sh.work);
}

// one ordinary launch per task: block b executes chunk b
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) gpuos_single_task_kernel(Record rec) {
  __shared__ Record s_rec;
  __shared__ alignas(16) float s_red[kScratchFloats];
  if (threadIdx.x == 0) s_rec = rec;
  __syncthreads();
  exec_chunk<POL_PLAIN>(&s_rec, RecHead::of(&s_rec), s_rec.impl, blockIdx.x, s_red, nullptr, threadIdx.x);   // built-in implementations only
}

// The workgroups of a stopped worker left holding work-unit numbers beyond the last published one
// (each claims a number, sees the stop flag and exits): hand those numbers out again, and lower
// the stop flag, before the next worker starts.
__global__ void gpuos_resume_fixup_kernel(DevCtl* d) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    d->claim = d->tail_units;
    d->stop_dev = 0;
  }
}

int launch_resume_fixup(DevCtl* d, void* stream) {
  hipLaunchKernelGGL(gpuos_resume_fixup_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, d);
  return (int)hipGetLastError();
}

// Device-side state (control block, ring mirror, work-unit ring, slot state, operator table) of the
// one context per GPU that gpuos_init_static creates: a file-scope array instead of hipMalloc.  In
// host code the name `scratch` is only a handle for the symbol, not a device address: the address
// on each GPU comes from hipGetSymbolAddress, once per device, with that device current, and that
// pointer is what the host passes on (memset, kernel arguments).
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kStaticScratchBytes];

int static_scratch(int device, void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices || !out) return (int)hipErrorInvalidValue;
  std::lock_guard<std::mutex> lk(mu);
  if (!ptr[device]) {
    int cur = 0;
    hipError_t e = hipGetDevice(&cur);
    if (e == hipSuccess && cur != device) e = hipSetDevice(device);
    void* p = nullptr;
    if (e == hipSuccess) e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess) return (int)e;
    if (!p) return (int)hipErrorInvalidSymbol;
    ptr[device] = p;
  }
  *out = ptr[device];
  return (int)hipSuccess;
}

int launch_worker(const WorkerArgs& a, uint32_t grid, void* stream) {
  hipLaunchKernelGGL(gpuos_worker_kernel, dim3(grid), dim3(kThreads), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

int worker_max_blocks_per_cu(int* out) {
  return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(out, gpuos_worker_kernel, (int)kThreads, 0);
}

int launch_single(const Record& r, void* stream) {
  const uint32_t grid = r.nchunks ? r.nchunks : 1u;
  hipLaunchKernelGGL(gpuos_single_task_kernel, dim3(grid), dim3(kThreads), 0, (hipStream_t)stream, r);
  return (int)hipGetLastError();
}

}  // namespace gpuos
