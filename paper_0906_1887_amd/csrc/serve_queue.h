// The serving queue: its layout, and the two protocols that meet on it, the
// claim of a work item (xeng_serve_kernel) and the update that publishes jobs
// (xeng_publish_kernel).  Both are written over a memory type M, so that what
// the kernels run is also what the CPU model of tests/serve_model.cpp runs
// through every order in which the loads and stores can take effect.
#pragma once

#include "common.h"

namespace corr {

// The host publishes each admitted job in a slot.  The job's generation is the
// number of the update that publishes it, so it differs from those of the
// slot's other jobs and tells which of two jobs came later.  The slot's claim
// word holds it in its upper half and counts claimed items in its lower one, so
// that one fetch-and-add both claims an item and says whose it is.  Every job
// runs 128-row tiles.
constexpr int kServeLine = 32;             // uint32 per 128-byte line
constexpr int kServeSlots = 64;
struct ServeJob {
  XArgs x;                  // the job's pass: samples, strides, output, n_tiles, n_items (channel x tile)
  uint32_t* flag;           // completion word in host memory (device view)
  uint32_t flag_value;      // written there when the job's last item is done
  uint32_t pad_;
  uint64_t ident;           // serve_ident: whose record this is and how many items it has, read as one word
};
constexpr uint64_t serve_ident(uint32_t gen, int32_t n_items) { return (uint64_t)gen << 32 | (uint32_t)n_items; }
// One update of the queue (xeng_publish_kernel), in mapped host memory: the
// admitted jobs with their slots, and the new list of active slots (an
// entry is a slot; whose job it holds, the claim tells).
struct ServeUpdate {
  uint64_t active[kServeSlots];
  int32_t slot[kServeSlots];
  ServeJob job[kServeSlots];
};
struct ServeQueue {
  ServeJob* slots;          // [n_slots]
  uint64_t* claim;          // slot s at claim[s * kServeLine / 2]
  uint32_t* done;           // slot s at done[s * kServeLine]: items done of its job
  uint64_t* active;         // [1 + n_slots]: count and version (upper half) of the list, then its entries
  uint64_t* last_claim;     // wall clock (s_memrealtime ticks) of the latest claim or grid start
  uint32_t* closing;        // highest grid generation that has closed (no more claims)
  uint32_t* host_closing;   // the same, in host memory (device view) for the scheduler
  uint64_t* host_claimed;   // host memory (device view): slot s at [s * kServeLine / 2 + 1] receives
                            // the job's generation once its last item is claimed
  uint32_t gen;             // this launch's generation (increasing from 1)
  uint32_t idle_ticks;      // queue idle this long (100 MHz ticks): the grid closes
  int32_t n_slots;
  int32_t max_polls;        // bound on one workgroup's empty polls (a safety net)
};

// What a workgroup remembers of the list between claims.
struct ServeView {
  uint32_t turn;      // its place in the round robin
  uint32_t n;         // length and version of the list when it last looked
  uint32_t version;
  uint64_t spent;     // places of that list whose jobs have no unclaimed item
  uint32_t acquired;  // the samples of jobs up to this update are visible to its loads
  bool cold;          // nothing acquired yet
  bool acquire;       // out: drop what the caches hold before the claimed job's samples are read
};

// One lane: claim one item; the slot, or -1 when the grid has closed (or this
// workgroup has polled max_polls times without work).  *word receives the
// claim word.  Memory takes microseconds to answer while the grid streams
// samples, so the next entry is fetched together with the list's length, on
// the guess that the list is the one last seen, and the job's identity
// together with the claim.
//
// The identity decides whether the claim holds.  A job's record is written
// before the claim word takes its generation, and stays until all of its items
// are done.  So if the identity has the claim word's generation, its item count
// is that job's; an older one was loaded before the add, and is loaded again
// after it; a newer one means that the job is complete, and the count past its
// items.  An entry of an old list therefore costs an add and claims nothing
// that is not there.  (With the item count in the list, beside a generation in
// a word of its own, an entry loaded while the slot's next job was listed could
// give that job its predecessor's count.)
//
// A list's entries are in memory before its head, so an entry that is loaded
// once the head has shown a list is that list's or a later one's: what is noted
// of its place holds for the list, or until the later head is seen.  The entry
// that came with a new head may be older, and is loaded again.  (A place noted
// as spent by it hid the new list's job there from the workgroup.)
//
// Samples may have been written since the grid started, into memory that this
// CU or XCD has cached.  What was published by an update was written before it,
// so one acquire after the list's head or a claim word has shown update u makes
// the samples of all jobs up to u visible, and a claim needs another one just
// if its job is newer than that, whichever list led to it.  (Asking whether the
// list had changed instead missed the job of a list whose entry was loaded
// after the former list's head.)
template <class M>
__host__ __device__ inline int serve_claim(M& m, const ServeQueue& q, ServeView& v, uint64_t* word) {
  for (int poll = 0; poll < q.max_polls; ++poll) {
    uint32_t at = v.turn % v.n;
    const uint32_t closing = m.load_agent(q.closing);
    uint64_t head, e;
    m.load2(q.active, q.active + 1 + at, head, e);
    if (closing >= q.gen) return -1;
    const uint32_t n = (uint32_t)head < (uint32_t)q.n_slots ? (uint32_t)head : (uint32_t)q.n_slots;
    bool fetched = true;
    if ((uint32_t)(head >> 32) != v.version) {
      v.version = (uint32_t)(head >> 32);
      v.spent = 0;
      if (n > 0) v.n = n;
      fetched = false;
    }
    for (uint32_t a = 0; a < n; ++a, fetched = false) {
      at = v.turn++ % n;
      if ((v.spent >> at) & 1u) continue;
      if (!fetched) e = m.load(q.active + 1 + at);
      const uint32_t s = (uint32_t)e;
      if (s >= (uint32_t)q.n_slots) continue;
      const uint64_t* const ident = &q.slots[s].ident;
      uint64_t w, id;
      m.add_load(q.claim + (size_t)s * (kServeLine / 2), ident, w, id);
      if ((id >> 32) != (w >> 32)) id = m.load(ident);
      const uint32_t limit = (id >> 32) == (w >> 32) ? (uint32_t)id : 0u;
      if ((uint32_t)w >= limit) {
        v.spent |= 1ull << at;
        continue;
      }
      const uint32_t gen = (uint32_t)(w >> 32);
      v.acquire = v.cold || (int32_t)(gen - v.acquired) > 0;
      if (v.acquire) v.acquired = (int32_t)(v.version - gen) > 0 ? v.version : gen;
      v.cold = false;
      m.claimed(q);
      // the job's last item: tell the host, which then lists the job no more
      if ((uint32_t)w + 1 == limit) m.store(q.host_claimed + (size_t)s * (kServeLine / 2) + 1, w >> 32);
      *word = w;
      return (int)s;
    }
    if (m.idle(q)) return -1;
  }
  return -1;
}

// One of nt threads (at least one more than kServeSlots) of an update: the
// jobs' records and done counts, then their slots' claim words (no item of a
// job is claimed before its claim word is set, so its record is seen first),
// then the list's entries, then its head.  The slots' former jobs are complete.
// settle() returns once every store of every thread before it has reached
// memory.  The words that later steps store are read from host memory ahead of
// the first wait.
template <class M>
__host__ __device__ inline void serve_publish(M& m, const ServeUpdate* u, int n_jobs, int n_active, uint32_t version,
                                              const ServeQueue& q, int tid, int nt) {
  constexpr int kWords = sizeof(ServeJob) / 8;
  const uint64_t* src = reinterpret_cast<const uint64_t*>(u->job);
  for (int k = tid; k < n_jobs * kWords; k += nt)
    m.store(reinterpret_cast<uint64_t*>(q.slots + u->slot[k / kWords]) + k % kWords, src[k]);
  const int slot = tid < n_jobs ? u->slot[tid] : 0;
  const uint64_t word = (uint64_t)version << 32;
  const uint64_t entry = tid < n_active ? u->active[tid] : 0;
  if (tid < n_jobs) m.exchange(q.done + (size_t)slot * kServeLine, 0u);
  m.settle();
  if (tid < n_jobs) m.exchange(q.claim + (size_t)slot * (kServeLine / 2), word);
  m.settle();
  if (tid < n_active) m.store(q.active + 1 + tid, entry);
  m.settle();
  if (tid == nt - 1) m.store(q.active, (uint64_t)version << 32 | (uint64_t)n_active);
}

}  // namespace corr
