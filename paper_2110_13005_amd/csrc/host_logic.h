// Host-side decisions of the stage runtime, free of any HIP call: which posted message Alg. 2's receive loop
// takes next, the bookkeeping of the activation stash slots (Sec. 3.3: at most pipeline_limit microbatches in
// flight), when the deferred weight gradients of a group of microbatches are formed, how long the loop waits
// for a message, and the bucket plan of the offloaded optimizer (Sec. 5.2) with the chunks of the step that
// overlaps the backward tail (Sec. 5.3); and the tile a GEMM launch takes with the order of its workgroups (gemm.hip).
// stage.cpp calls these with its HIP streams and events around them; the CPU tests compile this header alone (with the
// address, undefined-behaviour and thread sanitizers) and drive it with simulated events.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cstddef>
#include <deque>
#include <vector>

namespace axonn {
namespace host {

// ------------------------------------------------------------------------------ stash slots
// A slot is FREE, LIVE (forward issued, backward not yet: it counts as in flight) or AWAIT_WGRAD (backward chain
// issued, the slot's tensors are still operands of a weight-gradient contraction that has not been issued).
// `Slots` is any container of records with the members `state` and `mb_id`.
enum SlotState { SLOT_FREE = 0, SLOT_LIVE = 1, SLOT_AWAIT_WGRAD = 2 };

template <class Slots>
int find_live(const Slots& slots, int mb_id) {
  int i = 0;
  for (const auto& s : slots) {
    if (s.state == SLOT_LIVE && s.mb_id == mb_id) return i;
    ++i;
  }
  return -1;
}
template <class Slots>
int find_free(const Slots& slots) {
  int i = 0;
  for (const auto& s : slots) {
    if (s.state == SLOT_FREE) return i;
    ++i;
  }
  return -1;
}
template <class Slots>
int count_state(const Slots& slots, int state) {
  int n = 0;
  for (const auto& s : slots) n += (s.state == state);
  return n;
}

// Forward(msg) for microbatch mb_id: may it start, and where?
enum ForwardAdmission {
  FWD_OK = 0,            // *slot is free
  FWD_NEEDS_FLUSH = 1,   // admissible, but every slot not in flight awaits its weight gradients: form them first
  FWD_NEGATIVE_ID = -1, FWD_ALREADY_LIVE = -2, FWD_PIPELINE_FULL = -3, FWD_NO_SLOT = -4
};
template <class Slots>
int admit_forward(const Slots& slots, int mb_id, int in_flight, int pipeline_limit, int* slot) {
  *slot = -1;
  if (mb_id < 0) return FWD_NEGATIVE_ID;
  if (find_live(slots, mb_id) >= 0) return FWD_ALREADY_LIVE;
  if (in_flight >= pipeline_limit) return FWD_PIPELINE_FULL;
  *slot = find_free(slots);
  if (*slot >= 0) return FWD_OK;
  return count_state(slots, SLOT_AWAIT_WGRAD) > 0 ? FWD_NEEDS_FLUSH : FWD_NO_SLOT;
}
template <class Slots>
void commit_forward(Slots& slots, int slot, int mb_id, int* in_flight) {
  slots[slot].state = SLOT_LIVE;
  slots[slot].mb_id = mb_id;
  ++*in_flight;
}
// Backward(msg): the slot of the microbatch's forward, or -1 if none is in flight.
template <class Slots>
int admit_backward(const Slots& slots, int mb_id) { return mb_id >= 0 ? find_live(slots, mb_id) : -1; }
// The backward chain of `slot` is issued: the microbatch leaves the pipeline; the slot waits for its weight
// gradients unless they were issued with the chain (activation checkpointing).
template <class Slots>
void commit_backward(Slots& slots, int slot, bool wgrad_issued_with_chain, int* in_flight) {
  slots[slot].mb_id = -1;
  slots[slot].state = wgrad_issued_with_chain ? SLOT_FREE : SLOT_AWAIT_WGRAD;
  --*in_flight;
}
// A weight-gradient pass over all waiting slots is issued (or a new batch drops them).
template <class Slots>
int release_awaiting(Slots& slots) {
  int n = 0;
  for (auto& s : slots)
    if (s.state == SLOT_AWAIT_WGRAD) { s.state = SLOT_FREE; ++n; }
  return n;
}

// What follows the backward chain of a microbatch with stored activations: the batch's last microbatch closes
// every open group (and that pass finishes the gradients layer by layer); otherwise a group closes once
// `group` microbatches wait (group == 0: only when a slot is needed or the batch ends).
enum WgradAction { WGRAD_NONE = 0, WGRAD_FLUSH = 1, WGRAD_FLUSH_FINAL = 2 };
inline int wgrad_action(bool last_of_batch, int group, int n_awaiting) {
  if (last_of_batch) return WGRAD_FLUSH_FINAL;
  return (group > 0 && n_awaiting >= group) ? WGRAD_FLUSH : WGRAD_NONE;
}
// Are the gradients of every backward so far complete once the next one's work is queued (`n_awaiting` slots wait
// before it)?  With checkpointing its weight gradients go with the chain; otherwise if a group closes.
inline bool gradients_complete(bool ckpt, bool last_of_batch, int group, int n_awaiting) {
  return ckpt || wgrad_action(last_of_batch, group, n_awaiting + 1) != WGRAD_NONE;
}

// ------------------------------------------------------------------------------ messages
// A message is admissible if its work may start now: a forward needs a pipeline place and must not be in
// flight already; a backward needs its forward.
template <class Slots>
bool admissible(int kind, int mb_id, const Slots& slots, int in_flight, int pipeline_limit) {
  return kind == 0 ? (in_flight < pipeline_limit && find_live(slots, mb_id) < 0) : (find_live(slots, mb_id) >= 0);
}

// The receive loop's choice: the first posted message (in posting order) that is admissible and has arrived.
// msg(i) -> (kind, mb_id) of posted message i; arrived(i) -> 1 arrived, 0 not yet, < 0 an error of the event
// layer (returned in *error, the choice is then -1).  *any_admissible tells a loop that found nothing whether
// waiting can help.
template <class Slots, class Msg, class Arrived>
int choose_message(size_t n_posted, Msg&& msg, Arrived&& arrived, const Slots& slots, int in_flight,
                   int pipeline_limit, bool* any_admissible, int* error) {
  *any_admissible = false;
  *error = 0;
  for (size_t i = 0; i < n_posted; ++i) {
    const auto km = msg(i);
    if (!admissible(km.first, km.second, slots, in_flight, pipeline_limit)) continue;
    *any_admissible = true;
    const int a = arrived(i);
    if (a < 0) { *error = a; return -1; }
    if (a == 0) continue;
    return (int)i;
  }
  return -1;
}

// The stage as it would be if every message ran by itself.  What that decides does not change when messages run together: the
// order in which messages are taken, and which microbatches' weight gradients are formed in one pass (so how their sums are
// rounded, and what is pending when a batch is cut short).  Microbatches go by a number of their own here, as an id may come
// again within a batch.
class OneByOne {
 public:
  struct Place { int state = SLOT_FREE, mb_id = -1, number = -1; };
  typedef std::vector<int> Pass;                  // numbers of one pass's microbatches, in the order of their sum

  void new_batch(int n_slots) {
    places.assign((size_t)n_slots, Place{});
    in_flight = backwards = 0;
    passes.clear();
  }
  // Of an admissible message; returns the microbatch's number (-1: it is not admissible).
  int forward(int mb_id) {
    if (find_free(places) < 0) close();
    const int i = find_free(places);
    if (i < 0) return -1;
    commit_forward(places, i, mb_id, &in_flight);
    return places[(size_t)i].number = next_number++;
  }
  int backward(int mb_id, bool ckpt) {
    const int i = find_live(places, mb_id);
    if (i < 0) return -1;
    commit_backward(places, i, ckpt, &in_flight);
    ++backwards;
    return places[(size_t)i].number;
  }
  int awaiting() const { return count_state(places, SLOT_AWAIT_WGRAD); }
  // The weight gradients of all waiting microbatches are formed here.
  void close() {
    Pass p;
    for (const Place& q : places)
      if (q.state == SLOT_AWAIT_WGRAD) p.push_back(q.number);
    if (p.empty()) return;
    passes.push_back(p);
    release_awaiting(places);
  }

  std::vector<Place> places;
  int in_flight = 0, backwards = 0;
  std::deque<Pass> passes;     // closed, not yet taken by the stage

 private:
  int next_number = 0;
};

// How many microbatches of T tokens may run as one pass over their concatenated tokens (1: each by itself); `overlap`: on
// several streams.  A small microbatch is bound by the latency of its launches and by tiles that do not fill the chip; up to
// 2^24 elements of an activation the narrowest contraction of a layer (T x h outputs) has at most a round of 256 tiles of
// 256 x 256.  Whole batches of two layers with a slot per microbatch, 2 streams, ms, by the largest activation of a pass:
//   hidden, tokens, microbatches    each alone   2^22    2^23    2^24    2^25
//   1024, 1024, 8                      2.92      2.40    2.17    2.17    2.17
//   2048, 2048, 8                     11.04     11.09   10.19   10.08    9.89
//   2048, 2048, 2                      2.95      2.95    2.75    2.76    2.75
//   4096, 2048, 4                     17.0      17.0    17.0    15.9    15.7
//   4096, 1024, 6                     14.01     14.01   13.03   14.21   12.99      (passes of 1, 1, 2, 3 and 6)
//   6144, 512, 8                      21.9      21.9    19.7    19.2    18.9
// Beyond 2^24 little is gained, and results come later than they have to.
constexpr int kMaxMerge = 8;
constexpr int64_t kMergeElements = int64_t(1) << 24;
// A backward pass of several microbatches keeps a gradient of h columns and one float per head in the place of the f columns
// of GeLU': narrower MLPs run one by one.
// The slots are dealt to passes of equal size (a smaller size where its T x h outputs fill the rounds of 256 tiles better was
// slower on 60 of 110 random stages, by up to 15 %).  With fewer slots than microbatches a pass takes at most 4 of them, and
// never all of an odd number: a pass that holds every slot has nothing to overlap with.  8 microbatches of 1280 tokens at h 1536,
// by the size of a pass, ms:
//   slots      1       2       3       4       5       6       8
//   2        6.35    6.93
//   3        6.76    6.43    6.54
//   4        6.14    5.57    5.83    5.67
//   5        6.07    5.85    5.59    5.80    5.98
//   6        6.02    5.39    5.63    5.61    5.87    5.77
//   8        5.80    5.33    5.28    4.83    5.16    5.10    4.81
// On several streams the forwards of single microbatches run beside backwards, which is worth more the better one of them
// fills the chip and the fewer slots there are.  Random stages with fewer slots than microbatches, one by one / together:
//   2 slots, even number      up to 2^20 elements 0.98 to 1.31 (26 stages), above 0.89 to 1.17, mean 0.98 (28)
//   2 slots, odd number       up to 2^17          0.95 to 1.15 (7),         above 0.88 to 1.14, mean 0.99 (16)
//   3 slots                   up to 2^20          0.98 to 1.59 (58),        above 0.95 to 1.31, mean 1.04 (60)
//   4 slots                   up to 2^21          0.99 to 1.76 (57),        above 0.96 to 1.10, mean 1.02 (12)
//   more                      1.01 to 1.94 at all sizes (60)
// (an odd number leaves the last microbatch's two passes behind all others; the upper ends are stages whose streams shared a
// hardware queue).  On one stream all gain.
inline int merge_limit(int64_t T, int64_t h, int64_t f, int64_t heads, int slots, int n_microbatches, bool overlap = false) {
  if (f < h + 2 * heads) return 1;
  const int64_t elements = T * std::max<int64_t>(h, (f + 3) / 4);
  const int64_t fits = std::min<int64_t>(kMaxMerge, kMergeElements / elements);
  if (fits < 1) return 1;
  const bool refill = slots < n_microbatches;
  if (overlap && refill && slots <= 4 && elements > int64_t(1) << (slots == 4 ? 21 : slots == 2 && n_microbatches % 2 ? 17 : 20)) return 1;
  const int64_t most = refill ? std::min<int64_t>(fits, 4) : fits;
  const int64_t passes = std::max<int64_t>((slots + most - 1) / most, refill && slots > 1 && slots % 2 ? 2 : 1);
  return (int)((slots + passes - 1) / passes);
}

// What the loop needs to know of a posted message to run it together with others.  `alone`: its own completion is waited
// for (a done_event: the neighbour's message hangs on it), so it is not made to wait for others.
struct MessageSpan {
  int kind, mb_id;
  bool alone;
  uint64_t in, in_end, out, out_end;          // payload and result in device memory
};
// May `later` start together with `earlier`, posted before it?  Not if one of the two reads or writes what the other writes.
inline bool independent(const MessageSpan& earlier, const MessageSpan& later) {
  const auto overlap = [](uint64_t a, uint64_t a_end, uint64_t b, uint64_t b_end) { return a < b_end && b < a_end; };
  return !overlap(earlier.out, earlier.out_end, later.in, later.in_end) &&
         !overlap(earlier.out, earlier.out_end, later.out, later.out_end) &&
         !overlap(earlier.in, earlier.in_end, later.out, later.out_end);
}
// The messages that run together with `chosen` (which a forward has a free slot for), out of those in the order that OneByOne
// takes them: messages of its kind that have arrived, are admissible then and there, and are independent of every message before
// them.  A forward does not pass another one by: each then finds the slot that it has one by one.  Their slots are consecutive,
// so that each tensor of the stash is one matrix over all their tokens.
// span(i) -> MessageSpan of message i.  picked: positions, in slot order, the chosen message first; returns their number.
template <class Slots, class Span, class Arrived>
int merge_messages(size_t n_posted, Span&& span, Arrived&& arrived, int chosen, const Slots& slots, int in_flight,
                   int pipeline_limit, int max_merge, int* picked) {
  picked[0] = chosen;
  const MessageSpan first = span((size_t)chosen);
  if (first.alone || max_merge < 2) return 1;
  int n = 1;
  const auto joins = [&](size_t i) {
    const MessageSpan m = span(i);
    if (m.kind != first.kind || m.alone || arrived(i) != 1) return false;
    for (size_t j = 0; j < i; ++j)
      if (!independent(span(j), m) || (m.kind == 0 && span(j).kind == 0 && arrived(j) == 1 && std::find(picked, picked + n, (int)j) == picked + n))
        return false;
    for (int k = 0; k < n; ++k) {
      if ((size_t)picked[k] == i || span((size_t)picked[k]).mb_id == m.mb_id) return false;
      if ((size_t)picked[k] > i && !independent(m, span((size_t)picked[k]))) return false;
    }
    return true;
  };
  const int slot0 = first.kind == 0 ? find_free(slots) : find_live(slots, first.mb_id);
  for (; slot0 >= 0 && n < max_merge && slot0 + n < (int)slots.size(); ++n) {
    const auto& next = slots[slot0 + n];
    int found = -1;
    for (size_t i = 0; i < n_posted && found < 0; ++i) {
      const MessageSpan m = span(i);
      const bool fits = m.kind == 0 ? next.state == SLOT_FREE && in_flight + n < pipeline_limit && find_live(slots, m.mb_id) < 0
                                    : next.state == SLOT_LIVE && next.mb_id == m.mb_id;
      if (fits && joins(i)) found = (int)i;
    }
    if (found < 0) break;
    picked[n] = found;
  }
  return n;
}

// post(): a message is refused if one of the same kind for the same microbatch is already posted, or if the
// batch has no room for another of its kind (issued + posted would exceed n_microbatches).
enum PostCheck { POST_OK = 0, POST_DUPLICATE = -1, POST_SURPLUS = -2 };
template <class Msg>
int check_post(int kind, int mb_id, size_t n_posted, Msg&& msg, int issued_of_kind, int n_microbatches) {
  int same = 0;
  for (size_t i = 0; i < n_posted; ++i) {
    const auto km = msg(i);
    if (km.first != kind) continue;
    ++same;
    if (km.second == mb_id) return POST_DUPLICATE;
  }
  return issued_of_kind + same >= n_microbatches ? POST_SURPLUS : POST_OK;
}

// Library stream of a message's work: backward chains keep to stream 0 (they share accumulators and the
// workspace), forwards go round robin over the others.
inline int stream_index(int kind, int n_streams, int* fwd_rr) {
  if (kind == 1 || n_streams == 1) return 0;
  return 1 + ((*fwd_rr)++ % (n_streams - 1));
}

// How long the blocking loop waits for the next message: the limit applies to each wait, from the moment the
// loop first found nothing to dispatch until a message is dispatched again.
struct WaitClock {
  double limit_s;
  double since = -1.0;          // < 0: not waiting
  explicit WaitClock(double limit) : limit_s(limit) {}
  void dispatched() { since = -1.0; }
  bool expired(double now) {    // call when nothing could be dispatched
    if (since < 0) since = now;
    return now - since > limit_s;
  }
};

// ------------------------------------------------------------------------------ optimizer state in place
// May a kernel work on `bytes` of host memory at device address `dev` (0: the memory has none)?  Only if all of them lie
// in the one allocation [alloc, alloc + alloc_bytes) that holds the first: the two ends may belong to different
// allocations with memory between them that the GPU cannot reach.  The kernel needs 16-byte alignment.
inline bool addressable_in_place(uint64_t dev, uint64_t bytes, uint64_t alloc, uint64_t alloc_bytes) {
  return dev != 0 && dev % 16 == 0 && dev >= alloc && dev - alloc <= alloc_bytes && bytes <= alloc_bytes - (dev - alloc);
}

// ------------------------------------------------------------------------------ optimizer buckets
inline uint64_t bucket_count(uint64_t n, uint64_t bucket) { return bucket ? (n + bucket - 1) / bucket : 0; }

// The i-th bucket a pass processes (ascending offsets, or descending for the pass that follows the backward
// tail from the last layer down): its index, element range and the device buffer set it uses.
struct BucketPlan { uint64_t index, offset, count; int set; };
inline BucketPlan bucket_plan(uint64_t n, uint64_t bucket, int n_sets, uint64_t i, bool descending) {
  const uint64_t nb = bucket_count(n, bucket);
  BucketPlan p;
  p.index = descending ? nb - 1 - i : i;
  p.offset = p.index * bucket;
  p.count = std::min<uint64_t>(bucket, n - p.offset);
  p.set = (int)(i % (uint64_t)n_sets);
  return p;
}
// Descending pass in chunks of k buckets: the element range [lo, hi) of the chunk that starts at processing
// index i (i a multiple of k).  The chunk's updates may start when every gradient in [lo, hi) is final.
inline void chunk_span(uint64_t n, uint64_t bucket, uint64_t k, uint64_t i, uint64_t* lo, uint64_t* hi) {
  const uint64_t nb = bucket_count(n, bucket);
  const BucketPlan first = bucket_plan(n, bucket, 1, i, true);
  const uint64_t n_in_chunk = std::min<uint64_t>(k, nb - i);
  *lo = (first.index + 1 - n_in_chunk) * bucket;
  *hi = first.offset + first.count;
}
// Gradients become final from the last layer down, so a range is final once the layer that holds its lowest
// element is: the largest l with layer_begin[l] <= lo (layer_begin ascending, layer_begin[0] == 0).
inline int lowest_layer(const uint64_t* layer_begin, int n_layers, uint64_t lo) {
  int l = 0;
  while (l + 1 < n_layers && layer_begin[l + 1] <= lo) ++l;
  return l;
}

// ------------------------------------------------------------------------------ order of a launch's workgroups
// Workgroups are dealt round-robin to the 8 XCDs: ids x, x + 8, ... run on XCD x.  The position of workgroup `id` in an
// order in which every XCD's workgroups are consecutive, for any number of workgroups.
constexpr uint32_t xcd_contiguous(uint32_t id, uint32_t n_workgroups) {
  const uint32_t xcd = id % 8, left = n_workgroups % 8;  // the first `left` XCDs have one workgroup more
  return xcd * (n_workgroups / 8) + (xcd < left ? xcd : left) + id / 8;
}

// Division by a number the host knows: recip_of(d) for recip_div on the GPU, exact for 0 <= n < 2^31, 1 <= d < 2^31 (an estimate
// that is at most one too large).  0 stands for d == 1, whose reciprocal does not fit.
constexpr uint32_t recip_of(uint32_t d) { return d <= 1 ? 0u : (uint32_t)((uint64_t(1) << 32) / d + 1); }
constexpr uint32_t recip_div(uint32_t n, uint32_t d, uint32_t recip) {
  if (recip == 0) return n;
  uint32_t q = (uint32_t)(((uint64_t)n * recip) >> 32);
  if (q * d > n) --q;
  return q;
}

// ------------------------------------------------------------------------------ tiles of the GEMM launcher
// Tile of the ring kernel for a problem that 256 x 256 tiles would not fill the chip with.
enum RingTile { RING_64x64, RING_128x64, RING_128x128, RING_128x192, RING_128x256, RING_TILES };
struct TileCost { int bm, bn; double fixed, step_few, step_full; };
// Microseconds: what a round of up to 256 tiles (one workgroup per CU) costs beside its k-steps, and a 64-wide k-step
// with few and with 256 tiles in flight.  From single launches with K = 1024 and K = 4096 of outputs of 256 x 256 to
// 2048 x 12288 (the difference gives the step, the rest the fixed part).
constexpr TileCost kRingCost[RING_TILES] = {{64, 64, 3.2, 0.20, 0.21}, {128, 64, 4.0, 0.28, 0.30},
                                            {128, 128, 5.0, 0.40, 0.47}, {128, 192, 7.5, 0.54, 0.68},
                                            {128, 256, 8.0, 0.65, 0.73}};
// The large-problem kernels.  Weights for the comparison with the ring tiles and no rates: their scale is the one that
// picks the faster kernel on 230 random shapes of 64 to 255 tiles of 256 x 256 (0.1 % slower than the better of the two on
// average; weight gradients with an fp32 result 1 % on 90 shapes of 40 to 420 tiles, for any weight of theirs from 0.9 to 1.4:
// 1.4 leaves their sums the order that they had when their large-problem kernel was the slower register-staged one).
constexpr double kBigFp32 = 1.4;
constexpr TileCost kBigCost[3] = {{256, 160, 12.0, 0.57, 0.80}, {256, 192, 12.0, 0.61, 0.84}, {256, 256, 12.0, 0.76, 1.06}};

// Modelled time of a problem with one tile size: whole rounds and a last one whose steps are faster the emptier it is.
inline double tile_cost(const TileCost& c, int64_t M, int64_t N, int64_t nk) {
  const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
  const double last = (double)(tiles % 256) / 256, steps = (double)nk;
  return (double)(tiles / 256) * (c.fixed + steps * c.step_full) +
         (last > 0 ? c.fixed + steps * (c.step_few + (c.step_full - c.step_few) * last) : 0.0);
}

// The fastest ring tile for an M x N x (nk k-steps) problem.
inline int fastest_ring_tile(int64_t M, int64_t N, int64_t nk) {
  int best = 0;
  for (int t = 1; t < RING_TILES; ++t)
    if (tile_cost(kRingCost[t], M, N, nk) < tile_cost(kRingCost[best], M, N, nk)) best = t;
  return best;
}

// Which ring tile an M x N x (nk k-steps) problem takes; -1: a large-problem kernel.  Those stay where their 256 x 256
// tiles fill the chip, and where the model prefers one of their widths.  Measured (bf16, single launches, the kernels
// before / now): 256 x 256 x 1024 17.0 / 5.7 us, 1024 x 1024 x 4096 52.6 / 16.1, 2048 x 1024 x 4096 52.6 / 23.8, 2048 x 2048 x
// 8192 103 / 67, 2048 x 3072 x 12288 226 / 137 (a kernel of 128 x 128 tiles staged through registers), 2048 x 4096 x 1024
// with GeLU 35.6 / 28.5 (half a round of 256 x 256 tiles).
// From 128 tiles on, which the large-problem kernels run well, the ring tile has to be modelled 8 % faster: without that,
// and with weights of 10, 0.75 / 0.80 / 1.0 and 1.05 / 1.10 / 1.4, 21 of 1050 launches of such shapes were more than 4 % slower
// than on the large-problem kernels, up to 2816 x 2944 x 10112 168 us against 137; now 5 are, by at most 5 %.
// `forced` (-1: none): number of 256 x 256 tiles from which the large-problem kernels are used whatever the model says.
// The rule does not look at whether the launch shares the chip: a ring kernel adds its two halves of k in another order
// than the large-problem kernels, and a batch's results should not depend on the number of streams it runs on.
// Measured, the choice would be the same: leaving half-filled rounds to the large-problem kernels beside other streams,
// or weighing in the CUs that a round leaves idle, changed whole batches by less than 1 % or made them slower.
inline int choose_ring_tile(int64_t M, int64_t N, int64_t nk, int64_t forced, bool fp32_result) {
  const int64_t big_tiles = ((M + 255) / 256) * ((N + 255) / 256);
  if (big_tiles >= (forced >= 0 ? forced : 256)) return -1;
  const int best = fastest_ring_tile(M, N, nk);
  const double limit = tile_cost(kRingCost[best], M, N, nk) * (big_tiles >= 128 ? 1.08 : 1.0) / (fp32_result ? kBigFp32 : 1.0);
  if (forced < 0)
    for (const TileCost& c : kBigCost)
      if (tile_cost(c, M, N, nk) < limit) return -1;
  return best;
}

// The 64 x 64 and 128 x 64 tiles have stages of 128 k and add it in another order than the others do by themselves.
constexpr bool adds_halves_of_128(int tile) { return tile == RING_64x64 || tile == RING_128x64; }

// The fastest tile for n problems whose tiles share one grid (modelled like one problem of all their tiles), such that each
// problem's sums are added in the order of own[i], the tile it takes by itself: halves_128[i] asks a kernel with 64-wide stages
// for the other order; one with 128-wide stages has only its own.
struct RingChoice { int tile; int64_t tiles; bool halves_128[4]; };
inline RingChoice same_order_tile(int n, const int64_t* M, const int64_t* N, int64_t nk, const int* own) {
  RingChoice best = {-1, 0, {}};
  double best_cost = 0;
  bool all_halves = true;
  for (int i = 0; i < n; ++i) all_halves = all_halves && adds_halves_of_128(own[i]);
  for (int t = 0; t < RING_TILES; ++t) {
    if (adds_halves_of_128(t) && !all_halves) continue;
    const TileCost& c = kRingCost[t];
    int64_t tiles = 0;
    for (int i = 0; i < n; ++i) tiles += ((M[i] + c.bm - 1) / c.bm) * ((N[i] + c.bn - 1) / c.bn);
    const double cost = tile_cost({1, 1, c.fixed, c.step_few, c.step_full}, tiles, 1, nk);
    if (best.tile < 0 || cost < best_cost) { best.tile = t; best.tiles = tiles; best_cost = cost; }
  }
  for (int i = 0; i < n; ++i) best.halves_128[i] = adds_halves_of_128(own[i]) && !adds_halves_of_128(best.tile);
  return best;
}

// Split of a long contraction with a small output over workgroups, for callers that can hand over a workspace: tile and
// number of parts (1: not split) with the lowest modelled time.  The parts cost a write and a read of their fp32 sums
// (4 TB/s) and a launch (5 us).  The LM head's input gradient, 2048 x 1024 x 51200 in four parts of 128 x 256 tiles: 345 -> 205 us.
struct RingSplit { int tile, parts; };
inline RingSplit choose_split(int64_t M, int64_t N, int64_t K, int64_t forced) {
  const int64_t nk = (K + 63) / 64;
  RingSplit best = {choose_ring_tile(M, N, nk, forced, false), 1};
  if (best.tile < 0) return best;
  double best_cost = tile_cost(kRingCost[best.tile], M, N, nk);
  for (int parts = 2; parts <= 16 && nk / parts >= 16; parts *= 2)
    for (int t = 0; t < RING_TILES; ++t) {
      const TileCost& c = kRingCost[t];
      const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * parts;
      const double cost = tile_cost({1, 1, c.fixed, c.step_few, c.step_full}, tiles, 1, (nk + parts - 1) / parts) +
                          5.0 + 8.0 * (double)parts * (double)M * (double)N / 4e6;
      if (cost < best_cost) { best = {t, parts}; best_cost = cost; }
    }
  return best;
}

}  // namespace host
}  // namespace axonn
