// CPU tests of the stage runtime's host logic (paper Alg. 2's receive loop, Sec. 3.3's pipeline_limit, the
// deferred weight-gradient groups, Sec. 5.2's bucket plan and Sec. 5.3's chunks) with a simulated event layer:
// no GPU, no HIP.  Built by tests/test_host_runtime.py with -fsanitize=address,undefined and with
// -fsanitize=thread.  The model stage below does with counters what stage.cpp does with streams and events,
// and takes every decision from host_logic.h, as stage.cpp does.
#include "../../paper_2110_13005_amd/csrc/host_logic.h"

#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <set>
#include <string>
#include <thread>
#include <utility>
#include <vector>

using namespace axonn::host;

#define CHECK(cond)                                                                   \
  do {                                                                                \
    if (!(cond)) {                                                                    \
      std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond);   \
      std::exit(1);                                                                   \
    }                                                                                 \
  } while (0)

namespace {

struct SlotRec { int state = SLOT_FREE; int mb_id = -1; };
struct Msg { int kind, mb_id; long ready_at; };   // ready_at: tick from which the payload "has arrived" (-1: no event)

// What stage.cpp keeps per stage, without the device.
struct ModelStage {
  int M, P, group, n_streams;
  bool ckpt;
  std::vector<SlotRec> slots;
  std::vector<Msg> inbox;
  int in_flight = 0, fwd_issued = 0, bwd_issued = 0, bwd_count = 0, fwd_rr = 0;
  long tick = 0;
  std::vector<std::pair<int, int>> log;            // (kind, mb) in dispatch order
  std::vector<std::vector<int>> wgrad_passes;      // microbatches of each weight-gradient pass
  std::vector<int> awaiting_mb;                    // microbatch of each slot in AWAIT_WGRAD, by slot
  OneByOne order;                                  // told of the same messages
  std::map<int, int> mb_of;                        // its number -> microbatch
  std::vector<int> stream_of;                      // stream index per dispatched message
  bool final_pass_seen = false;
  int max_in_flight = 0;

  ModelStage(int M_, int P_, int group_, int n_streams_, bool ckpt_ = false)
      : M(M_), P(P_), group(group_), n_streams(n_streams_), ckpt(ckpt_), slots(P_), awaiting_mb(P_, -1) { order.new_batch(P); }

  int post(int kind, int mb, long ready_at) {
    const auto posted = [this](size_t i) { return std::make_pair(inbox[i].kind, inbox[i].mb_id); };
    const int rc = check_post(kind, mb, inbox.size(), posted, kind == 0 ? fwd_issued : bwd_issued, M);
    if (rc == POST_OK) inbox.push_back(Msg{kind, mb, ready_at});
    return rc;
  }
  void flush(bool final_pass) {
    std::vector<int> pass;
    for (size_t i = 0; i < slots.size(); ++i)
      if (slots[i].state == SLOT_AWAIT_WGRAD) pass.push_back(awaiting_mb[i]);
    if (pass.empty()) return;
    CHECK(!final_pass_seen);
    wgrad_passes.push_back(pass);
    release_awaiting(slots);
    final_pass_seen = final_pass;
  }
  int forward(int mb) {
    int si = -1;
    int adm = admit_forward(slots, mb, in_flight, P, &si);
    if (adm == FWD_NEEDS_FLUSH) {
      flush(false);
      adm = admit_forward(slots, mb, in_flight, P, &si);
    }
    if (adm != FWD_OK) return adm;
    commit_forward(slots, si, mb, &in_flight);
    mb_of[order.forward(mb)] = mb;
    max_in_flight = std::max(max_in_flight, in_flight);
    return FWD_OK;
  }
  int backward(int mb) {
    const int si = admit_backward(slots, mb);
    if (si < 0) return -1;
    const bool last = bwd_count + 1 == M;
    ++bwd_count;
    commit_backward(slots, si, ckpt, &in_flight);
    CHECK(mb_of[order.backward(mb, ckpt)] == mb && order.in_flight == in_flight && order.backwards == bwd_count);
    if (!ckpt && gradients_complete(false, last, group, order.awaiting() - 1)) order.close();
    if (ckpt) {
      wgrad_passes.push_back({mb});
    } else {
      awaiting_mb[si] = mb;
      switch (wgrad_action(last, group, count_state(slots, SLOT_AWAIT_WGRAD))) {
        case WGRAD_FLUSH_FINAL: flush(true); break;
        case WGRAD_FLUSH: flush(false); break;
        default: break;
      }
    }
    return 0;
  }
  // The receive loop.  Returns 0 when the batch is dispatched, 1 when a non-blocking call has nothing more to do,
  // -2 if nothing can ever be scheduled, -3 when a wait expired.  One tick passes per fruitless look.
  int run(bool blocking, double wait_limit_ticks, int* n_dispatched = nullptr) {
    WaitClock wait(wait_limit_ticks);
    const auto posted = [this](size_t i) { return std::make_pair(inbox[i].kind, inbox[i].mb_id); };
    const auto arrived = [this](size_t i) { return (inbox[i].ready_at < 0 || inbox[i].ready_at <= tick) ? 1 : 0; };
    while (fwd_issued < M || bwd_issued < M) {
      bool any = false;
      int err = 0;
      const int c = choose_message(inbox.size(), posted, arrived, slots, in_flight, P, &any, &err);
      CHECK(err == 0);
      if (c < 0) {
        if (!blocking) return 1;
        if (!any) return -2;
        if (wait.expired((double)tick)) return -3;
        ++tick;
        continue;
      }
      wait.dispatched();
      const Msg m = inbox[c];
      inbox.erase(inbox.begin() + c);
      stream_of.push_back(stream_index(m.kind, n_streams, &fwd_rr));
      if (m.kind == 0) { CHECK(forward(m.mb_id) == FWD_OK); ++fwd_issued; }
      else { CHECK(backward(m.mb_id) == 0); ++bwd_issued; }
      log.push_back({m.kind, m.mb_id});
      if (n_dispatched) ++*n_dispatched;
      // invariants of Sec. 3.3 / Alg. 2 after every dispatch
      CHECK(in_flight <= P);
      CHECK(count_state(slots, SLOT_LIVE) == in_flight);
    }
    return 0;
  }
  void check_batch_complete() const {
    CHECK((int)log.size() == 2 * M);
    std::vector<int> f(M, -1), b(M, -1);
    for (size_t i = 0; i < log.size(); ++i) {
      auto& v = log[i].first == 0 ? f : b;
      CHECK(v[log[i].second] < 0);            // each message exactly once
      v[log[i].second] = (int)i;
    }
    for (int i = 0; i < M; ++i) CHECK(f[i] >= 0 && b[i] > f[i]);   // backward only after its forward
    // every microbatch's weight gradients formed exactly once, none left waiting, the last pass marked final
    std::multiset<int> seen;
    for (const auto& p : wgrad_passes) for (int mb : p) seen.insert(mb);
    CHECK((int)seen.size() == M);
    for (int i = 0; i < M; ++i) CHECK(seen.count(i) == 1);
    CHECK(count_state(slots, SLOT_AWAIT_WGRAD) == 0 && in_flight == 0);
    if (!ckpt) CHECK(final_pass_seen);
    // the passes that OneByOne closes
    std::vector<std::vector<int>> closed;
    for (const OneByOne::Pass& p : order.passes) {
      closed.emplace_back();
      for (int number : p) closed.back().push_back(mb_of.at(number));
    }
    CHECK(closed == (ckpt ? std::vector<std::vector<int>>() : wgrad_passes));
  }
};

void test_pipeline_limit_and_order(unsigned seed) {
  std::mt19937 rng(seed);
  for (int rep = 0; rep < 200; ++rep) {
    const int M = 1 + rng() % 12, P = 1 + rng() % M, group = rng() % 5, ns = 1 + rng() % 4;
    const bool ckpt = rng() % 4 == 0;
    ModelStage st(M, P, group, ns, ckpt);
    // a random valid interleaving of posts (posting order != arrival order: random ready ticks)
    std::vector<std::pair<int, int>> posts;
    for (int i = 0; i < M; ++i) { posts.push_back({0, i}); posts.push_back({1, i}); }
    std::shuffle(posts.begin(), posts.end(), rng);
    for (auto& pm : posts) CHECK(st.post(pm.first, pm.second, (long)(rng() % 50) - 5) == POST_OK);
    CHECK(st.run(true, 1e9) == 0);
    st.check_batch_complete();
    CHECK(st.max_in_flight <= P);
    if (!ckpt && group > 0)
      for (size_t i = 0; i + 1 < st.wgrad_passes.size(); ++i) CHECK((int)st.wgrad_passes[i].size() <= std::max(group, 1) || P < group);
    for (size_t i = 0; i < st.log.size(); ++i) {
      if (st.log[i].first == 1 || ns == 1) CHECK(st.stream_of[i] == 0);       // backward chains on stream 0
      else CHECK(st.stream_of[i] >= 1 && st.stream_of[i] < ns);
    }
  }
}

void test_arrival_order_decides() {
  // two forwards posted; the second arrives first: it is dispatched first (Alg. 2 runs whatever has arrived)
  ModelStage st(2, 2, 0, 2);
  CHECK(st.post(0, 0, 10) == POST_OK);
  CHECK(st.post(0, 1, 0) == POST_OK);
  CHECK(st.post(1, 0, 20) == POST_OK);
  CHECK(st.post(1, 1, 12) == POST_OK);
  CHECK(st.run(true, 1e9) == 0);
  CHECK(st.log[0] == std::make_pair(0, 1) && st.log[1] == std::make_pair(0, 0));
  CHECK(st.log[2] == std::make_pair(1, 1) && st.log[3] == std::make_pair(1, 0));
  st.check_batch_complete();
}

void test_duplicates_and_surplus() {
  ModelStage st(3, 2, 0, 2);
  CHECK(st.post(0, 0, -1) == POST_OK);
  CHECK(st.post(0, 0, -1) == POST_DUPLICATE);
  CHECK(st.post(1, 0, -1) == POST_OK);                 // same microbatch, other kind: fine
  CHECK(st.post(0, 1, -1) == POST_OK);
  CHECK(st.post(0, 2, -1) == POST_OK);
  CHECK(st.post(0, 3, -1) == POST_SURPLUS);            // a fourth forward in a batch of three
  int n = 0;
  CHECK(st.run(false, 1e9, &n) == 1);                  // non-blocking: f0 f1 (limit 2) b0 f2, then nothing admissible has arrived
  CHECK(n == 4 && st.in_flight == 2);
  CHECK(st.post(0, 1, -1) == POST_SURPLUS);            // issued forwards count towards the batch
  CHECK(st.forward(1) == FWD_ALREADY_LIVE);
  CHECK(st.forward(7) == FWD_PIPELINE_FULL);
  CHECK(st.forward(-1) == FWD_NEGATIVE_ID);
  CHECK(st.backward(0) == -1);                         // already consumed
  CHECK(st.run(true, 1e9) == -2);                      // two backwards expected, none posted: cannot progress
  CHECK(st.post(1, 2, -1) == POST_OK && st.post(1, 1, -1) == POST_OK);
  CHECK(st.run(true, 1e9) == 0);
  st.check_batch_complete();
}

void test_backward_without_forward_never_runs() {
  ModelStage st(2, 1, 0, 1);
  CHECK(st.post(1, 0, -1) == POST_OK);                 // gradient for a microbatch whose forward is not even posted
  CHECK(st.run(true, 1e9) == -2);
  CHECK(st.log.empty());
  CHECK(st.post(0, 0, -1) == POST_OK);
  int n = 0;
  CHECK(st.run(false, 1e9, &n) == 1 && n == 2);
  CHECK(st.log[0] == std::make_pair(0, 0) && st.log[1] == std::make_pair(1, 0));
}

void test_wait_limit_is_per_wait() {
  // messages arrive every 40 ticks, the limit is 50: a batch of 6 takes > 200 ticks in all and still succeeds
  ModelStage st(3, 3, 0, 2);
  for (int i = 0; i < 3; ++i) { CHECK(st.post(0, i, 40 * (i + 1)) == POST_OK); CHECK(st.post(1, i, 40 * (i + 4)) == POST_OK); }
  CHECK(st.run(true, 50.0) == 0);
  CHECK(st.tick > 200);
  st.check_batch_complete();
  // one message later than the limit: the wait expires; the posted message is still there and a second run resumes
  ModelStage late(1, 1, 0, 1);
  CHECK(late.post(0, 0, 0) == POST_OK && late.post(1, 0, 500) == POST_OK);
  CHECK(late.run(true, 50.0) == -3);
  CHECK(late.inbox.size() == 1 && late.fwd_issued == 1 && late.in_flight == 1);
  CHECK(late.run(true, 1e9) == 0);
  late.check_batch_complete();
  WaitClock w(10.0);
  CHECK(!w.expired(100.0) && !w.expired(109.0) && w.expired(111.0));
  w.dispatched();
  CHECK(!w.expired(200.0));
}

void test_wgrad_groups() {
  // stored activations, 8 microbatches all in flight, groups of 3: passes of 3, 3 and 2, the last one final
  ModelStage st(8, 8, 3, 2);
  for (int i = 0; i < 8; ++i) CHECK(st.post(0, i, -1) == POST_OK);
  for (int i = 0; i < 8; ++i) CHECK(st.post(1, i, -1) == POST_OK);
  CHECK(st.run(true, 1e9) == 0);
  CHECK(st.wgrad_passes.size() == 3);
  CHECK(st.wgrad_passes[0].size() == 3 && st.wgrad_passes[1].size() == 3 && st.wgrad_passes[2].size() == 2);
  CHECK(st.wgrad_passes[2].back() == 7 || st.wgrad_passes[2].front() == 7);
  st.check_batch_complete();
  // group 0 with fewer slots than microbatches: a pass is forced whenever a forward finds no free slot
  ModelStage tight(6, 2, 0, 2);
  for (int i = 0; i < 6; ++i) { CHECK(tight.post(0, i, -1) == POST_OK); CHECK(tight.post(1, i, -1) == POST_OK); }
  CHECK(tight.run(true, 1e9) == 0);
  tight.check_batch_complete();
  CHECK(tight.wgrad_passes.size() >= 3);
  CHECK(wgrad_action(false, 0, 100) == WGRAD_NONE && wgrad_action(false, 2, 1) == WGRAD_NONE);
  CHECK(wgrad_action(false, 2, 2) == WGRAD_FLUSH && wgrad_action(true, 0, 1) == WGRAD_FLUSH_FINAL);
  CHECK(gradients_complete(true, false, 0, 0) && gradients_complete(false, true, 0, 3));
  CHECK(gradients_complete(false, false, 1, 0) && gradients_complete(false, false, 2, 1));
  CHECK(!gradients_complete(false, false, 0, 3) && !gradients_complete(false, false, 2, 0));
}

void test_bucket_plan(unsigned seed) {
  std::mt19937_64 rng(seed);
  for (int rep = 0; rep < 300; ++rep) {
    const uint64_t bucket = 8 * (1 + rng() % 64), n = 1 + rng() % (bucket * 9);
    const uint64_t nb = bucket_count(n, bucket);
    CHECK(nb == (n + bucket - 1) / bucket);
    for (int desc = 0; desc < 2; ++desc) {
      uint64_t covered = 0;
      std::vector<char> hit(nb, 0);
      for (uint64_t i = 0; i < nb; ++i) {
        const BucketPlan p = bucket_plan(n, bucket, 3, i, desc != 0);
        CHECK(p.index == (desc ? nb - 1 - i : i) && !hit[p.index]);
        hit[p.index] = 1;
        CHECK(p.offset == p.index * bucket && p.count >= 1 && p.count <= bucket && p.offset + p.count <= n);
        CHECK((p.index + 1 < nb) == (p.count == bucket) || p.count == bucket);   // only the last bucket is ragged
        if (p.index + 1 == nb) CHECK(p.offset + p.count == n);
        CHECK(p.set == (int)(i % 3));                    // three buffer sets in rotation, in processing order
        covered += p.count;
      }
      CHECK(covered == n);
    }
    // chunks of k buckets of the descending pass tile [0, n) from the top down
    const uint64_t k = 1 + rng() % 5;
    uint64_t expect_hi = n;
    for (uint64_t i = 0; i < nb; i += k) {
      uint64_t lo = 0, hi = 0;
      chunk_span(n, bucket, k, i, &lo, &hi);
      CHECK(hi == expect_hi && lo < hi && lo % bucket == 0);
      CHECK((hi - lo + bucket - 1) / bucket == std::min<uint64_t>(k, nb - i));
      expect_hi = lo;
    }
    CHECK(expect_hi == 0);
    // the gate of a chunk: the layer that holds its lowest element; every layer the chunk touches is at or
    // above it, i.e. final no later (gradients become final from the last layer down)
    const int L = 1 + (int)(rng() % 6);
    std::vector<uint64_t> begin(L);
    for (int l = 0; l < L; ++l) begin[l] = (uint64_t)l * (n / L + 1);
    for (uint64_t i = 0; i < nb; i += k) {
      uint64_t lo = 0, hi = 0;
      chunk_span(n, bucket, k, i, &lo, &hi);
      const int l = lowest_layer(begin.data(), L, lo);
      CHECK(l >= 0 && l < L && begin[l] <= lo && (l + 1 == L || begin[l + 1] > lo));
    }
  }
  // the benchmark's optimizer problem: 1.6e9 parameters in buckets of 2^26 -> 24 buckets, the last of 56 496 128
  CHECK(bucket_count(1600000000ull, 1ull << 26) == 24);
  CHECK(bucket_plan(1600000000ull, 1ull << 26, 3, 23, false).count == 56496128ull);
  CHECK(bucket_plan(1600000000ull, 1ull << 26, 3, 0, true).count == 56496128ull);
}

void test_addressable_in_place() {
  const uint64_t a = 1ull << 32, n = 1 << 20;
  CHECK(addressable_in_place(a, n, a, n) && addressable_in_place(a + 16, n - 16, a, n) && addressable_in_place(a, 12, a, n));
  CHECK(!addressable_in_place(a + 4, 64, a, n));                // alignment
  CHECK(!addressable_in_place(0, n, 0, n));                     // no device address
  CHECK(!addressable_in_place(a, n + 1, a, n) && !addressable_in_place(a + 16, n, a, n));   // reaches past the allocation
  // the last byte lies in a second pinned allocation at a + 2 n: what is between the two has no mapping
  CHECK(!addressable_in_place(a + n - 4096, n + 8192, a, n));
  CHECK(!addressable_in_place(a - 16, 64, a, n) && !addressable_in_place(a + n + 16, 64, a, n) && !addressable_in_place(a, n, 0, 0));
  CHECK(!addressable_in_place(a + 16, ~0ull - 8, a, n));        // no wrap-around
}

void test_workgroup_order() {
  for (int n = 1; n <= 600; ++n) {
    std::vector<int> xcd_at(n, -1);
    for (int id = 0; id < n; ++id) {
      const int p = (int)xcd_contiguous(id, n);
      CHECK(p >= 0 && p < n && xcd_at[p] < 0);            // every position once
      xcd_at[p] = id % 8;
    }
    for (int p = 1; p < n; ++p) CHECK(xcd_at[p] >= xcd_at[p - 1]);   // one run per XCD
  }
}

void test_gemm_tiles() {
  // the large-problem kernels: from 256 tiles of 256 x 256, from a threshold given, and where they are the faster ones
  CHECK(choose_ring_tile(4096, 4096, 16, -1, false) == -1 && choose_ring_tile(512, 512, 16, 4, false) == -1);
  CHECK(choose_ring_tile(4080, 4000, 2, 1000, false) >= 0);
  CHECK(choose_ring_tile(2816, 2944, 158, -1, false) == -1);     // 132 tiles, two full rounds of 128 x 128: 137 us against 168
  CHECK(choose_ring_tile(5632, 1408, 24, -1, false) == -1);
  CHECK(choose_ring_tile(2768, 2944, 11, -1, true) >= 0);        // with an fp32 result 29.9 us against 40.5
  CHECK(choose_ring_tile(3968, 3712, 188, -1, true) == -1);
  // the ring kernel where a round of its tiles covers the problem: 28.5 us against 35.6, 137 against 226
  CHECK(choose_ring_tile(2048, 4096, 16, -1, false) == RING_128x256 && choose_ring_tile(2048, 3072, 192, -1, false) >= 0);
  CHECK(choose_ring_tile(256, 256, 16, -1, false) == RING_64x64);
  // division by reciprocal
  for (uint32_t d : {1u, 2u, 3u, 7u, 8u, 24u, 1000u, 65535u, 65536u, 1u << 30, (1u << 31) - 1})
    for (uint32_t n : {0u, 1u, d - 1, d, d + 1, 3 * d - 1, 12345u, (1u << 31) - 1})
      if (n < 1u << 31) CHECK(recip_div(n, d, recip_of(d)) == n / d);
  // a shared grid keeps the order of sums that each problem has by itself
  const int64_t gm[4] = {1000, 384, 384, 384}, gn[4] = {384, 1000, 384, 1152};
  for (int mask = 0; mask < 16; ++mask) {
    int own[4];
    for (int i = 0; i < 4; ++i) own[i] = mask >> i & 1 ? RING_128x128 : RING_64x64;
    const RingChoice r = same_order_tile(4, gm, gn, 21, own);
    CHECK(r.tile >= 0 && r.tiles > 0 && (mask == 0 || !adds_halves_of_128(r.tile)));
    for (int i = 0; i < 4; ++i)
      CHECK(adds_halves_of_128(own[i]) == (adds_halves_of_128(r.tile) || r.halves_128[i]));
  }
  const int alone = RING_64x64;
  CHECK(same_order_tile(1, gm, gn, 21, &alone).tile == fastest_ring_tile(1000, 384, 21));
  // a split is bounded (16 parts of 16 k-steps at least) and none where the problem fills the chip
  std::mt19937 rng(3);
  for (int rep = 0; rep < 2000; ++rep) {
    const int64_t M = 8 * (1 + rng() % 1024), N = 8 * (1 + rng() % 1024), K = 8 * (1 + rng() % 8192);
    const RingSplit r = choose_split(M, N, K, -1);
    CHECK(r.parts >= 1 && r.parts <= 16 && (r.parts == 1 || ((K + 63) / 64) / r.parts >= 16));
    CHECK(r.parts == 1 || (r.tile >= 0 && ((M + 255) / 256) * ((N + 255) / 256) < 256));
  }
}

void test_merged_messages() {
  // sizes: one microbatch each where an activation has 2^24 elements, never more than 8 or pipeline_limit, wide MLPs count
  const auto limit_of = [](int64_t T, int64_t h, int64_t f, int slots, int M) { return merge_limit(T, h, f, h / 64, slots, M); };
  CHECK(limit_of(4096, 4096, 16384, 8, 8) == 1 && limit_of(8192, 8192, 32768, 8, 8) == 1);
  CHECK(limit_of(2048, 2048, 8192, 8, 8) == 4 && limit_of(2048, 4096, 16384, 8, 8) == 2);
  CHECK(limit_of(256, 256, 1024, 3, 3) == 3 && limit_of(256, 256, 1024, 64, 64) == kMaxMerge && limit_of(256, 256, 1024, 9, 9) == 5);
  CHECK(limit_of(2048, 2048, 32768, 8, 8) == 1 && limit_of(256, 256, 256, 8, 8) == 1 && limit_of(256, 256, 264, 8, 8) == 8);
  const int refilled[9] = {0, 1, 2, 2, 4, 3, 3, 4, 4};       // fewer slots than microbatches
  for (int p = 1; p <= 8; ++p) CHECK(limit_of(256, 256, 1024, p, 16) == refilled[p]);
  // few slots and several streams: up to 2^20 elements with two or three (2^17 with two and an
  // odd number of microbatches), 2^21 with four
  const auto overlapped = [](int64_t T, int slots, int M, bool overlap = true) { return merge_limit(T, 256, 1024, 4, slots, M, overlap); };
  CHECK(overlapped(4096, 2, 4) == 2 && overlapped(4104, 2, 4) == 1 && overlapped(512, 2, 3) == 2 && overlapped(520, 2, 3) == 1);
  CHECK(overlapped(4096, 3, 4) == 2 && overlapped(4104, 3, 5) == 1 && overlapped(8192, 4, 5) == 4 && overlapped(8200, 4, 5) == 1);
  CHECK(overlapped(8200, 5, 6) == 3 && overlapped(8200, 2, 2) == 2 && overlapped(8200, 4, 4) == 4 && limit_of(4097, 256, 1028, 2, 4) == 2);
  for (int slots = 1; slots <= 8; ++slots)
    for (int M = slots; M <= 9; ++M) CHECK(overlapped(8200, slots, M, false) >= overlapped(8200, slots, M));

  std::vector<MessageSpan> box;
  std::vector<int> here;                       // arrived(i)
  std::vector<SlotRec> slots(6);
  int picked[kMaxMerge];
  const auto span = [&](size_t i) { return box[i]; };
  const auto arrived = [&](size_t i) { return here[i]; };
  const auto add = [&](int kind, int mb, uint64_t in, uint64_t out, bool alone = false, int arr = 1) {
    box.push_back(MessageSpan{kind, mb, alone, in, in + 100, out, out ? out + 100 : 0});
    here.push_back(arr);
  };
  const auto merge = [&](int chosen, int in_flight, int limit, int max) {
    return merge_messages(box.size(), span, arrived, chosen, slots, in_flight, limit, max, picked);
  };
  for (int i = 0; i < 6; ++i) add(0, i, 1000 + 100 * i, 5000 + 100 * i);
  CHECK(merge(0, 0, 6, 4) == 4 && picked[0] == 0 && picked[3] == 3);
  CHECK(merge(0, 0, 3, 8) == 3);               // pipeline_limit
  CHECK(merge(0, 0, 6, 1) == 1);
  slots[2].state = SLOT_AWAIT_WGRAD;           // consecutive free slots only
  CHECK(merge(0, 0, 6, 8) == 2);
  slots[2].state = SLOT_FREE;
  here[1] = 0;                                 // not arrived: passed over
  CHECK(merge(0, 0, 6, 8) == 5 && picked[1] == 2 && picked[4] == 5);
  box[2].alone = true;                         // its completion is waited for: by itself, and no later forward passes it by
  CHECK(merge(0, 0, 6, 8) == 1 && merge(2, 0, 6, 8) == 1);
  here[1] = 1;
  CHECK(merge(0, 0, 6, 8) == 2);
  box[2].alone = false;
  box[3].in = box[1].out + 50; box[3].in_end = box[3].in + 100;        // message 3 reads what message 1 (and 2) writes
  CHECK(merge(0, 0, 6, 8) == 3);
  box[3].in = 1300; box[3].in_end = 1400;
  CHECK(merge(0, 0, 6, 8) == 6);
  box[4].out = box[2].in; box[4].out_end = box[2].in_end;              // message 4 overwrites what message 2 reads
  box[5].out = box[0].out; box[5].out_end = box[0].out_end;            // two results in one buffer
  CHECK(merge(0, 0, 6, 8) == 4);

  // backwards: the microbatches of the slots behind the chosen one's, in slot order, also past a forward between them
  box.clear(); here.clear();
  for (int i = 0; i < 6; ++i) { slots[i].state = SLOT_LIVE; slots[i].mb_id = 10 + i; }
  add(1, 11, 1000, 5000); add(1, 13, 1100, 5100); add(0, 20, 1200, 5200); add(1, 12, 1300, 5300); add(1, 10, 1400, 0);
  CHECK(merge(0, 6, 6, 8) == 3 && picked[1] == 3 && picked[2] == 1);   // 11, 12, 13; 14 is not posted, 10 lies before
  CHECK(merge(4, 6, 6, 2) == 2 && picked[1] == 0);
  box[3].in = 5200; box[3].in_end = 5300;      // 12 reads what the forward posted before it writes
  CHECK(merge(0, 6, 6, 8) == 1);
  slots[2].state = SLOT_AWAIT_WGRAD;
  CHECK(merge(0, 6, 6, 8) == 1);

  // whatever is merged is a subset of what the loop could have taken one by one, in every state
  std::mt19937 rng(9);
  for (int rep = 0; rep < 3000; ++rep) {
    box.clear(); here.clear();
    int in_flight = 0;
    std::set<int> live;
    for (int i = 0; i < 6; ++i) {
      slots[i].state = (int)(rng() % 3);
      slots[i].mb_id = slots[i].state == SLOT_LIVE ? i : -1;
      if (slots[i].state == SLOT_LIVE) { ++in_flight; live.insert(i); }
    }
    const int limit = std::max(in_flight, 1 + (int)(rng() % 6));
    std::set<std::pair<int, int>> posted;
    for (int i = 0; i < 10; ++i) {
      const int kind = (int)(rng() % 2), mb = (int)(rng() % 12);
      if (!posted.insert({kind, mb}).second) continue;
      add(kind, mb, 1000 + 100 * (rng() % 30), 1000 + 100 * (rng() % 30), rng() % 5 == 0, rng() % 4 != 0);
    }
    bool any = false;
    int err = 0;
    const auto msg = [&](size_t i) { return std::make_pair(box[i].kind, box[i].mb_id); };
    const int c = choose_message(box.size(), msg, arrived, slots, in_flight, limit, &any, &err);
    if (c < 0) continue;
    if (box[c].kind == 0 && find_free(slots) < 0) release_awaiting(slots);
    if (box[c].kind == 0 && find_free(slots) < 0) continue;
    const int n = merge(c, in_flight, limit, kMaxMerge);
    CHECK(n >= 1 && picked[0] == c);
    std::set<int> mbs;
    int flying = in_flight;
    const int s0 = box[c].kind == 0 ? find_free(slots) : find_live(slots, box[c].mb_id);
    for (int k = 0; k < n; ++k) {
      const MessageSpan& m = box[picked[k]];
      CHECK(m.kind == box[c].kind && here[picked[k]] == 1 && mbs.insert(m.mb_id).second && (n == 1 || !m.alone));
      CHECK(admissible(m.kind, m.mb_id, slots, flying, limit));
      CHECK(m.kind == 0 ? slots[s0 + k].state == SLOT_FREE : slots[s0 + k].mb_id == m.mb_id);
      if (m.kind == 0) ++flying;
      for (int q = 0; q < k; ++q) {
        const MessageSpan& o = box[picked[q]];
        CHECK(m.out + 100 <= o.out || o.out + 100 <= m.out);
        CHECK(m.out + 100 <= o.in || o.in + 100 <= m.out);
        CHECK(m.in + 100 <= o.out || o.out + 100 <= m.in);
      }
    }
  }
}

void test_two_stages_two_threads() {
  // handles are independent: two host threads each drive a stage of their own (no shared state in the logic)
  auto work = [](unsigned seed) { test_pipeline_limit_and_order(seed); test_bucket_plan(seed); };
  std::thread a(work, 11u), b(work, 12u);
  a.join();
  b.join();
}

}  // namespace

// With the arguments "tile M N K": the GEMM launcher's choice for a problem of one segment (ring tile or -1, and the
// parts of a split over k where a workspace is at hand).
int main(int argc, char** argv) {
  if (argc == 5 && std::string(argv[1]) == "tile") {
    const long M = std::atol(argv[2]), N = std::atol(argv[3]), K = std::atol(argv[4]);
    std::printf("%d %d\n", choose_ring_tile(M, N, (K + 63) / 64, -1, false), choose_split(M, N, K, -1).parts);
    return 0;
  }
  test_pipeline_limit_and_order(1);
  test_arrival_order_decides();
  test_duplicates_and_surplus();
  test_backward_without_forward_never_runs();
  test_wait_limit_is_per_wait();
  test_wgrad_groups();
  test_bucket_plan(2);
  test_addressable_in_place();
  test_workgroup_order();
  test_gemm_tiles();
  test_merged_messages();
  test_two_stages_two_threads();
  std::puts("host logic: all checks passed");
  return 0;
}
