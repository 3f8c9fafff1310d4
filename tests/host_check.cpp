// Checks of the library's host side on the stand-in runtime (host_hip.h): what
// a call leaves behind when memory runs out.  One check per name; exits with
// the number of expectations that failed.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <random>

#include "host_hip.h"
#include "sccg.h"
#include "sccg_common.h"

static int failed = 0;
#define EXPECT(cond, ...)                              \
  do {                                                 \
    if (!(cond)) {                                     \
      ++failed;                                        \
      printf("%s:%d: %s: ", __FILE__, __LINE__, #cond); \
      printf(__VA_ARGS__);                             \
      printf("\n");                                    \
    }                                                  \
  } while (0)

static int64_t* const off = (int64_t*)((uintptr_t)1 << 45);  // device arrays that no allocation of the library holds
static int32_t* const arr = (int32_t*)((uintptr_t)1 << 46);
static sccg_polys polys(int64_t n) { return sccg_polys{n, off, arr}; }

// ---------------------------------------------------------------- the join
static int64_t join_cells, join_entries, join_pairs;  // what the kernels would find
static int join(sccg_ctx* c, int64_t n, int64_t cells, int64_t entries, int64_t sets = 1) {
  join_cells = cells;
  join_entries = entries;
  join_pairs = 5;
  const sccg_polys A = polys(n), B = polys(n);
  int64_t total = -1;
  const int r = sccg_join_sets(c, &A, &B, sets, off, off, 0, 100, arr, arr, off, &total);
  if (r == SCCG_OK) EXPECT(total == join_pairs, "%lld pairs", (long long)total);
  return r;
}
static void watch_join(const Launch& l) {
  if (l.is("k_join_cellsILb0")) {  // counts are added to what is there
    const int64_t room = l.arg<int64_t>(7);
    EXPECT(fake.cleared(l.arg<void*>(8), (size_t)room * 4), "counts of %lld cells", (long long)room);
  }
  if (l.is("k_join_write")) {
    int64_t* sizes = l.arg<int64_t*>(8);
    sizes[0] = join_cells;
    sizes[1] = join_entries;
    sizes[2] = join_pairs;
  }
}

// Whichever allocation of a larger call is refused, the next call finds its
// counts cleared.
static void join_out_of_memory() {
  fake.on_launch = watch_join;
  for (int k = 0;; ++k) {
    sccg_ctx* c = nullptr;
    EXPECT(sccg_create(&c, 0, nullptr, nullptr) == SCCG_OK, "create");
    EXPECT(join(c, 1000, 500, 900) == SCCG_OK, "small join");
    fake.fail_at = fake.allocations + k;
    const int r = join(c, 100000, 50000, 90000);
    const bool refused = fake.allocations > fake.fail_at;
    fake.fail_at = -1;
    EXPECT(r == (refused ? SCCG_E_NOMEM : SCCG_OK), "allocation %d refused: %d", k, r);
    EXPECT(join(c, 100000, 50000, 90000) == SCCG_OK, "after allocation %d was refused: %s", k, sccg_last_error(c));
    sccg_destroy(c);
    if (!refused) {
      EXPECT(k >= 9, "only %d allocations", k);
      return;
    }
  }
}

// A join is launched for the cells that it and the calls shortly before it have:
// small ones after a large one are soon launched as small again, and a large one
// every other call is not run twice.
static void join_launch_sizes() {
  unsigned scan = 0;  // workgroups of the scan of the cells' counts
  long runs = 0;
  fake.on_launch = [&](const Launch& l) {
    watch_join(l);
    if (l.is("k_scan_write") || l.is("k_scan_one")) {
      if (l.is("ILb1E")) scan = l.grid;
    }
    if (l.is("k_join_write")) runs += 1;
  };
  sccg_ctx* c = nullptr;
  EXPECT(sccg_create(&c, 0, nullptr, nullptr) == SCCG_OK, "create");
  EXPECT(join(c, 2000, 900, 4000) == SCCG_OK && scan == 1, "%u workgroups for a small join", scan);
  EXPECT(join(c, 2000, 10000000, 4000) == SCCG_OK, "large join");
  EXPECT(scan > 1000, "%u workgroups for a large join", scan);
  const long before = runs;
  for (int k = 0; k < 40; ++k) EXPECT(join(c, 2000, 900, 4000) == SCCG_OK, "small join");
  EXPECT(scan == 1, "%u workgroups for the 40th small join", scan);
  EXPECT(runs == before + 40, "%ld runs of 40 joins", runs - before);
  EXPECT(join(c, 2000, 10000000, 4000) == SCCG_OK, "large join");
  const long pairs = runs;
  for (int k = 0; k < 50; ++k) {
    EXPECT(join(c, 2000, 900, 4000) == SCCG_OK, "small join");
    EXPECT(join(c, 2000, 10000000, 4000) == SCCG_OK, "large join");
  }
  EXPECT(runs == pairs + 100, "%ld runs of a hundred joins", runs - pairs);
  sccg_destroy(c);
}

// A refused allocation is reported once: the next call of any kind works.
static void errors_are_reported_once() {
  fake.on_launch = watch_join;
  const sccg_polys P = polys(100000);
  for (int k = 0; k < 3; ++k) {
    sccg_ctx* c = nullptr;
    fake.fail_at = fake.allocations + k;
    EXPECT(sccg_create(&c, 0, nullptr, nullptr) == SCCG_E_NOMEM, "allocation %d of a context", k);
    fake.fail_at = -1;
    EXPECT(sccg_create(&c, 0, nullptr, nullptr) == SCCG_OK, "create");
    EXPECT(join(c, 1000, 500, 900) == SCCG_OK, "after allocation %d of a context was refused: %s", k, sccg_last_error(c));
    sccg_destroy(c);
  }
  for (int first = 0; first < 5; ++first)
    for (int second = 0; second < 5; ++second) {
      sccg_ctx* c = nullptr;
      EXPECT(sccg_create(&c, 0, nullptr, nullptr) == SCCG_OK, "create");
      auto call = [&](int k) {
        int64_t* o = off;
        if (k == 0) return sccg_area_pairs(c, &P, &P, 1000, arr, arr, o, o, SCCG_BATCHED);
        if (k == 1) return sccg_area_pairs(c, &P, &P, 1000, arr, arr, o, o, SCCG_PLAIN);
        if (k == 2) return join(c, 1000, 500, 900);
        if (k == 3) return sccg_relate_pairs(c, &P, &P, 1000, arr, arr, o, (uint32_t*)arr);
        return sccg_jaccard_sets(c, 10, o, o, o, 0, o, o, o, (double*)o, nullptr);
      };
      fake.fail_at = fake.allocations;
      EXPECT(call(first) == SCCG_E_NOMEM, "call %d", first);
      fake.fail_at = -1;
      EXPECT(call(second) == SCCG_OK, "call %d after call %d had no memory: %s", second, first, sccg_last_error(c));
      sccg_destroy(c);
    }
}

// ------------------------------------------------------------- rings' tiles
// A call whose tiles cannot be allocated does without, and later ones too: no
// waits, no dropped graph, no further attempts, until the scratch is asked for
// again; smaller tiles that are there stay.
static void tiles_out_of_memory() {
  sccg_params p;
  memset(&p, 0, sizeof(p));
  p.sweep_pair_box = 2;
  sccg_ctx* c = nullptr;
  EXPECT(sccg_create(&c, 0, (void*)1, &p) == SCCG_OK, "create");
  const int64_t pairs = 1000000, few = 10000, many = 400000;  // rings of a set
  auto call = [&](int64_t n) {
    const sccg_polys P = polys(n);
    const int r = sccg_area_pairs(c, &P, &P, pairs, arr, arr, off, off, SCCG_BATCHED);
    EXPECT(r == SCCG_OK, "%lld rings: %s", (long long)n, sccg_last_error(c));
  };
  call(few);
  EXPECT(fake.launched("k_ring_tiles") == 1, "no tiles of few rings");
  fake.most = (size_t)64 << 20;
  call(many);
  EXPECT(fake.refused == 1, "%ld refused", fake.refused);
  EXPECT(fake.launched("k_ring_tiles") == 1, "tiles without memory");
  const FakeHip before = fake;
  for (int k = 0; k < 12; ++k) call(many);
  call(many - 1);  // of what was asked for there was too little
  EXPECT(fake.captures == before.captures + 1, "%ld captures", fake.captures - before.captures);
  EXPECT(fake.replays == before.replays + 6, "%ld replays", fake.replays - before.replays);
  EXPECT(fake.waits == before.waits, "%ld waits", fake.waits - before.waits);
  EXPECT(fake.refused <= before.refused + 1, "%ld attempts", fake.refused - before.refused);
  call(few);
  EXPECT(fake.allocations == before.allocations + (fake.refused - before.refused), "the tiles of few rings were given up");
  EXPECT(fake.launched("k_ring_tiles") == 2, "no tiles of few rings");
  // asked for again: refused, then, with memory, there
  long refused = fake.refused;
  EXPECT(sccg_reserve(c, many, many, pairs) == SCCG_OK, "reserve");
  EXPECT(fake.refused == refused + 1, "%ld attempts", fake.refused - refused);
  fake.most = ~(size_t)0;
  call(many);
  EXPECT(fake.launched("k_ring_tiles") == 2, "memory looked for by a call");
  EXPECT(sccg_reserve(c, many, many, pairs) == SCCG_OK, "reserve");
  call(many);
  EXPECT(fake.launched("k_ring_tiles") == 3, "no tiles after reserve");
  sccg_destroy(c);
}
// So do calls after set_params.
static void tiles_tried_again_with_new_parameters() {
  sccg_params p;
  memset(&p, 0, sizeof(p));
  p.sweep_pair_box = 2;
  sccg_ctx* c = nullptr;
  EXPECT(sccg_create(&c, 0, (void*)1, &p) == SCCG_OK, "create");
  const sccg_polys P = polys(400000);
  auto call = [&]() { EXPECT(sccg_area_pairs(c, &P, &P, 1000000, arr, arr, off, off, SCCG_BATCHED) == SCCG_OK, "%s", sccg_last_error(c)); };
  fake.most = (size_t)64 << 20;
  call();
  EXPECT(fake.launched("k_ring_tiles") == 0, "tiles without memory");
  fake.most = ~(size_t)0;
  EXPECT(sccg_set_params(c, &p) == SCCG_OK, "set_params");
  call();
  EXPECT(fake.launched("k_ring_tiles") == 1, "no tiles");
  sccg_destroy(c);
}

// ---------------------------------------------------------------- the graph
// Captured with the first call's arguments, replayed with the same, and given
// up only for others that come eight times in a row.
static void graph_of_repeated_arguments() {
  sccg_ctx* c = nullptr;
  EXPECT(sccg_create(&c, 0, (void*)1, nullptr) == SCCG_OK, "create");
  const sccg_polys P = polys(1000);
  long sweeps = 0;
  auto call = [&](int out, long captures, long replays, const char* what) {
    const FakeHip before = fake;
    EXPECT(sccg_area_pairs(c, &P, &P, 1000, arr, arr, off + out, off, SCCG_BATCHED) == SCCG_OK, "%s", sccg_last_error(c));
    EXPECT(fake.captures == before.captures + captures, "%s: %ld captures", what, fake.captures - before.captures);
    EXPECT(fake.replays == before.replays + replays, "%s: %ld replays", what, fake.replays - before.replays);
    sweeps += captures || !replays;  // kernels launched, into the graph or the stream
    EXPECT(fake.launched("k_batch_sweep") == sweeps, "%s: %ld sweeps", what, (long)fake.launched("k_batch_sweep"));
  };
  call(0, 1, 1, "first call");
  call(0, 0, 1, "the same");
  for (int k = 0; k < 3; ++k) {
    call(1, 0, 0, "others");
    call(2, 0, 0, "others again");
  }
  call(0, 0, 1, "the graph's");
  for (int k = 0; k < 7; ++k) call(2, 0, 0, "others after it");
  call(0, 0, 1, "the graph's again");
  for (int k = 0; k < 7; ++k) call(2, 0, 0, "others, counted anew");
  call(2, 1, 1, "eight in a row");
  call(2, 0, 1, "the new graph's");
  for (int k = 0; k < 7; ++k) call(0, 0, 0, "the old graph's");
  call(0, 1, 1, "eight of those");
  sccg_destroy(c);
}

// ---------------------------------------------------------------- launches
// A dispatch has fewer than 2^32 threads: whatever sizes the entry points
// take, their launches do.
static void launches_within_a_dispatch() {
  fake.on_launch = watch_join;
  const int64_t most = ((int64_t)1 << 31) - 1;
  for (const int64_t n : {((int64_t)1 << 24) + 1, (int64_t)1 << 27, (int64_t)1 << 28, (int64_t)1 << 29, most}) {
    sccg_ctx* c = nullptr;
    EXPECT(sccg_create(&c, 0, nullptr, nullptr) == SCCG_OK, "create");
    const sccg_polys P = polys(n);
    const int64_t pairs = n == most ? (int64_t)1 << 34 : n;
    EXPECT(sccg_validate_polys(c, &P, off) == SCCG_OK, "validate %lld: %s", (long long)n, sccg_last_error(c));
    EXPECT(sccg_area_pairs(c, &P, &P, n, arr, arr, off, off, SCCG_PLAIN) == SCCG_OK, "plain %lld: %s", (long long)n, sccg_last_error(c));
    EXPECT(sccg_area_pairs(c, &P, &P, n, arr, arr, off, off, SCCG_BATCHED) == SCCG_OK, "batched %lld: %s", (long long)n, sccg_last_error(c));
    EXPECT(join(c, n, n, n) == SCCG_OK, "join %lld: %s", (long long)n, sccg_last_error(c));
    EXPECT(join(c, 1000, n, n, n) == SCCG_OK, "join of %lld sets: %s", (long long)n, sccg_last_error(c));
    EXPECT(sccg_relate_pairs(c, &P, &P, pairs, arr, arr, off, (uint32_t*)arr) == SCCG_OK, "relate %lld: %s", (long long)pairs,
           sccg_last_error(c));
    EXPECT(sccg_jaccard_sets(c, n, off, off, off, 0, off, off, off, (double*)off, nullptr) == SCCG_OK, "jaccard of %lld sets: %s",
           (long long)n, sccg_last_error(c));
    for (const auto& k : fake.too_large) EXPECT(false, "%lld: %s", (long long)n, k.c_str());
    fake.too_large.clear();
    sccg_destroy(c);
  }
}

// ------------------------------------------------------------------- lists
// Whatever the pairs, the grids and the shares' runs: a stream's pairs fit its
// parts of the lists, and the parts the room that is allocated for the pairs.
static void lists_hold_their_pairs() {
  using namespace sccg;
  std::mt19937_64 rng(1);
  auto below = [&](int64_t n) { return (int64_t)(rng() % (uint64_t)n); };
  for (int k = 0; k < 3000000 && failed < 10; ++k) {
    const int64_t n = std::max<int64_t>(1, (int64_t)exp((double)below(1000000) / 1e6 * log(2147483647.0)));
    const int64_t cus = int64_t(32) << below(4), chunk = 1 + below(64);
    const int64_t sweep = std::min(cus * (1 + below(8)), (n + 3) / 4), medium = std::min(cus * (1 + below(16)), n);
    const int64_t cap = stream_cap_of(sweep, 4, most_share(n, sweep * 4, chunk)), run = run_cap_of(n, medium);
    // every eighth long pair, and shares of the others that differ by one
    const int64_t longs = below(3) == 0 ? n : below(n + 1), rest = n - longs, waves = 2 * medium;
    const int64_t share = (medium + kStreams - 1) / kStreams * 2 * ((rest + waves - 1) / waves);
    const int64_t listed = medium < kStreams ? n : std::min(n, (longs + kStreams - 1) / kStreams + std::min(rest, share));
    EXPECT(listed <= run, "%lld pairs, %lld long, %lld workgroups: %lld in %lld", (long long)n, (long long)longs, (long long)medium,
           (long long)listed, (long long)run);
    const int64_t room = pair_list_room(n + below(n / 4 + 2));
    EXPECT((kLptBuckets + 1) * kStreams * cap + kLptBuckets * kStreams * run <= room, "%lld pairs, %lld and %lld workgroups", (long long)n,
           (long long)sweep, (long long)medium);
    // the pairs that the rings' tiles leave stand where the persistent kernel's will
    if (n >= kRingTilePairs) EXPECT(cap <= kLptBuckets * run, "%lld pairs", (long long)n);
  }
}

int main(int argc, char** argv) {
  static const struct {
    const char* name;
    void (*run)();
  } checks[] = {
      {"join_out_of_memory", join_out_of_memory},
      {"join_launch_sizes", join_launch_sizes},
      {"errors_are_reported_once", errors_are_reported_once},
      {"tiles_out_of_memory", tiles_out_of_memory},
      {"graph_of_repeated_arguments", graph_of_repeated_arguments},
      {"launches_within_a_dispatch", launches_within_a_dispatch},
      {"lists_hold_their_pairs", lists_hold_their_pairs},
      {"tiles_tried_again_with_new_parameters", tiles_tried_again_with_new_parameters},
  };
  for (const auto& k : checks)
    if (argc > 1 && !strcmp(argv[1], k.name)) {
      k.run();
      return failed > 100 ? 100 : failed;
    }
  printf("no such check\n");
  return 101;
}
