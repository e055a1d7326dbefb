// The C ABI's host code in whole calls, on the runtime of fake_hip.cpp: what
// the calls wait for and the sizes that they ask for.  Run with the name of a
// case; exit status 0 when it holds.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "../include/trevr2.h"
#include "fake_hip.h"

namespace {
int failures = 0;
#define EXPECT(c)                                        \
  do {                                                   \
    if (!(c)) {                                          \
      std::printf("FAIL line %d: %s\n", __LINE__, #c);   \
      ++failures;                                        \
    }                                                    \
  } while (0)

void* const A = (void*)0x1000;   // streams
void* const B = (void*)0x2000;

// The level table and counts that a build reads back, as (67 ranges, {sort
// again, nodes, depth, levels of large cells}), for a tree of two levels of
// large cells over four buckets; every other readback is left zero but for
// its second word: a compute's active buckets.
constexpr size_t kLevelBytes = (2 * 67 + 4) * sizeof(uint32_t);
uint32_t active_buckets = 0;
void readback(void* dst, const void*, size_t bytes) {
  uint32_t* w = (uint32_t*)dst;
  std::memset(w, 0, bytes);
  if (bytes == kLevelBytes) {
    const uint32_t ends[4] = {0, 1, 3, 7};
    for (int d = 0; d < 67; ++d) {
      w[2 * d] = d < 3 ? ends[d] : 7;
      w[2 * d + 1] = d < 3 ? ends[d + 1] : 7;
    }
    w[134] = 0;
    w[135] = 7;
    w[136] = 3;
    w[137] = 2;
  } else if (bytes > 8) {
    w[1] = active_buckets;
  }
}

struct Case {
  trevr_params p{};
  int64_t n;
  size_t tree_bytes = 0, scratch_bytes = 0;
  // never read: no kernel runs
  std::unique_ptr<char[]> ws, scratch;
  float in[1];
  double out[1];
  trevr_tree* t = nullptr;
  explicit Case(uint32_t flags = TREVR_NEAR_FIELD, int bands = 1, int nside = 1, int64_t size = 4000)
      : n(size) {
    p.nside = nside;
    p.leaf_size = 8;
    p.n_bands = bands;
    p.flags = flags;
    p.theta = 0.75;
    EXPECT(trevr_workspace_bytes(&p, n, &tree_bytes, &scratch_bytes) == TREVR_OK);
    ws.reset(new char[tree_bytes]);
    scratch.reset(new char[scratch_bytes]);
    fake::on_readback = readback;
  }
  trevr_status build(void* st) {
    const float* x = in;
    return trevr_build_tree(&p, n, x, x, x, x, x, x, x, ws.get(), tree_bytes, st, &t);
  }
  trevr_status forward(void* st, size_t bytes) {
    return trevr_compute_J(t, nullptr, in, out, scratch.get(), bytes, st);
  }
  size_t needed() {
    size_t b = 0;
    EXPECT(trevr_scratch_needed(t, &b) == TREVR_OK);
    return b;
  }
};

// A tree built on one stream and used on another, or given up: nothing may
// run beside the build's last kernels.
void stream_order() {
  using Call = std::function<trevr_status(Case&)>;
  const Call calls[] = {
      [](Case& c) { return c.forward(B, c.scratch_bytes); },
      [](Case& c) { return trevr_compute_J_noalloc(c.t, nullptr, nullptr, c.out, B); },
      [](Case& c) {
        double* o = c.out;
        return trevr_compute_J_backward(c.t, nullptr, nullptr, o, o, o, o, c.scratch.get(),
                                        c.scratch_bytes, B);
      },
      [](Case& c) {   // refused before anything is launched, then another stream
        EXPECT(c.forward(B, 16) == TREVR_E_CAPACITY);
        return c.forward((void*)0x3000, c.scratch_bytes);
      },
  };
  for (const Call& call : calls) {
    fake::reset();
    Case c;
    EXPECT(c.build(A) == TREVR_OK);
    EXPECT(call(c) == TREVR_OK);
    EXPECT(fake::loose_operations() == 0);
    EXPECT(trevr_tree_destroy(c.t) == TREVR_OK);
    EXPECT(fake::host_waited_for(A));
  }
  // given up on another stream than its own, which never ran
  fake::reset();
  Case c;
  EXPECT(c.build(A) == TREVR_OK);
  EXPECT(c.forward(B, 16) == TREVR_E_CAPACITY);
  EXPECT(trevr_tree_destroy(c.t) == TREVR_OK);
  EXPECT(fake::host_waited_for(A));
}

// Scratch of the kept depths, per band count: each group of 64 rays of each
// bucket keeps what fits one window of the far-field kernels.
void kept_depths() {
  for (int bands = 1; bands <= 16; ++bands)
    for (int nside : {1, 4})
      for (uint32_t bg : {0u, (uint32_t)TREVR_BACKGROUND}) {
        const size_t window = bands == 1 ? 512 : bands <= 3 ? 448 : bands == 4 ? 192 : bands == 6 ? 224 : 256;
        const size_t rays = 12 * nside * nside, groups = (rays + 63) / 64;
        size_t need[2];
        for (uint32_t keep : {0u, (uint32_t)TREVR_KEEP_DEPTHS}) {
          fake::reset();
          active_buckets = 3;
          Case c(TREVR_NEAR_FIELD | bg | keep, bands, nside);
          EXPECT(c.build(A) == TREVR_OK);
          EXPECT(trevr_compute_J(c.t, nullptr, c.in, c.out, c.scratch.get(),
                                 c.scratch_bytes, A) == TREVR_OK);
          need[keep != 0] = c.needed();
          EXPECT(trevr_tree_destroy(c.t) == TREVR_OK);
        }
        size_t kept = active_buckets * groups * window * bands * sizeof(float);
        if (bg) kept = (kept + 255) / 256 * 256 + active_buckets * rays * bands * sizeof(float);
        EXPECT(need[1] - need[0] == kept);
      }
  active_buckets = 0;
}

// Room for an adjoint is asked for where one can follow in the same scratch: not
// in the fixed array (which cannot grow), nor with the complex source model.
void adjoint_room() {
  fake::reset();
  Case c(TREVR_NEAR_FIELD, 1, 1, 4000000);   // accumulators of 96 MB, past the array
  EXPECT(c.build(A) == TREVR_OK);
  EXPECT(trevr_compute_J_noalloc(c.t, nullptr, nullptr, c.out, A) == TREVR_OK);
  EXPECT(c.forward(A, c.scratch_bytes) == TREVR_OK);
  const size_t plain = c.needed();
  EXPECT(trevr_tree_tune(c.t, TREVR_TUNE_ADJOINT, 1) == TREVR_OK);
  EXPECT(trevr_compute_J_noalloc(c.t, nullptr, nullptr, c.out, A) == TREVR_OK);
  EXPECT(c.forward(A, plain) == TREVR_E_CAPACITY);
  EXPECT(c.needed() >= plain + 3 * sizeof(double) * (size_t)c.n);
  EXPECT(trevr_tree_destroy(c.t) == TREVR_OK);
  fake::reset();
  Case d(TREVR_NEAR_FIELD | TREVR_COMPLEX_SRC, 1, 1);
  EXPECT(d.build(A) == TREVR_OK);
  EXPECT(trevr_tree_tune(d.t, TREVR_TUNE_ADJOINT, 1) == TREVR_OK);
  EXPECT(d.needed() == 0);
  EXPECT(d.forward(A, d.scratch_bytes) == TREVR_OK);
  const size_t with = d.needed();
  EXPECT(trevr_tree_tune(d.t, TREVR_TUNE_ADJOINT, 0) == TREVR_OK);
  EXPECT(d.forward(A, d.scratch_bytes) == TREVR_OK);
  EXPECT(d.needed() == with);
  EXPECT(trevr_tree_destroy(d.t) == TREVR_OK);
}

// The estimate for a forward and its adjoint takes the receivers that it is told
// of: two columns per ray and band of each.
void adjoint_estimate() {
  const size_t rays = 48, bands = 2;
  size_t need[3];
  const int64_t told[3] = {-1, 4000, 400};   // -1: nothing said, every element
  for (int k = 0; k < 3; ++k) {
    fake::reset();
    Case c(TREVR_NEAR_FIELD, bands, 2);
    EXPECT(c.build(A) == TREVR_OK);
    if (told[k] >= 0) EXPECT(trevr_tree_tune(c.t, TREVR_TUNE_RECEIVERS, told[k]) == TREVR_OK);
    EXPECT(trevr_tree_tune(c.t, TREVR_TUNE_ADJOINT, 1) == TREVR_OK);
    need[k] = c.needed();
    EXPECT(trevr_tree_tune(c.t, TREVR_TUNE_RECEIVERS, -1) == TREVR_E_INVALID);
    EXPECT(trevr_tree_tune(c.t, TREVR_TUNE_RECEIVERS, c.n + 1) == TREVR_E_INVALID);
    EXPECT(trevr_tree_destroy(c.t) == TREVR_OK);
  }
  EXPECT(need[0] == need[1]);
  const size_t less = (4000 - 400) * rays * bands * 2 * sizeof(float);
  EXPECT(need[2] + less <= need[1]);
}

const std::map<std::string, void (*)()> cases = {
    {"adjoint_estimate", adjoint_estimate},
    {"adjoint_room", adjoint_room},
    {"kept_depths", kept_depths},
    {"stream_order", stream_order},
};
}  // namespace

int main(int argc, char** argv) {
  const auto it = argc == 2 ? cases.find(argv[1]) : cases.end();
  if (it == cases.end()) {
    for (const auto& c : cases) std::printf("%s\n", c.first.c_str());
    return 2;
  }
  it->second();
  std::printf("%s: %d failures\n", argv[1], failures);
  return failures ? 1 : 0;
}
