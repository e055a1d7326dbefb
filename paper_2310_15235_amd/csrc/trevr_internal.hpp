// Host-side internals shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>
#include <utility>
#include <vector>

#include "trevr_common.hpp"

namespace trevr {

// Traversal stacks live in LDS: the small one keeps the traversal kernels
// at 8 wavefronts per SIMD (the deepest stacks seen are a few hundred
// entries); a tree whose traversal overflows it switches to the large one.
constexpr int kStackSmall = 1024;
constexpr int kStackLarge = 8192;
constexpr uint32_t kCutCap = 2048;   // cut-list entries per bucket the buffer is sized for
constexpr size_t kStageCap = 4096;   // most staging words per bucket for the p-p set
constexpr uint32_t kNoRuns = 0xFFFFFFFFu;   // a staged p-p set that did not fit
// Staged runs (two words each after a two-word header) sorted in LDS: their
// count bound and the bits of a staging index in a sort key.
constexpr uint32_t kSortRuns = 2048;
constexpr int kSortIdxBits = 11;
static_assert((kStageCap - 2) / 2 <= kSortRuns && kSortRuns <= (1u << kSortIdxBits),
              "staged runs must fit the sort");

// Bump allocator over a caller-owned buffer (base == nullptr: size only).
struct Carve {
  char* base;
  size_t off = 0;
  explicit Carve(void* b) : base((char*)b) {}
  template <class T> T* take(size_t count) {
    off = (off + 255) & ~(size_t)255;
    T* p = base ? (T*)(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

// Elements of the subtrees whose moments one workgroup forms, and the mark
// of larger cells in TreeBufs::depth.
constexpr int kSubtree = 512;
constexpr uint32_t kDeepBig = 128;
static_assert(kMaxLevels + 3 < (int)kDeepBig, "a depth and its mark share a byte");
constexpr int kInfoWords = 4;

// Counters of a build on the device (zeroed at its start).
struct BuildWords {
  unsigned long long diff;              // bits in which some keys differ
  uint32_t resort;                      // the short sort left a run unsorted
  uint32_t nroots;                      // entries of roots
  uint32_t bigdepth;                    // levels holding cells of more than kSubtree elements
  uint32_t lcnt[kMaxLevels + 3];        // nodes per depth
  uint32_t lcur[kMaxLevels + 3];        // nodes of each depth placed
};
static_assert(sizeof(BuildWords) % 4 == 0 && sizeof(BuildWords) / 4 <= 256, "cleared by 256 threads");

// Floats of an element's packed record (a multiple of four).
__host__ __device__ inline int rec_floats(int B) { return (5 + 2 * B + 3) & ~3; }

// Tiles of the radix sort: 1024 elements each up to this many, 4096 above.
constexpr int64_t kSortTileSwitch = 1 << 19;
inline int64_t sort_tiles(int64_t n) {
  const int64_t tile = n <= kSortTileSwitch ? 1024 : 4096;
  return (n + tile - 1) / tile;
}

// Mutable device pointers of a tree (same memory the DevTree views).
struct TreeBufs {
  double* hdr;
  uint32_t* bbox_u;           // ordered-uint min/max of x, y, z
  BuildWords* words;          // counters of the build
  uint64_t *keys, *keys_alt;  // sorted; in input order (build only)
  uint32_t *vals, *vals_alt, *top, *top_alt, *hist, *dtot;   // radix passes
  float* rec;                 // [n][rec_floats(B)] elements packed for the gather
  uint32_t *starts, *tsum;    // nodes starting at each slot, then their prefix sum
  uint32_t* roots;            // subtrees of at most kSubtree elements
  uint32_t *r_end, *r_split, *r_par;   // radix tree (share the sort's buffers)
  float *x, *y, *z, *m, *rho, *kappa, *lum;
  double *h, *lbol;
  uint32_t* perm;
  uint32_t* b_pre;            // nodes grouped by depth (see DevTree)
  int32_t *b_lown, *b_split;
  uint4* nk;
  uint2* nlink;
  uint32_t* next;
  uint8_t* depth;             // per node; kDeepBig marks more than kSubtree elements
  double4 *cen, *sl;
  double *Lb, *kmass, *alpha64;
  float* alpha32;
  double* ray_n;
  int32_t* ray_class;
  int32_t* ray_anti;          // [nray] ray of the opposite direction
  uint64_t* rcand;            // candidate rays (see DevTree)
  double *csrc_d, *csrc_a;    // complex source model: [node][nray] lengths,
                              // [node][nray][B] absorption (null when off)
  double* geom;               // [64][nclass][3]: log w1, log w12, chord / L
  uint32_t* err;
  unsigned long long* counters;
  DevTree* dev;               // device copy of the tree's DevTree (one-scene table)
  uint2* levels;              // [kMaxLevels + 3] BFS index ranges per depth
  uint32_t* info;             // [kInfoWords] {sort again, nodes, depth, levels of large
                              // cells}, behind levels: read back together
};

// Direction tables of an N_side: centres, classes (rays sharing |n_x|,
// |n_y|, |n_z| see the same transmission averages) and the combine
// geometry per prefix length and class.
struct DirTables {
  int nside = 0, nray = 0, nclass = 0;
  std::vector<double> ray_n;      // [nray][3]
  std::vector<int32_t> ray_class; // [nray]
  std::vector<int32_t> ray_anti;  // [nray] ray of the opposite direction
  std::vector<double> geom;       // [64][nclass][3]
  std::vector<double> block;      // ray_n, geom, ray_class, ray_anti: uploaded in one copy
};
// Doubles of DirTables::block.
inline size_t dir_block(int nray, int nclass) {
  return 3 * (size_t)nray + (size_t)kMaxLevels * nclass * 3 + (size_t)nray;
}
DirTables make_dir_tables(int nside);
// The tables of an N_side, made on first use and kept (one set per N_side up
// to kMaxNside; constants of the method).
const DirTables& dir_tables(int nside);
// Their block in pinned memory, for uploads that do not wait (made on first
// use; the pageable block where pinned memory cannot be had).
const double* dir_block_pinned(int nside);

// Pinned blocks of kHostWords words for the readbacks of trees: a few are
// kept when trees go, since a program that builds a tree per step would
// otherwise allocate and free pinned memory in each (any thread; a block is
// given back after its tree's stream is synchronised).
trevr_status pinned_take(uint32_t** out);
void pinned_give(uint32_t* block);

size_t layout_tree(const trevr_params& p, int64_t n, int nclass, void* base, TreeBufs* out);

}  // namespace trevr

// What the scratch holds after a compute_J (or a backward that redid the
// setup): bucket lists, p-p radii and lists, the cut lists of the last
// batch and the p-p columns for the active set with this fingerprint.
struct FwdState {
  bool valid;
  const void* scratch;
  uint64_t epoch;       // the library's write to that scratch that left it
  uint64_t hash;
  uint32_t nb;
  uint64_t near_total, tpp_total, ptau_total, jraw_total;
  bool cuts_kept;       // the cut buffer holds every bucket's cut list
  uint32_t cut_stride;  // ... at this many entries per bucket
  bool kept;            // far-source optical depths of the forward are in the scratch
};

namespace trevr {
// Kernel timing of a tree or a forest (trevr_profile_enable,
// trevr_forest_profile_enable): HIP event pairs recorded on the owner's
// stream around launches, folded into per-slot totals when read.
struct Prof {
  bool on = false;
  std::vector<hipEvent_t> pool;
  size_t used = 0;
  std::vector<std::pair<int, std::pair<hipEvent_t, hipEvent_t>>> pending;
  double ms[TREVR_PROF_SLOTS] = {};
  int64_t calls[TREVR_PROF_SLOTS] = {};
};
}  // namespace trevr

struct trevr_tree {
  uint64_t magic;
  trevr_params p;
  int64_t n;
  int32_t B, nray, nclass, depth;
  int64_t num_nodes, num_leaves;
  hipStream_t stream;
  hipEvent_t built;                         // end of the build's last kernels (or null)
  bool building;                            // they may still run: other streams wait for it
  void* ws;
  size_t ws_bytes;
  trevr::TreeBufs buf;
  trevr::DevTree dev;
  const trevr::DirTables* dirs;             // of its N_side (kept by the library)
  std::vector<std::pair<uint32_t, uint32_t>> levels;  // BFS index ranges per depth
  size_t scratch_needed;
  bool counters_valid;
  uint32_t* host_u32;                       // pinned readback buffer (kHostWords)
  FwdState fwd;
  bool stack_large;                         // traversals need the large LDS stack
  uint32_t cut_default;                     // cut-list entries per bucket to try first
  uint32_t stage_limit;                     // most staging words per bucket for p-p sets
  bool adjoint_room;                        // compute_J asks for the adjoint's scratch too
  int64_t receivers;                        // active elements, at most (for the estimate)
  trevr::Prof prof;                         // kernel timing (trevr_profile_enable)
};

namespace trevr {
constexpr int kHostWords = 512;
// What the p-p sources' parts take of a scratch's fixed part.
size_t parts_bytes(int64_t leaves);
trevr_status set_error(trevr_status s, const std::string& msg);
trevr_status hip_check(hipError_t e, const char* what);
trevr_status build_tree_impl(trevr_tree* t, const float* x, const float* y, const float* z,
                             const float* m, const float* rho, const float* kappa,
                             const float* lum);
// (fixed: the scratch can neither grow nor serve an adjoint)
trevr_status compute_J_impl(trevr_tree* t, const uint8_t* active, const float* bg, double* J,
                            void* scratch, size_t scratch_bytes, bool fixed);
trevr_status compute_J_backward_impl(trevr_tree* t, const uint8_t* active, const float* bg,
                                     const double* gJ, double* gL, double* gkappa, double* grho,
                                     void* scratch, size_t scratch_bytes);
// Clears words of device memory with a kernel (a captured graph may hold it).
trevr_status zero_words(hipStream_t st, void* p, size_t words);
size_t scratch_fixed_bytes(int64_t n);
// Scratch that a compute_J and its adjoint are likely to need (adjoint_room).
size_t adjoint_scratch_guess(const trevr_tree* t);
// Every call that writes a scratch buffer takes a new epoch for it; a
// state recorded at epoch e is still in the buffer iff no call (on any
// tree) has written it since.
uint64_t scratch_mark(const void* scratch);
bool scratch_unchanged(const void* scratch, uint64_t epoch);
// Record an event pair on stream st around a phase (no-op unless profiling
// is on; p may be null).
hipEvent_t prof_begin(Prof* p, hipStream_t st);
void prof_end(Prof* p, hipStream_t st, int slot, hipEvent_t begin);
inline hipEvent_t prof_begin(trevr_tree* t) { return t ? prof_begin(&t->prof, t->stream) : nullptr; }
inline void prof_end(trevr_tree* t, int slot, hipEvent_t begin) {
  if (t) prof_end(&t->prof, t->stream, slot, begin);
}
// Start (clearing the totals) or stop recording; creates the event pool.
trevr_status prof_enable(Prof* p, hipStream_t st, bool on);
// Synchronise st and copy the totals out (any pointer may be null).
trevr_status prof_read(Prof* p, hipStream_t st, double* ms, int64_t* launches);
void prof_destroy(Prof* p);
}  // namespace trevr
