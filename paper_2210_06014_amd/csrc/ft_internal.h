// Internal structures shared by the host plan, the kernels and the C-ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "fastertucker.h"

namespace ft {

// Factor-pass work item: a whole light row (kind LIGHT), the first chunk of
// a heavy row (HEAD, result written to the row's head vector) or a later
// chunk of a heavy row (COMPOSE, its affine map written to a map slot).
enum : int32_t { ITEM_LIGHT = 0, ITEM_HEAD = 1, ITEM_COMPOSE = 2 };

struct FItem {
  int64_t start;  // first CSR position
  int32_t len;    // elements (0 for padding)
  int32_t row;    // row of the updated mode
  int32_t slot;   // head-vector slot (HEAD) or map slot (COMPOSE)
  int32_t kind;
};
static_assert(sizeof(FItem) == 24, "FItem layout");

// A block of whole short rows, consecutive in the CSR: slot t holds element
// start + t of row[t], the at[t] & 255-th of its row's at[t] >> 8 elements.
struct Pack {
  int64_t start;
  int32_t n;      // elements (at most 16)
  int32_t pad;
  int32_t row[16];
  int32_t at[16];
};
static_assert(sizeof(Pack) == 144, "Pack layout");

// One step of the combine reduction: fold `count` consecutive maps starting
// at in_off (in order) into one; write it to out_off, or if out_off < 0
// apply it to the head vector `heavy` and write row `row` of A(m).
struct CItem {
  int64_t in_off;
  int64_t out_off;
  int32_t count;
  int32_t row;
  int32_t heavy;
  int32_t pad;
};
static_assert(sizeof(CItem) == 32, "CItem layout");

// A piece of a row for the core, loss and gradient passes.
struct Seg {
  int64_t start;
  int32_t len;
  int32_t row;
};
static_assert(sizeof(Seg) == 16, "Seg layout");

struct ModeHost {
  std::vector<int64_t> row_ptr;   // I+1
  std::vector<int32_t> idx;       // (N-1) * nnz
  std::vector<float> val;         // nnz
  std::vector<int64_t> perm;      // nnz: CSR position -> input position
  std::vector<FItem> compose;     // COMPOSE items, padded to multiples of 4
  std::vector<FItem> apply;       // HEAD items and longer LIGHT items, padded to a multiple of 4, then the others, padded
  std::vector<Pack> packs;        // the rows of at most kPackRow elements, which are also the last of `apply`
  std::vector<std::vector<CItem>> levels;
  std::vector<CItem> relax;       // FT_RELAXED: group items (chunk slots -> group record), then one merge item per
                                  // heavy row (its group records; out_off = elements after the head)
  std::vector<Seg> segs;
  std::vector<int64_t> seg_first; // I+1: first segment of a row (its ceil(L / seg_len) segments are consecutive)
  std::vector<int32_t> fid;       // nnz: fiber of the element at each CSR position
  std::vector<int32_t> fib_idx;   // (N-1) x fibers: fixed indices of each fiber (modes m+1, ..., m-1)
  // FT_RELAXED with rows longer than the head: idx, val and perm with those
  // rows dealt in stride order (the order of the factor passes); empty otherwise
  std::vector<int32_t> fidx;
  std::vector<float> fval;
  std::vector<int64_t> fperm;     // host only (ft_plan_host_csr)
};

struct ModeDev {
  int64_t* row_ptr = nullptr;
  int32_t* idx = nullptr;
  float* val = nullptr;
  int32_t* perm = nullptr;  // device permutation (int32: nnz < 2^31 required with FT_WITH_PERM)
  FItem* compose = nullptr;
  FItem* apply = nullptr;
  Pack* packs = nullptr;
  CItem* levels = nullptr;  // all levels back to back
  CItem* relax = nullptr;
  Seg* segs = nullptr;
  int64_t* seg_first = nullptr;
  int32_t* fid = nullptr;
  int32_t* fib_idx = nullptr;
  int32_t* fidx = nullptr;  // factor-order copies (FT_RELAXED), or null: the factor passes read idx, val
  float* fval = nullptr;
};

// Byte offsets of a mode's arrays in the caller's plan workspace (SIZE_MAX:
// the array is empty and its device pointer stays null).
struct ModeOff {
  size_t row_ptr, idx, val, perm, compose, apply, packs, levels, relax, segs, seg_first, fid, fib_idx, fidx, fval;
};

// Every array in a device workspace starts on this boundary.
constexpr size_t kAlign = 256;

// Sequential layout of arrays in one device buffer.
struct Layout {
  size_t bytes = 0;
  size_t add(size_t n) {
    if (n == 0) return SIZE_MAX;
    const size_t o = (bytes + kAlign - 1) / kAlign * kAlign;
    bytes = o + n;
    return o;
  }
};

// Scratch of one parameter set (ft_params.scratch): what the passes write
// between launches.  Byte offsets, sized for the largest mode of the plan.
struct ScratchOff {
  size_t maps = SIZE_MAX;       // float: chunk maps (J^2 + J each; FT_RELAXED: increments, then FP64 group records)
  size_t map_scale = SIZE_MAX;  // double: rho^length of each map
  size_t hvec = SIZE_MAX;       // float: head vectors of long rows (J each)
  size_t partials = SIZE_MAX;   // float: per-workgroup J x R partial sums
  size_t dpartials = SIZE_MAX;  // double: per-workgroup FP64 loss partials, then those of the sums of squares of A(n)
  size_t tseg = SIZE_MAX;       // float: per-segment sums of the gradient pass (R each)
  size_t gfib = SIZE_MAX;       // float: the shared g of each fiber (J each)
};

// Device pointers of a parameter set's scratch for one call.
struct Scratch {
  float* maps = nullptr;
  double* map_scale = nullptr;
  float* hvec = nullptr;
  float* partials = nullptr;
  double* dpartials = nullptr;
  float* tseg = nullptr;
  float* gfib = nullptr;
};

struct ModeMeta {
  int64_t I = 0;
  int64_t n_compose = 0;  // padded counts
  int64_t n_apply = 0;
  int64_t n_packs = 0;
  int64_t n_wave = 0;     // entries of the apply list before the rows that packs cover (a multiple of 4)
  int64_t row_elems = 0;  // elements of the entries between those of a workgroup each and n_wave
  int64_t n_team = 0;     // in-place items (heads, then longer rows) that a workgroup takes each
  int64_t n_heavy = 0;
  int64_t n_maps = 0;     // COMPOSE items (unpadded)
  std::vector<int64_t> level_off;  // offset of each level in the device array
  std::vector<int64_t> level_len;
  std::vector<int64_t> level_ncomp;  // folds of each level (0: the last level, whose items are final)
  int64_t n_fold_out = 0;          // map slots that the folds write, after those of the chunks
  int64_t n_segs = 0;
  int64_t n_long_segs = 0;  // segments taken by a wavefront each; the short rows' follow, by descending length
  int64_t n_relax_groups = 0;  // FT_RELAXED level-1 items
  int64_t n_relax = 0;         // FT_RELAXED level-2 items (heavy rows)
  int64_t n_fibers = 0;
  int64_t n_runs = 0;  // runs of equal column-0 index within rows
  int64_t head = 0;      // ft_desc.head or its default
  int64_t in_place = 0;  // elements of a long row updated in place before its chunks
  bool use_fiber = false;
  ft_mode_info info{};
};

}  // namespace ft

struct ft_prof_rec {
  int kid;
  hipEvent_t start, stop;
};

struct ft_plan {
  ft_desc desc{};
  int N = 0, J = 0, R = 0;
  int64_t nnz = 0;
  int chunk = 512, head = 1024, fanin = 16;  // head 0: chosen per mode (ModeMeta::head), at most head_cap
  int64_t head_cap = 0;
  int seg_len = 512;  // longest segment of the core, loss and gradient passes
  bool no_c_cache = false;  // FT_NO_C_CACHE
  bool relaxed = false;     // FT_RELAXED
  bool fused = true;        // exact factor passes launch in-place items and chunk maps together (not FT_SPLIT_FACTOR)
  bool run_reuse = false;   // segment passes reuse the column-0 C row along runs (FT_RUN_REUSE)
  int loss_mode = 0;        // the mode whose CSR the loss and forward passes walk
  std::vector<ft::ModeMeta> meta;
  std::vector<ft::ModeHost> host;
  std::vector<ft::ModeDev> dev;
  bool host_valid = false;
  bool uploaded = false;
  // device arrays of the plan: byte offsets in the caller's workspace (ft_plan_upload)
  std::vector<ft::ModeOff> off;
  size_t device_bytes = 0;
  // scratch every parameter set brings (ft_params.scratch)
  ft::ScratchOff soff;
  size_t scratch_bytes = 0;
  // kernel timing (ft_profile_enable); launches on a const plan append to it
  mutable bool prof_on = false;
  mutable std::vector<ft_prof_rec> prof;
};

namespace ft {
void set_error(const std::string& msg);
ft_status fail(ft_status s, const std::string& msg);

// kernel launchers (ft_refresh.hip, ft_factor.hip, ft_segment.hip); return hipSuccess or the launch error
constexpr int kPartials = 2048;  // max workgroups of the reduction kernels
constexpr int kSumsqBlocks = 256;  // max workgroups per matrix of the sums of squares
constexpr int kSegLen = 512;     // max elements per segment (ft_plan::seg_len)
constexpr int kShortSeg = 32;    // rows of at most this many elements may be listed as short
constexpr int kMinShort = 16384; // a mode with fewer of them lists none (one launch instead of two)
constexpr int kTeamRow = 1024;   // rows longer than this are updated by a workgroup, shorter ones by a wavefront
constexpr int kTeamHeads = 512;  // so many heads of kTeamRow elements are updated by a workgroup each, more by a wavefront
constexpr int kPackRow = 16;      // rows of at most this many elements share blocks of 16
// Items that go four to a wavefront (quad_items in ft_factor.hip), J <= 16.
//
// Chunks: from the number on at which the longer time of a chunk is hidden; a
// launch of few lasts as long as one chunk does (512 elements: 95 us against 45
// at J = 16).  us per iteration in the factor launches, one to a wavefront
// against four, at (chunks per mode): maps, J = 16, 264 and 303 (1900 to 3500),
// 444 and 446 (3000 to 6500), 661 and 600 (5500 to 9500), 100M elements 7700
// and 6960; maps, J = 8, 136 and 194 (700 to 1100), 270 and 219 (2100), 100M
// 7700 and 4490; order 8, where more rows are gathered per element, 796 and
// 1005 (2300), 1704 and 1765 (6500), 3240 and 3190 (14200).  Increments, J =
// 16, 143 and 163 (2400 to 4100), 221 and 204 (4300 to 7400), J = 8 121 and
// 136, 179 and 167 at the same, order 8 1206 and 1321 (6500), 3990 and 3799
// (24000).
inline bool quad_chunks(int N, int J, bool relaxed, int64_t n) {
  if (J > 16) return false;
  if (relaxed) return n >= (N > 4 ? 16384 : 4096);
  return n >= (N > 4 ? 8192 : J >= 16 ? 4096 : 2048);
}
// Rows (and heads) of 17 to kTeamRow elements: beside maps that go four to a
// wavefront too, unless they are so short that the start of an item counts
// (Netflix-shaped, us per iteration in the factor launches, maps four to a
// wavefront and rows one, or both: J = 16, 5M elements 457 and 441, 100M 7118 and
// 6769, J = 8, 8M 439 and 410); and on their own where there are many long ones
// (us per pass: 10,000 rows of 500 elements, J = 16 107 and 86, J = 8 87 and 74;
// 100,000 of 100, J = 16 266 and 282; relaxed, 5M, J = 16 212 and 278).
inline bool quad_rows(int N, int J, bool relaxed, int64_t n, int64_t elements, int64_t n_chunks) {
  if (J > 16 || N > 4) return false;
  if (!relaxed && quad_chunks(N, J, relaxed, n_chunks)) return n >= 2048 && elements >= 64 * n;
  return n >= 8192 && elements >= 256 * n;
}
constexpr int kRelaxGroup = 256; // chunks per level-1 group of the relaxed merge

// FT_RELAXED scratch in the map region: J + 1 floats per chunk slot, then
// (8-byte aligned) J + 1 doubles per level-1 group
inline int64_t relax_incr_floats(int64_t n_maps, int J) { return (n_maps * (J + 1) + 1) / 2 * 2; }

// Launches on this thread inside an UntimedScope create no timing events
// (the entry point that must not allocate).
inline bool& untimed_flag() {
  static thread_local bool f = false;
  return f;
}
struct UntimedScope {
  bool prev;
  UntimedScope() : prev(untimed_flag()) { untimed_flag() = true; }
  ~UntimedScope() { untimed_flag() = prev; }
};

// Brackets one kernel launch with events when timing is enabled on the plan.
struct KTimer {
  const ft_plan* P;
  int kid;
  hipStream_t s;
  hipEvent_t a = nullptr;
  KTimer(const ft_plan* P_, int kid_, hipStream_t s_) : P(P_), kid(kid_), s(s_) {
    if (P && P->prof_on && !untimed_flag() && hipEventCreate(&a) == hipSuccess) (void)hipEventRecord(a, s);
  }
  ~KTimer() {
    if (!a) return;
    hipEvent_t b = nullptr;
    if (hipEventCreate(&b) == hipSuccess && hipEventRecord(b, s) == hipSuccess)
      P->prof.push_back(ft_prof_rec{kid, a, b});
    else
      (void)hipEventDestroy(a);
  }
};

inline double* relax_partials(const ft_plan* P, const Scratch& S, int m) {
  return reinterpret_cast<double*>(S.maps + relax_incr_floats(P->meta[m].n_maps, P->J));
}

// Scratch pointers of a parameter set (its buffer checked by the caller).
Scratch scratch_of(const ft_plan* P, const ft_params* p);

hipError_t launch_refresh(const ft_plan* P, int n0, int n1, const ft_params* p, hipStream_t s);  // modes n0..n1-1
hipError_t launch_factor(const ft_plan* P, int m, const ft_params* p, const Scratch& S, double lr, double lam,
                         hipStream_t s);
hipError_t launch_core_grad(const ft_plan* P, int m, const ft_params* p, const Scratch& S, float* G_out,
                            hipStream_t s);
hipError_t launch_core_update(const ft_plan* P, int m, const ft_params* p, const Scratch& S, double lr, double lam,
                              hipStream_t s);
hipError_t launch_loss(const ft_plan* P, const ft_params* p, const Scratch& S, double lam_a, double lam_b,
                       double* out4, hipStream_t s);
// bad: null, or int32[N] that receives 1 for every mode with an index out of range
hipError_t launch_predict(const ft_plan* P, const ft_params* p, const int32_t* coords, int64_t q, float* out,
                          int32_t* bad, hipStream_t s);
// ft_loss_noalloc: the loss with its partials in the library's static device
// array (capacity and the bytes a plan needs, in bytes)
size_t noalloc_loss_capacity();
size_t noalloc_loss_need(const ft_plan* P);
hipError_t launch_loss_noalloc(const ft_plan* P, const ft_params* p, double lam_a, double lam_b, double* out4,
                               hipStream_t s);
hipError_t launch_forward(const ft_plan* P, const ft_params* p, const Scratch& S, float* out, hipStream_t s);
hipError_t launch_grad(const ft_plan* P, const ft_params* p, const Scratch& S, const float* upstream,
                       float* const* gA, float* const* gB, hipStream_t s);
bool supported(int N, int J, int R);
int max_fanin();  // default and largest number of maps per fold
}  // namespace ft
