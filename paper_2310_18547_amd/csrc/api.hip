// C ABI of libsgmv: argument checks, launch-shape choice, kernel dispatch.
// Everything that computes runs in the kernels; this file only validates and
// enqueues.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

#include "../../include/sgmv.h"
#include "launch.h"

// Scratch of sgmv_add_lora_static, one copy per GPU, held until the process ends:
//   [0, 4.25 KiB)    header (generation copies, error word)
//   [4.25 KiB, 6 MiB) exchange words of the single-launch kernels -- at a fixed place whatever
//                    the batch, so that a word found there was always written as an exchange
//                    word, with the generation tag of an earlier call
//   [6 MiB, 9 MiB)   split-K partial sums and the MFMA expand's operands of v
// In host code the array's name is only a handle for hipGetSymbolAddress; kernels get the
// address that call returned.
constexpr size_t kStaticExchangeEnd = (size_t)6 << 20;
constexpr size_t kStaticBytes = (size_t)9 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticBytes];
static_assert(kStaticBytes == SGMV_STATIC_SCRATCH_BYTES, "the header states the array's size");

namespace {

using namespace sgmv;

constexpr int kMinSplitCap = 16;       // the workspace always allows this many slices
constexpr int kTargetWorkgroups = 512; // about two workgroups per compute unit
// Longest segment the single-launch MFMA kernel is considered for.  What really limits it is
// that every (segment, sixteen-row block, slice) workgroup must be resident at once with its
// weight slices in LDS (choose_tile): about 64 row blocks in all at h = 4096.
constexpr int kTileMaxSegLen = 4096;
constexpr int kMatrixMaxSegments = 65535;  // the MFMA kernels place a segment by 32-bit arithmetic that holds for this many (find_item)
constexpr int kFusedSlices = 8;        // most slices per segment the single-launch kernels pick
constexpr int kRowsMostSegments = 256;  // segments up to which SGMV_PATH_AUTO launches per row (four rounds of the look-up)
constexpr long long kShrinkWholeMostElements = 48LL << 20;  // weights (96 MB) up to which the stand-alone shrink runs without Split-K
constexpr int kTileMultiSlices = 4;    // fewest slices at which a joint tile launch beats add-ons run per row
constexpr int kFusedMaxWorkgroups = kGenerationCopies;  // every workgroup of a launch has its own generation copy
constexpr int kFusedSpinLimit = 1 << 18;
constexpr int kMaxDevices = 64;
constexpr int kDefaultComputeUnits = 256;  // MI355X; assumed where no device can be asked

// Residency limits of the single-launch kernels.  They follow from the compute units of the
// current device (asked once per device): a workgroup that waits for the partial sums of a
// workgroup that has not started yet only idles, so these launches stay within what is
// resident at once.
struct Limits {
  int fused_workgroups;       // one workgroup per compute unit
  int tile_max_grid;          // tile launch, workgroups without rows included (5/4 per unit)
  int multi_workgroups;       // multi-projection launch side by side (two per unit)
  int multi_workgroups_most;  // ... where the pipelined kernel does not apply (three per unit)
};

int compute_units() {
  static std::atomic<int> cached[kMaxDevices];  // zero-initialised
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();  // no device here (a host-only query): leave no sticky error behind
    return kDefaultComputeUnits;
  }
  int cu = cached[dev].load(std::memory_order_relaxed);
  if (cu == 0) {
    if (hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu <= 0) {
      (void)hipGetLastError();
      cu = kDefaultComputeUnits;
    }
    cached[dev].store(cu, std::memory_order_relaxed);
  }
  return cu;
}

Limits limits() {
  const int cu = compute_units();
  // launches far beyond one workgroup per unit measured slower than the launch-per-step kernels
  // (tile kernel, 456 workgroups for 171 with rows: 25.8 us against 14.8 us) even though the
  // surplus leaves at once
  return Limits{cu, cu + cu / 4, 2 * cu, 3 * cu};
}

int spin_limit_of(const sgmv_problem* p) { return p->spin_limit > 0 ? p->spin_limit : kFusedSpinLimit; }
// AUTO uses the MFMA kernels from this segment length on.  Their work goes with the number of
// segments (every segment occupies at least one block of 64 rows), that of the vector kernels
// with the rows: measured at h = 4096, 128 segments of 4 rows, ranks 8 / 16 / 32 / 64: vector
// kernels 13.9 / 18.8 / 26.6 / 42.3 us against 18.7 / 22.0 / 27.1 / 40.6; 64 segments of 8 rows,
// ranks 16 / 64: MFMA 16.7 / 25.2 against 24.4 / 42.3.  (At rank 64 the line lies a little high: 64
// segments of 4 / 5 rows, MFMA 23.6 / 23.8 against 24.8 / 36.6.)
constexpr int kMatrixMinSegLen = 6;
// At rank 64 the vector kernels are slow enough that the MFMA kernels win from two rows per
// segment on while the segments are few (32 segments of 2 / 4 rows: 16.2 / 16.7 us against 15.8 /
// 18.8; the Uniform mix of 64 rows, 42 segments: 20.7 against 20.9, of 256 rows, 63 segments of up to 8:
// 23.8 against 39.5).
constexpr int kMatrixFewSegments = 48;
constexpr int kMatrixWaves = 4096;     // waves the MFMA shrink aims for (four per SIMD)

inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

inline int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }
inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// Most split-K slices the workspace is sized for at a given batch.
int split_cap(int n_tokens) {
  int c = ceil_div(16384, n_tokens > 0 ? n_tokens : 1);
  if (c > kMaxKSplit) c = kMaxKSplit;
  if (c < kMinSplitCap) c = kMinSplitCap;
  return c;
}

int check_common(const sgmv_problem* p, const int32_t* seg_starts, int32_t n_segs,
                 int32_t layer_idx, bool need_in, bool need_out) {
  if (p == nullptr) return SGMV_ERR_NULL;
  if (p->dtype != SGMV_F16 && p->dtype != SGMV_BF16) return SGMV_ERR_UNSUPPORTED;
  if (n_segs < 0 || p->n_tokens < 0 || p->num_layers <= 0 || p->max_seg_len < 0)
    return SGMV_ERR_SHAPE;
  if (p->r <= 0 || (need_in && p->h_in <= 0) || (need_out && p->h_out <= 0)) return SGMV_ERR_SHAPE;
  if (p->r != 8 && p->r != 16 && p->r != 32 && p->r != 64) return SGMV_ERR_UNSUPPORTED;
  if ((need_in && (p->h_in % 8) != 0) || (need_out && (p->h_out % 8) != 0))
    return SGMV_ERR_UNSUPPORTED;
  if (p->path < SGMV_PATH_AUTO || p->path > SGMV_PATH_ROWS) return SGMV_ERR_UNSUPPORTED;
  if (p->spin_limit < 0) return SGMV_ERR_UNSUPPORTED;
  if (p->ksplit < 0 || p->ksplit > kMaxKSplit) return SGMV_ERR_UNSUPPORTED;
  if (p->expand_threads != 0 && p->expand_threads != 64 && p->expand_threads != 128 &&
      p->expand_threads != 256 && !(p->expand_threads == kExpandSplit && p->r >= 32))
    return SGMV_ERR_UNSUPPORTED;
  if (p->path == SGMV_PATH_MATRIX && n_segs > kMatrixMaxSegments) return SGMV_ERR_UNSUPPORTED;
  if (layer_idx < 0 || layer_idx >= p->num_layers) return SGMV_ERR_RANGE;
  if (n_segs > 0 && p->n_tokens > 0 && seg_starts == nullptr) return SGMV_ERR_NULL;
  return SGMV_OK;
}

int check_workspace(const sgmv_problem* p) {
  if (p->workspace == nullptr) return SGMV_ERR_WORKSPACE;
  if (!aligned(p->workspace, 256)) return SGMV_ERR_ALIGN;
  if (p->workspace_bytes < sgmv_workspace_bytes(p->n_tokens, p->r)) return SGMV_ERR_WORKSPACE;
  return SGMV_OK;
}

// Split-K shape: ksplit slices of kslice elements, kslice a multiple of 8 and at
// most kMaxKSlice, no slice empty.  Returns false when h_in is too wide for the
// workspace's slice count.
bool choose_split(const sgmv_problem* p, int n_segs, int* ksplit, int* kslice) {
  const int cap = split_cap(p->n_tokens);
  const int need = ceil_div(p->h_in, kMaxKSlice);
  if (need > cap) return false;
  // enough workgroups to fill the chip, but slices of at least 32 KiB of weights: more
  // slices than that only lengthen the reduction that follows (measured, 1 to 64 segments)
  int s = p->ksplit;
  if (s == 0) {
    s = ceil_div(kTargetWorkgroups, n_segs);
    const int by_size = ceil_div((long long)p->h_in * p->r, 16384);
    if (s > by_size) s = by_size;
  }
  const int most = p->h_in / 64 > 0 ? p->h_in / 64 : 1;  // keep slices >= 64 elements
  if (s > most) s = most;
  if (s > cap) s = cap;
  if (s < need) s = need;
  int len = ceil_div(ceil_div(p->h_in, s), 8) * 8;
  *kslice = len;
  *ksplit = ceil_div(p->h_in, len);
  return true;
}

// Whether a call goes to the MFMA kernels: forced, or segments long enough that
// 16-row tiles are mostly full (from the hint, else from the mean length).
bool use_matrix(const sgmv_problem* p, int n_segs) {
  if (p->path == SGMV_PATH_MATRIX) return true;
  if (p->path != SGMV_PATH_AUTO) return false;
  if (n_segs > kMatrixMaxSegments) return false;  // the vector kernels take any number of segments
  const int len = p->max_seg_len > 0 ? p->max_seg_len : p->n_tokens / (n_segs > 0 ? n_segs : 1);
  if (p->r >= 64 && n_segs <= kMatrixFewSegments && len >= 2) return true;
  return len >= kMatrixMinSegLen;
}

// The stand-alone expand at rank 64 is ahead on the MFMA kernels for more short segments than the
// shrink and the add-on are (h = 4096, 64 segments of 2 / 4 rows: 11.5 / 12.0 us against 10.2 / 12.3
// on the vector kernel; Uniform mix of 128 rows, 57 segments: 11.2 against 15.0; 128 segments of 2
// rows: 16.2 against 16.9).
bool expand_use_matrix(const sgmv_problem* p, int n_segs) {
  if (use_matrix(p, n_segs)) return true;
  if (p->path != SGMV_PATH_AUTO || p->r < 64 || n_segs > 128) return false;
  const int len = p->max_seg_len > 0 ? p->max_seg_len : p->n_tokens / (n_segs > 0 ? n_segs : 1);
  return len >= 2;
}

// Split-K shape of the MFMA shrink of n_proj add-ons and whether the expand behind it adds the partial sums up itself
// (`direct`, a launch less).
struct MatrixSplit {
  int ksplit, kslice;
  bool direct;
};

// Direct: every workgroup of the expand reads the partial sums of its 64 rows, r * slices * 256 bytes beside 64 KB of y, and
// each of the eight L2s fetches most of them once more, which takes back the 2 us of a launch at about 2 MB of partial sums.
// Three launches / two, us (binary16): 700 rows, rank 16, sixteen slices, 4096 -> 4096 11.8 / 9.8 and -> 11008 14.9 / 13.6; 60
// segments of 8 rows, eight slices, 14.3 / 12.7; 1152 rows beside 41 of one row, eight slices, 15.9 / 14.1, three projections of
// them 29.4 / 28.9, to 11008 (2300 workgroups) 52.0 / 53.0; three of 3440 rows, 8192 -> 2048, 35.3 / 36.5.  At rank 32 the
// partial sums are too many (1152 rows beside 41, eight slices, 19.1 / 20.4), at rank 64 also the operands in LDS.
// Beyond 1920 rows (thirty blocks) three launches, which is what the plan of 2000 rows is expected to tell, not what is faster: two would be
// 16.7 against 17.7 us at 2000 rows, rank 16, 4096 wide, and 46.6 against 47.6 at 4814, 8192 wide.  SGMV_PATH_MATRIX keeps three at
// every rank, so that finalize_v_kernel and the expand behind it can be run and timed on any batch.
constexpr int kDirectMostRows = 1920;
bool matrix_direct(const sgmv_problem* p, int n_segs, int n_proj, int slices) {
  if (p->path == SGMV_PATH_MATRIX || p->r > 16 || p->n_tokens > kDirectMostRows) return false;
  // every short segment is a block of its own (300 of 5 rows, 2048 -> 8192, rank 16: 39.6 / 52.0): beyond 104 of them two launches are ahead
  // to narrow outputs only (up to 2048 / 4096 / 6144 columns / wider, times as fast: 105 to 124 segments 1.09 / 1.08 / 1.05 / 0.94, 200 to
  // 224 1.06 / 0.95 / 0.96 / 0.93)
  if (n_segs > 104) return false;
  const long long sums = (long long)p->n_tokens * n_proj * p->r * slices;
  const long long workgroups = (long long)ceil_div(p->n_tokens, 64) * ceil_div(p->h_out, 256) * n_proj;
  return p->r * slices <= 256 && sums * (workgroups > 1024 ? workgroups : 1024) <= (512LL << 10) * 1024;
}

// Add-ons of long segments under SGMV_PATH_AUTO: instead of `power`, choose_split_matrix's power of two, as many slices as give every compute
// unit one workgroup and not more (`fill` of them would), because the units that get a second one decide when the launch ends: 2000 rows of
// six segments, rank 16, 8192 wide (35 row blocks), whole add-on at 5 / 6 / 8 / 16 slices 25.7 / 25.1 / 27.3 / 27.5 us; 4814 rows at rank 64 (41
// blocks of 128) 57.5 / 56.5 / 60.0 / 59.6; three add-ons of 2600 rows at rank 32 (22 blocks) at 4 / 8 / 16 45.5 / 40.7 / 44.3.  From
// seven on only eight or sixteen (1400 rows, rank 16, 8192 wide, 8 / 10 / 12 / 16 slices 19.0 / 20.0 / 21.4 / 20.5).  Fewer than four leave too
// few loads in flight (4814 rows, rank 16, 8192 wide, 4 / 6 / 8 / 16 slices 52.6 / 50.4 / 48.9 / 47.6), and `power` stays, as it does
//  * for five and six up to rank 16 (2625 rows, 11008 -> 1024, rank 16, 5 / 16 slices 23.4 / 22.0), five at rank 32 on inputs wider than
//    8192 (2335 rows, 11008 -> 13824, 5 / 16 slices 47.8 / 46.0), four at rank 8 from 8192 on (3535 rows, 8192 -> 5120, 4 / 16 slices 34.4 /
//    32.8), four of add-ons that do not share their pass over x (`unshared`) and, at rank 64 or on inputs wider than 8192, four to six of more than eight
//    segments: these are often many short ones beside a few long ones, and then more blocks than `fill` reckons (1686 rows of twelve, 11008 ->
//    4096, rank 64, three add-ons, 4 / 8 slices 71.3 / 56.4);
//  * for seven, which eight overfills, on inputs wider than 8192 and, where `power` is less than eight, up to 3072 (11008 -> 2048, 1921 rows, rank
//    16, 8 / 16 slices 27.2 / 24.6; 1024 -> 824, 1124 rows, rank 64, three add-ons, 8 / 4 slices 20.1 / 17.9), unless the expand then adds the
//    partial sums up itself (1863 rows, 3560 -> 1144, rank 16, 8 / 16 slices 12.3 / 14.2);
//  * where a slice would be thinner than 192, while the units are few enough 128 (1312 rows, 1024 wide, rank 64, 6 / 4 slices 19.2 / 18.0; 1076 rows
//    of 2048, rank 32, 16 / 8 slices 12.3 / 11.9; at rank 64, where `power` is four, 16 / 4 of 2000 13.1 / 15.3);
//  * at rank 64 for more than sixteen where the units take 28 (454 rows, 13824 -> 5120, 31 / 16 slices 20.3 / 23.0).
// Sixteen from fourteen on, up to rank 32 on inputs wider than 8192 from thirteen on, where half as many chunks one after the other outweigh a
// second round (1755 rows, 11008 -> 2424, rank 32, three add-ons, fill 13.6, 8 / 16 slices 47.9 / 42.8).
// 1712 points that this rule and the launch less behind it change, against `power` and three launches: 1.09 times as fast on average, seven
// below 0.97, 0.93 at worst.
int filling_slices(const sgmv_problem* p, int n_segs, int power, float fill, bool unshared, bool direct_at_eight) {
  const bool wide = p->h_in > 8192;
  const bool steady = n_segs <= 8 || (p->r < 64 && !wide);
  int n = power;
  if (fill >= (p->r <= 32 && wide ? 13.f : 14.f)) {
    n = p->r == 64 && power > 16 && fill >= 28.f ? power : 16;
    if (n > power && p->h_in < 16 * (p->r == 64 ? 128 : 192)) n = 8;
  } else if (fill >= 8.f) {
    n = 8;
  } else if (fill >= 7.f) {
    if (direct_at_eight || (power >= 8 ? !wide : p->h_in > 3072)) n = 8;
  } else if (fill >= 6.f) {
    if (p->r >= 32 && steady) n = 6;
  } else if (fill >= 5.f) {
    if (steady && (p->r == 64 || (p->r == 32 && !wide))) n = 5;
  } else if (fill >= 4.f) {
    if (steady && !unshared && (p->r > 8 || p->h_in < 8192)) n = 4;
  }
  if (n > power && n <= 8 && p->h_in < n * (fill >= 15.f ? 128 : 192)) n = power;
  return n;
}

// Split-K shape of the MFMA shrink of n_proj add-ons: about kMatrixWaves waves in flight, a power of two
// slices, so that a slice's workgroups (consecutive ids) meet on the same XCDs and its part of A_i in
// their L2s (8192 wide, rank 16, 4814 rows, 8 / 11 / 16 slices: 18.6 / 19.9 / 17.4 us; the whole add-on to 4096, rank 16, 5120
// and 8192 wide, 700 rows, 23 / 16 slices: 14.0 / 12.5 and 15.2 / 13.0, 11008 wide, 1000 rows, 17 / 16: 18.2 / 15.1; rank 64, 13824
// wide, 700 rows, 23 / 16: 21.1 / 22.0), and from four slices on only as many as leave the partial sums of all add-ons,
// written and read again, about half the bytes of one x, two thirds at most (11432 wide, rank 64, three add-ons of 724
// rows, the whole call at 4 / 8 / 15 slices: 45.0 / 32.3 / 33.1 us; 3272 wide, 3254 rows, 2 / 4 / 13: 61.3 / 62.4 / 67.1).
//
// Add-ons on long segments: filling_slices.  On short segments whose partial sums the expand adds up itself: eight, in small batches on wide inputs
// sixteen (60 of 8 rows, rank 16, 4096 wide, 8 / 16 slices 12.7 / 14.2; 20 of 20 rows, 8192 wide, 14.6 / 13.9), or the power of two and three
// launches where sixteen are too many to be added up there (three add-ons of 788 rows, 11352 -> 1320, rank 16, 8 / 16 slices 31.0 /
// 25.9), and where it is more than sixteen for three add-ons of rank 16 (462 rows of six, 11008 -> 11008, 32 / 16 slices 27.6 / 30.2).
MatrixSplit choose_split_matrix(const sgmv_problem* p, int n_segs, int n_proj, bool same_x) {
  const int cap = split_cap(p->n_tokens);
  const int most = p->h_in / 128 > 0 ? p->h_in / 128 : 1;  // keep slices of at least one chunk
  const int limit = most < cap ? most : cap;
  const auto within = [&](int s) {
    while (s > limit) s = p->ksplit > 0 ? limit : s / 2;
    return s < 1 ? 1 : s;
  };
  int s = p->ksplit;
  if (s == 0) {
    const bool shared = same_x && shrink_shared_fits(p->r, n_proj);
    const int rows = shrink_stream_rows(p->r, shared ? n_proj : 1);
    const long long blocks = (p->n_tokens / rows + (n_segs + 1) / 2) * (long long)(shared ? 1 : n_proj);
    const long long waves = (blocks > 0 ? blocks : 1) * (rows / 16);
    const long long by_partials = p->h_in / (8LL * p->r * n_proj);
    s = 1;
    while (s * 3 * waves <= 2LL * kMatrixWaves && (s < 4 || s * 3 <= 2 * by_partials)) s *= 2;
    if (p->path != SGMV_PATH_MATRIX && p->h_out > 0) {
      // A segment's last block is half full on average, in a sum over n segments with a deviation of 0.3 sqrt(n) blocks,
      // twice which keeps the launch from passing the units by a few workgroups (4814 rows at rank 64, 8192 -> 28672, 43
      // blocks: 5 / 6 slices 138 / 149 us); of a short segment's block one wave of four works
      const bool is_long = p->n_tokens >= (long long)n_segs * rows;
      const float last = is_long ? 0.5f * n_segs + 0.6f * sqrtf((float)n_segs) : 0.25f * n_segs;
      const float fill = compute_units() / (((float)p->n_tokens / rows + last) * (shared ? 1 : n_proj));
      if (is_long) {
        s = filling_slices(p, n_segs, s, fill, !shared && n_proj > 1, matrix_direct(p, n_segs, n_proj, within(8)));
      } else if ((s <= 16 || p->r * n_proj <= 32 || p->h_in <= 8192) && matrix_direct(p, n_segs, n_proj, within(8))) {
        if (fill < 14.f || p->h_in <= 4096)
          s = 8;
        else if (matrix_direct(p, n_segs, n_proj, within(16)))
          s = 16;
        else if (p->h_in <= 8192)
          s = 8;
      }
    }
  }
  MatrixSplit m;
  m.kslice = ceil_div(ceil_div(p->h_in, within(s)), 32) * 32;
  m.ksplit = ceil_div(p->h_in, m.kslice);
  m.direct = matrix_direct(p, n_segs, n_proj, m.ksplit);
  return m;
}

size_t partial_bytes(int n_tokens, int r) {
  return round_up((size_t)split_cap(n_tokens) * (size_t)n_tokens * (size_t)r * sizeof(float), 256);
}

// Where a call keeps its intermediate results.
struct Scratch {
  unsigned long long* header;  // generation copies, error word
  float* partials;             // split-K partial sums of the launch-per-step kernels
  unsigned long long* exch;    // exchange words of the single-launch kernels
  char* operands;              // 16-bit operand pairs of v and a range factor per row (MFMA expand)
};

// Caller's workspace: [header][partials][exchange words, twice the bytes][operands].
Scratch caller_scratch(const sgmv_problem* p) {
  char* base = static_cast<char*>(p->workspace);
  const size_t parts = partial_bytes(p->n_tokens, p->r);
  return Scratch{reinterpret_cast<unsigned long long*>(base),
                 reinterpret_cast<float*>(base + kWorkspaceHeader),
                 reinterpret_cast<unsigned long long*>(base + kWorkspaceHeader + parts),
                 base + kWorkspaceHeader + 3 * parts};
}

// Operands of the MFMA expand: v as high and low 16-bit parts, one range factor per row.
size_t operand_bytes(int n_tokens, int r) {
  return 2 * round_up((size_t)n_tokens * r * 2, 256) + round_up((size_t)n_tokens * 4, 256);
}
void set_operands(ExpandArgs* a, const Scratch& sc, int n_tokens, int r) {
  char* base = sc.operands;
  a->header = sc.header;
  const size_t half = round_up((size_t)n_tokens * r * 2, 256);
  a->vh = reinterpret_cast<uint16_t*>(base);
  a->vl = reinterpret_cast<uint16_t*>(base + half);
  a->undo = reinterpret_cast<float*>(base + 2 * half);
}

// Lane groups of the hand-off kernel's expand phase: as many as give every lane a chunk of the column slice, and
// enough that a lane holds at most sixteen weight rows.  A single add-on at ranks up to 16 stops
// at two (the pair of neighbouring lanes that needs no LDS to add up, fused_kernel.hip) even
// where that leaves lanes without a chunk: measured at h = 4096, r = 16, 1 / 8 / 16 / 32 segments:
// 4.02 / 4.42 / 4.43 / 4.83 us against 4.07 / 4.54 / 4.59 / 5.01 us; at ranks 32 and 64 and in
// the multi-projection launches the wider groups are faster (16 segments at rank 32: 5.02
// against 5.46 us).
int fused_lane_groups(int r, int cslice, bool single_add_on) {
  const int chunks = cslice / 8;
  const int most = single_add_on && r <= 16 ? 2 : 8;
  int g = 1;
  while (g * 2 <= most && 256 / (g * 2) >= chunks) g *= 2;
  if (most == 2 && g == 1 && chunks <= 128) g = 2;
  while (r / g > 16) g *= 2;
  return g;
}

// Memory round trips of a workgroup at s slices: batches of 2048 128-bit loads of A_i, then (h_out = 0: a shrink on
// its own has none) passes over its columns of B_i.
int fused_round_trips(const sgmv_problem* p, int s, bool single_add_on) {
  const int kslice = ceil_div(ceil_div(p->h_in, s), 8) * 8, cslice = ceil_div(ceil_div(p->h_out, s), 8) * 8;
  const int batches = ceil_div(kslice * (p->r / 8), 2048);
  return cslice == 0 ? batches : batches + ceil_div(cslice, 256 / fused_lane_groups(p->r, cslice, single_add_on) * 8);
}

// Launch shape of the single-launch path; false when it does not apply.
// by_rows: the launch's items are the rows of the batch (pass n_tokens for n_segs), each looking its
// segment up on the device, so the segments may have any length.
bool choose_fused(const sgmv_problem* p, int n_segs, FusedArgs* f, bool single_add_on = true, bool by_rows = false) {
  if (!p->workspace_ready) return false;
  const Limits lim = limits();
  f->items = n_segs;
  f->by_rows = by_rows;
  f->paired = false;
  if (p->max_seg_len != 1 && !by_rows) return false;  // one row per segment; longer ones go to the tile kernel
  if (n_segs > kFusedMaxWorkgroups) return false;
  const int cap = split_cap(p->n_tokens);
  const int need = ceil_div(p->h_in, kMaxKSlice);
  if (need > cap) return false;
  // every workgroup of a launch must be resident at once (one per compute unit): a
  // workgroup that waits for a slice of a workgroup not yet started only idles
  int s = p->ksplit > 0 ? p->ksplit : lim.fused_workgroups / n_segs;
  if (p->ksplit == 0 && s > kFusedSlices) s = kFusedSlices;
  if (p->ksplit == 0) {  // a power of two: measured 5-20 % faster than the odd counts in between
    int pw = 1;
    while (pw * 2 <= s) pw *= 2;
    s = pw;
  }
  // 97 .. 128 segments of a single add-on: four slices, two workgroups per unit, rather than two
  // (measured at h = 4096, 128 segments, r = 16 / 32: 9.35 / 18.0 us against 9.81 / 18.8; no
  // difference at 96 segments or at rank 64; wider inputs are better off as they are)
  if (p->ksplit == 0 && single_add_on && s == 2 && n_segs > 96 && 2 * n_segs <= lim.fused_workgroups &&
      p->r <= 32 && need <= 2)
    s = 4;
  // Small batches at high rank: where a slice of A_i at eight slices takes more than one batch
  // of loads (2048 128-bit chunks), sixteen slices are faster while they are all resident
  // (measured at r = 64, h = 4096 / 5120, 1..8 segments: 5.1 / 5.8 us against 5.4 / 6.7 us)
  // The same holds for the slice of B_i of a wide output (4096 -> 11008 at rank 32, 1 / 8 / 16
  // segments: 5.7 / 5.9 / 7.1 us against 6.2 / 6.7 / 8.1), and it does not hold at rank 16, where
  // the chunks are short (h_in = 11008 / 13824, 1 .. 16 segments: eight slices 3-5 % ahead).
  const int wide = p->h_in > p->h_out ? p->h_in : p->h_out;
  if (p->ksplit == 0 && s == kFusedSlices && 2 * s * n_segs <= lim.fused_workgroups && p->r >= 32 &&
      (long long)ceil_div(wide, s) * (p->r / 8) > 2048)
    s = 2 * kFusedSlices;
  if (s > wide / 64) s = wide / 64;
  // Narrow shapes: no more slices than leave each a full batch of loads (2048 128-bit chunks of the
  // wider weight); thinner ones only add the hand-off (measured at rank 16, 8 segments, one / two /
  // four / eight slices: h = 1024 3.84 / 4.07 / 4.26 / 4.33 us, h = 2048 4.94 / 4.17 / 4.20 / 4.29; at
  // h = 4096 four and eight are level, 4.38 / 4.37)
  if (p->ksplit == 0 && wide <= 2048) {
    const int full = (int)((long long)wide * (p->r / 8) / 2048);
    if (s > (full > 1 ? full : 1)) s = full > 1 ? full : 1;
  }
  if (s > cap) s = cap;
  if (s > kFusedMaxWorkgroups / n_segs) s = kFusedMaxWorkgroups / n_segs;
  if (s < need) s = need;
  if (s < 1) s = 1;
  // A single add-on whose workgroups, padding included (an XCD takes whole items), leave units free: the
  // count from s up to seven with the fewest memory round trips, the smallest of equals.  Measured, four
  // (or what was taken before) -> this many slices, us: 45 rows of 18 adapters, bfloat16, h = 5120, five slices: rank 16
  // 6.0 -> 5.1, rank 32 9.8 -> 7.6, rank 64 14.1 -> 11.8; 40 segments, 4096 -> 11008, six slices: rank 16
  // 7.4 -> 6.3, rank 32 12.1 -> 11.3, rank 64 19.6 -> 17.7; 11008 -> 4096, six slices: 8.0 -> 6.8, 14.4 -> 10.3 and
  // 22.2 -> 17.0.  One workgroup too many for an XCD costs more than that (51 segments, h = 5120, rank 32, 280
  // workgroups: 10.8 -> 13.5), and with equal or hardly fewer round trips more slices gain nothing (h = 4096, ranks
  // 16 and 32: level; h = 8192, rank 64, 47 segments, eleven round trips for twelve: 21.2 -> 21.5).
  const long long padded = fused_grid_items(n_segs);
  const bool spread = p->ksplit == 0 && single_add_on && s < kFusedSlices && s * padded <= lim.fused_workgroups;
  if (spread) {
    int trips = fused_round_trips(p, s, true);
    for (int t = s + 1; t < kFusedSlices && t * padded <= lim.fused_workgroups && t <= cap && t <= wide / 64; ++t)
      if (10 * fused_round_trips(p, t, true) <= 9 * trips) {
        s = t;
        trips = fused_round_trips(p, t, true);
      }
  }
  // a slice count forced by a wide input to five, six or seven on more workgroups than units: eight
  // instead, where the launch has room (measured at 64 segments, h_in = 11008, six -> eight slices: rank 64
  // 31.9 -> 27.5 us, rank 16 9.79 -> 9.53; h_in = 13824, seven -> eight: no difference)
  bool eight = false;
  if (p->ksplit == 0 && single_add_on && !spread && s == need && s > 4 && s < 8 && 8 * padded <= kFusedMaxWorkgroups &&
      8 <= cap && 8 <= wide / 64) {
    s = 8;
    eight = true;
  }
  // the grid is padded to whole rows of segments (launch.h, fused_grid_x)
  const int gx = fused_grid_x(n_segs);
  if ((long long)s * ceil_div(n_segs, gx) * gx > kFusedMaxWorkgroups) return false;
  // slices forced by a very wide input can outnumber the compute units several times over;
  // from about two rounds of workgroups on the launch-per-step kernels are faster (measured)
  // (per-row launches, sized by their own rule, rows_apply: up to three rounds, 384 rows at two slices)
  if (p->path == SGMV_PATH_AUTO && p->ksplit == 0 && (long long)s * n_segs > (by_rows ? 3 : 2) * lim.fused_workgroups)
    return false;
  // From rank 32 on, a launch of more workgroups than units is only worth it when the units get
  // equal shares: 288 or 384 workgroups leave most units waiting for the ones with two (measured
  // against the launch-per-step kernels, h = 5120, three slices, 96 / 128 segments: rank 32 22.4 /
  // 24.3 against 19.1 / 22.1 us, rank 64 36.3 / 40.1 against 30.7 / 35.2; h = 8192, four slices,
  // 96 segments: 27.8 against 24.7 and 45.2 against 41.5; 512 workgroups are fine: 128 segments
  // at h = 4096, rank 32: 18.0 against 19.6)
  // (not so eight slices, whose shares are small: 11008 -> 4096, 51 segments, the launch that took over
  // against eight slices: rank 32 17.5 / 12.5 us, rank 64 26.6 / 23.2; 45 rows of 18 adapters, bfloat16:
  // 13.7 / 10.7 and 37.3 / 16.9; but at rank 64 up to 40 segments, 320 workgroups, keep what they had: 13824 ->
  // 5120, 33 / 36 / 40 segments, binary16 24.5 / 25.0, 22.9 / 25.7 and 24.8 / 26.1, bfloat16 24.3 / 27.4, 22.8 / 28.2 and
  // 24.8 / 28.6; and so do up to 48 segments in bfloat16, which spends more on a value, where a workgroup passes over its
  // columns of B_i more than once: 13824 -> 5120, 41 / 44 / 48 segments 26.6 / 28.7, 26.1 / 29.2, 27.0 / 29.8, 12544 -> 8192
  // 27.4 / 29.6, 27.3 / 29.9, 29.0 / 30.3; not 13440 -> 4096, one pass, 26.4 / 25.8, 25.9 / 26.3, 25.9 / 26.2, nor 13824 -> 5120 in
  // binary16 26.7 / 26.3, 26.2 / 26.9, 27.3 / 27.5.  At rank 32, where two passes are needed from 8192 columns on, the
  // launch-per-step kernels are ahead as long as their expand, a workgroup per segment and 512 columns, is resident at once, four per
  // unit: 12544 -> 9216, 36 / 40 / 48 segments 16.3 / 19.4, 17.2 / 19.9, 19.2 / 20.3, -> 11008, 46 / 48 segments 20.8 / 21.3, 21.9 /
  // 21.5, -> 13824, 36 / 39 segments 18.1 / 21.0, 22.6 / 21.3; beyond 48 segments, 53 of 11008 -> 9216 20.6 / 19.7)
  const int cslice = ceil_div(ceil_div(p->h_out, s), 8) * 8;
  const bool one_pass = cslice == 0 || cslice <= 256 / fused_lane_groups(p->r, cslice, single_add_on) * 8;
  const bool many = padded > 48 || (p->r >= 64 ? padded > 40 && (p->dtype == SGMV_F16 || one_pass)
                                               : one_pass || (long long)n_segs * ceil_div(p->h_out, 512) > 4 * lim.fused_workgroups);
  if (p->path == SGMV_PATH_AUTO && p->ksplit == 0 && p->r >= 32 &&
      !(eight && (by_rows || many)) && (long long)s * n_segs > lim.fused_workgroups) {
    const long long wg = (long long)s * n_segs;
    const long long rounds = ceil_div((int)wg, lim.fused_workgroups);
    if (rounds * lim.fused_workgroups * 5 > wg * 6) return false;  // more than 20 % of the slots idle
  }
  // likewise batches of more than 128 segments that need two slices each (measured at
  // h = 4096, r = 16: 192 segments 17.3 us here against 15.5 us, 256 segments 20.0 against 18.3)
  // (not so rows of longer segments: 129 .. 256 of them at two slices share their weights)
  if (p->path == SGMV_PATH_AUTO && p->ksplit == 0 && !by_rows && n_segs > lim.fused_workgroups / 2 &&
      (long long)s * n_segs > lim.fused_workgroups)
    return false;
  f->S = s;
  f->kslice = ceil_div(ceil_div(p->h_in, s), 8) * 8;
  f->cslice = ceil_div(ceil_div(p->h_out, s), 8) * 8;
  f->G = fused_lane_groups(p->r, f->cslice, single_add_on);
  return true;
}

// Launch shape of the single-launch kernel without hand-off (one-row segments, every workgroup
// computes the whole shrink); false when it does not apply.
// by_rows: the launch's items are the rows of the batch (pass n_tokens for n_segs), each looking its
// segment up on the device, so the segments may have any length.
bool choose_whole(const sgmv_problem* p, int n_segs, WholeArgs* w, bool by_rows = false) {
  w->by_rows = by_rows;
  if (p->max_seg_len != 1 && !by_rows) return false;
  if (p->h_in > kWholeMaxHin) return false;
  // A_i is walked in whole steps of 256 128-bit loads
  if ((long long)p->h_in * (p->r / 8) % 256 != 0) return false;
  if (n_segs > 8 * 65535) return false;  // grid depth
  const Limits lim = limits();
  // as many column slices as keep the launch within one workgroup per compute unit
  int s = p->ksplit > 0 ? p->ksplit : lim.fused_workgroups / n_segs;
  if (p->ksplit == 0 && s > kFusedSlices) s = kFusedSlices;
  if (p->ksplit == 0) {
    int pw = 1;
    while (pw * 2 <= s) pw *= 2;
    s = pw;
  }
  if (s > p->h_out / 64) s = p->h_out / 64;
  if (s < 1) s = 1;
  w->S = s;
  w->cslice = ceil_div(ceil_div(p->h_out, s), 8) * 8;
  const int chunks = w->cslice / 8;
  const int most = p->r <= 16 ? 2 : 8;  // lane groups: as choose_fused
  int g = 1;
  while (g * 2 <= most && 256 / (g * 2) >= chunks) g *= 2;
  if (most == 2 && g == 1 && chunks <= 128) g = 2;
  while (p->r / g > 16) g *= 2;
  w->G = g;
  return true;
}

// Launch shape of the single-launch MFMA kernel; false when it does not apply.
// n_proj > 1: that many add-ons of this shape side by side in one launch (each segment's row blocks
// and slices once per add-on, all resident together).
bool choose_tile(const sgmv_problem* p, int n_segs_one, TileArgs* t, int n_proj = 1) {
  const int n_segs = n_segs_one * n_proj;
  const long long n_rows = (long long)p->n_tokens * n_proj;
  if (!p->workspace_ready) return false;
  const Limits lim = limits();
  if (p->max_seg_len <= 0 || p->max_seg_len > kTileMaxSegLen) return false;
  if (n_segs > kFusedMaxWorkgroups) return false;
  // At rank 64 a full block of sixteen rows hands 8 KB of tagged words per slice from workgroup
  // to workgroup, and the launch-per-step MFMA kernels are ahead from about ten rows per segment
  // on (h = 4096, one segment of 16 / 64 / 256 rows: 13.1 / 15.5 / 15.7 us against 21.2 / 20.8 /
  // 21.3 here; four segments of 12 rows: 13.5 against 18.0; sixteen of 8 rows: 14.5 against 15.6)
  // (a joint launch of several add-ons hands them over side by side in the same 20 us, where the
  // launch-per-step kernels ran one add-on after the other: 47.7 us for three of two segments of 64
  // rows.  Side by side these are ahead too, 20.5 against 23.3 here, of 32 rows 18.4 against 22.5, so
  // from 64 rows on a joint launch is no longer the better one, by 10-20 %)
  if (p->path == SGMV_PATH_AUTO && p->r >= 64 && p->max_seg_len > 8 && (n_proj < 2 || p->n_tokens < 64)) return false;
  const int cap = split_cap(p->n_tokens);
  const int narrow = p->h_in < p->h_out ? p->h_in : p->h_out;
  int z = ceil_div(p->max_seg_len, 16);
  // The launch has n_segs * z row blocks, but only those that hold rows keep a compute unit
  // (the others leave at once): at most n_segs + n_tokens / 16 of them.  These, times the
  // slices, must all be resident together (one workgroup per unit).
  long long blocks = (long long)n_segs * z;
  long long live = blocks < (long long)n_segs + n_rows / 16 ? blocks : (long long)n_segs + n_rows / 16;
  if (live > lim.fused_workgroups) {  // too many even with one slice: fewer row blocks, walked with a stride
    z = lim.fused_workgroups / n_segs > 0 ? lim.fused_workgroups / n_segs : 1;
    blocks = live = (long long)n_segs * z;
  }
  // (Fewer row blocks per segment than the longest one needs would leave room for more slices
  // where the weight slices do not fit the LDS, but workgroups that walk several blocks in turn
  // measured slower than the launch-per-step kernels.)
  int s = p->ksplit > 0 ? p->ksplit : (int)(lim.fused_workgroups / live);
  if (p->ksplit == 0 && s > kFusedSlices) s = kFusedSlices;
  if (p->ksplit == 0 && s > lim.tile_max_grid / blocks) s = (int)(lim.tile_max_grid / blocks);  // workgroups launched in all
  if (s > narrow / 64) s = narrow / 64;  // no slice thinner than 64
  if (s > cap / n_proj) s = cap / n_proj;  // every add-on its own exchange words
  if (s < 1) s = 1;
  if (s * n_proj > cap) return false;
  if (s * live > lim.fused_workgroups || s * blocks > lim.tile_max_grid) return false;
  for (;; ++s) {  // more slices make the LDS-resident weight slices smaller
    t->kslice = ceil_div(ceil_div(p->h_in, s), 32) * 32;
    t->cslice = ceil_div(ceil_div(p->h_out, s), 64) * 64;
    t->lds_bytes = tile_lds_bytes(p->r, t->kslice, t->cslice);
    if (t->lds_bytes <= kTileMaxLds) break;
    if (p->ksplit > 0 || (s + 1) * n_proj > cap || (s + 1) * live > lim.fused_workgroups || (s + 1) * blocks > lim.tile_max_grid)
      return false;
  }
  t->S = s;
  t->Z = z;
  t->n_proj = n_proj;
  return true;
}

void fill_fused(FusedArgs* f, const sgmv_problem* p, const Scratch& sc, const int32_t* seg_starts,
                int n_segs, int layer_idx, float scale) {
  f->bf16 = p->dtype == SGMV_BF16;
  f->r = p->r;
  f->h_in = p->h_in;
  f->h_out = p->h_out;
  f->n_tokens = p->n_tokens;
  f->n_segs = n_segs;
  f->spin_limit = spin_limit_of(p);
  f->offA = (long long)layer_idx * p->h_in * p->r;
  f->offB = (long long)layer_idx * p->r * p->h_out;
  f->seg_starts = seg_starts;
  f->exch = sc.exch;
  f->header = sc.header;
  f->scale = scale;
  f->n_proj = 0;
  f->Z = 1;
  f->y = nullptr;
  f->x = nullptr;
  f->A_ptrs = f->B_ptrs = nullptr;
}

// Everything of a tile launch but its shape (choose_tile) and the add-on's own pointers.
void fill_tile(TileArgs* t, const sgmv_problem* p, const Scratch& sc, const int32_t* seg_starts, int n_segs,
               int layer_idx, float scale) {
  t->bf16 = p->dtype == SGMV_BF16;
  t->r = p->r;
  t->h_in = p->h_in;
  t->h_out = p->h_out;
  t->n_tokens = p->n_tokens;
  t->n_segs = n_segs;
  t->spin_limit = spin_limit_of(p);
  t->offA = (long long)layer_idx * p->h_in * p->r;
  t->offB = (long long)layer_idx * p->r * p->h_out;
  t->y = nullptr;
  t->x = nullptr;
  t->A_ptrs = t->B_ptrs = nullptr;
  t->seg_starts = seg_starts;
  t->exch = sc.exch;
  t->header = sc.header;
  t->scale = scale;
}

// Workgroup shape of the vector expand for `n_segs` items (segments, or rows of a per-row launch):
// 64, 128 or 256 threads of eight columns each, or kExpandSplit.
int choose_expand_threads(const sgmv_problem* p, int n_segs) {
  if (p->expand_threads) return p->expand_threads;
  // From rank 32 on a lane of the plain kernel walks its R weight rows sixteen at a time, one
  // memory round trip after the other; while the launch is small the kernel whose four waves
  // divide the rows among themselves is ahead (measured at h = 4096, one-row segments, us per
  // call, plain against divided: rank 64, 1 / 16 / 64 / 128 segments 8.5 / 10.2 / 12.9 / 17.2
  // against 3.9 / 5.4 / 8.4 / 14.6; rank 32, 16 / 64 / 128: 6.0 / 7.7 / 10.2 against 3.9 / 5.5 /
  // 8.2; 4096 -> 11008, 64 segments, rank 32 / 64: 11.7 / 19.0 against 9.9 / 17.1), up to about
  // five and a half of its workgroups per compute unit (1408: ahead; 192 segments at rank 64,
  // 1536: 19.2 against 20.6; 256 at rank 32, 2048: 13.3 against 14.5)
  if (p->r >= 32 && (long long)n_segs * ceil_div(p->h_out, 512) <= 11LL * compute_units() / 2) return kExpandSplit;
  const int sizes[3] = {256, 128, 64};
  for (int i = 0; i < 3; ++i)
    if ((long long)n_segs * ceil_div(p->h_out, sizes[i] * 8) >= kTargetWorkgroups / 2 ||
        i == 2)
      return sizes[i];
  return 64;
}

ShrinkArgs make_shrink(const sgmv_problem* p, const Scratch& sc, const void* x,
                       const void* const* A_ptrs, const int32_t* seg_starts, int n_segs,
                       int layer_idx) {
  ShrinkArgs a;
  a.bf16 = p->dtype == SGMV_BF16;
  a.r = p->r;
  a.h_in = p->h_in;
  a.n_tokens = p->n_tokens;
  a.n_segs = n_segs;
  a.ksplit = a.kslice = 0;
  a.max_seg_len = p->max_seg_len;
  a.by_rows = false;
  a.layer_off = (long long)layer_idx * p->h_in * p->r;
  a.x = x;
  a.A_ptrs = A_ptrs;
  a.seg_starts = seg_starts;
  a.partials = sc.partials;
  a.header = sc.header;
  a.n_proj = 1;
  a.same_x = false;
  a.xs[0] = x;
  a.As[0] = A_ptrs;
  a.partials_of[0] = sc.partials;
  return a;
}

ExpandArgs make_expand(const sgmv_problem* p, void* y, const float* v_parts, int nparts,
                       const void* const* A_ptrs, const void* const* B_ptrs,
                       const int32_t* seg_starts, int n_segs, int layer_idx, float scale) {
  ExpandArgs a;
  a.bf16 = p->dtype == SGMV_BF16;
  a.r = p->r;
  a.h_out = p->h_out;
  a.n_tokens = p->n_tokens;
  a.n_segs = n_segs;
  a.threads = choose_expand_threads(p, n_segs);
  a.layer_off = (long long)layer_idx * p->r * p->h_out;
  a.y = y;
  a.v_parts = v_parts;
  a.nparts = nparts;
  a.A_ptrs = A_ptrs;
  a.B_ptrs = B_ptrs;
  a.seg_starts = seg_starts;
  a.scale = scale;
  a.three_parts = false;
  a.vh = a.vl = nullptr;
  a.undo = nullptr;
  a.header = nullptr;
  a.by_rows = false;
  return a;
}

// A per-row launch whose items are pairs of rows of one segment, which then read the segment's weights once.  Only where
// a launch of an item per row is out, being too many workgroups (wide inputs, whose slices are many): where it applies it
// is ahead although it reads more, the second row's arithmetic and the empty places costing 0.3 to 1 us (45 rows of 18
// segments, 5120 wide, rank 32, bfloat16 8.1 / 8.5 us per row / per pair; 64 rows of 42, 4096 wide, rank 16 5.5 / 6.4).
// Fewer than four slices leave a workgroup too much (120 rows of 15 segments, 5120 wide, rank 32, three slices 11.0 with the
// tile kernel / 12.7).
bool choose_fused_pairs(const sgmv_problem* p, int n_segs, FusedArgs* f) {
  if (p->path != SGMV_PATH_AUTO || p->n_tokens <= 64 || p->r > 32 || n_segs > p->n_tokens) return false;
  if (!choose_fused(p, pair_places(p->n_tokens, n_segs), f, true, true) || f->S < 4) return false;
  f->paired = true;
  return true;
}

// The add-on in such a launch (`tile_slices`: of the tile kernel, 0 where it does not apply).  Measured, us, what was taken
// before / pairs: 11008 -> 4096, rank 8, 128 rows: Uniform 15.5 / 10.0, Skewed 11.3 / 9.0, 64 x 2 rows 12.0 / 9.0; 13824 -> 5120, rank
// 8, 16 x 8 rows 9.6 / 7.1; rank 16, Skewed of 120 rows 14.0 / 12.8, 9992 -> 3000, 64 x 2 rows 14.4 / 11.9; 8192 -> 8192, rank 8, Skewed of
// 256 rows 13.0 / 11.5; rank 32: 5120 -> 5120, Skewed of 96 rows 14.2 / 12.0, 6144 -> 4096 15.4 / 10.1, 8192 -> 8192 16.5 / 14.0.
// Left to the others:
//  * from rank 16 on where the tile kernel has six slices or more (12000 -> 1024, rank 16, 33 x 3 rows 10.0 / 13.0; 9992 ->
//    3000, 6 x 20 rows 8.9 / 11.4), at rank 8 six or seven (128 rows of 42 segments 8.9 / 9.7; eight 9.6 / 7.1, above);
//  * from rank 16 on more than 128 rows (8192 -> 8192, rank 16, Skewed of 256 rows 14.5 / 18.4);
//  * column slices beyond 1024 columns at rank 16, a pass with two lane groups, and beyond 2048 at the others, a pass of rank 8 with one
//    and two passes of rank 32 with two (11008 -> 11008, rank 16, Skewed of 128 rows 13.9 / 18.7;
//    8192 -> 28672, rank 8, 12 x 20 rows 16.0 / 21.9, rank 32, Skewed of 66 rows 19.9 / 25.7);
//  * at rank 32 more than a workgroup per unit (11008 -> 4096, Skewed of 128 rows 16.8 / 17.3);
//  * to the tile kernel up to rank 16, where pairs are more than two workgroups per unit and no segment is long (three rows take two
//    pairs' places but one block of the tile kernel, which takes several for more than sixteen): at rank 16 segments of 3 to 48 rows (9992 ->
//    1024, 101 rows of 51 10.4 / 13.8, 110 rows of 23 10.4 / 12.2; 253 such points 1.08 times as fast on the tile kernel, 147 others
//    1.24 times on pairs, 0.99 at least: 13824 -> 2048, 51 x 2 rows 12.5 / 11.1), at rank 8, where the tile kernel has five slices and more,
//    of 5 to 32 rows, more than three and a half on average (9992 -> 1024, 116 rows of 20 8.1 / 9.7; 74 points 1.02 times on the tile
//    kernel, 326 others 1.27 times on pairs: 11008 -> 4096, 101 rows of 47, in a layer of seven projections 40.9 / 36.5).
//    Segments all of one even length up to twelve are pairs without an empty place: 39 points 1.13 times as fast on pairs, 0.89 at worst
//    (13824 -> 368, rank 16, 15 x 8 rows 1.35; 13824 -> 5120, rank 8, 16 x 8 rows 9.6 / 7.1; 9992 -> 320, rank 8, 38 x 6 rows 0.89).
bool choose_add_on_pairs(const sgmv_problem* p, int n_segs, int tile_slices, FusedArgs* f) {
  if (p->r == 8 ? tile_slices == 6 || tile_slices == 7 : tile_slices >= 6 || p->n_tokens > 128) return false;
  if (!choose_fused_pairs(p, n_segs, f) || f->cslice > (p->r == 16 ? 1024 : 2048)) return false;
  const int units = limits().fused_workgroups;
  if (p->r == 32) return (long long)f->S * f->items <= units;
  if (tile_slices == 0 || f->S * fused_grid_items(f->items) <= 2 * units) return true;
  if (p->max_seg_len % 2 == 0 && p->max_seg_len <= 12 && p->n_tokens == (long long)n_segs * p->max_seg_len) return true;
  if (p->r == 8) return tile_slices < 5 || p->max_seg_len <= 4 || p->max_seg_len > 32 || 2LL * p->n_tokens <= 7LL * n_segs;
  return p->max_seg_len > 48 || (p->max_seg_len == 2 && 4LL * p->n_tokens > 7LL * n_segs);
}

// The stand-alone shrink: rank 8, 13824 wide, Uniform of 128 rows 15.4 / 7.2, 11008 wide, 16 x 8 rows 10.5 / 5.3; rank 16, 13824 wide,
// 64 x 2 rows 12.3 / 9.9, 9992 wide, Skewed of 256 rows, five slices, 12.5 / 10.1.  With four slices the workgroup per row without
// Split-K is ahead on most batches (7168 wide, rank 16, Uniform of 256 rows 8.4 / 10.1), and at rank 32 pairs gain for sure only
// on many short segments (11008 wide, Uniform of 120 rows 21.2 / 13.2, 9992 wide, 64 x 2 rows 14.9 / 12.0; 33 x 3 rows 11.4 /
// 11.9; against the MFMA kernels 128 rows of 6 segments, 12000 wide, 7.9 / 9.1).
bool choose_shrink_pairs(const sgmv_problem* p, int n_segs, FusedArgs* f) {
  if (!choose_fused_pairs(p, n_segs, f) || f->S < 5) return false;
  return p->r < 32 || (f->S >= kFusedSlices && !use_matrix(p, n_segs) && 2LL * p->n_tokens <= 5LL * n_segs);
}

// Small batches of segments longer than a row (or of unknown length): whether AUTO runs the
// one-row kernel with the hand-off per ROW of the batch (SGMV_PATH_ROWS), every row's workgroups
// reading the row's adapter through the caches, rather than the tile kernel (`tile`: it applies, with
// `tile_slices` slices) or the launch-per-step kernels.  Measured on MI355X, binary16, us per add-on,
// per row against what AUTO took before:
//  * up to 64 rows it wins at every rank and width measured (ranks 8 .. 64; 4096, 5120, 8192 square,
//    4096 -> 11008, 11008 -> 4096; 31 segment mixes and five popularity mixes each: 129 of 132 cases at
//    rank 64 faster, the rest within 2 %).  At 4096 x 4096, rank 16, 64 rows: Uniform 5.33 against
//    7.16 (tile kernel), Skewed 4.88 against 7.58, Identical 4.88 against 7.23, 8 segments of 8 rows
//    4.85 against 7.12; rank 64: Uniform 11.7 against 22.7 (MFMA kernels), 8 x 8 rows 9.4 against 14.2.
//  * 65 .. 128 rows: ahead up to rank 32 (rank 16, 128 rows: Uniform 6.40 against 9.29, Skewed 6.13
//    against 11.9, one segment 5.79 against 7.27, 16 x 8 rows 5.85 against 7.60; rank 32: 4 x 32 rows
//    7.96 against 10.3, Uniform 9.16 against 11.4; behind by at most 12 % on 24 segments of 4 rows
//    at rank 32 and on 32 x 4 rows at 5120), not at rank 64 (two slices per row leave each workgroup
//    half of B_i: 4096 -> 11008, 8 x 16 rows: 27.2 against 17.3).
//  * 129 .. 256 rows, ranks up to 16: ahead where the tile kernel does not apply or gets fewer than
//    its eight slices (Skewed of 256 rows 9.05 against 18.9, Uniform 7.88 against 9.83, 128 x 2 rows
//    11.7 against 14.7; behind on 40 .. 64 segments of 4 rows, by up to 17 %), 4-8 % ahead elsewhere,
//    which is left to the tile kernel.
bool rows_apply(const sgmv_problem* p, int n_segs, bool tile, int tile_slices) {
  if (p->max_seg_len == 1 || p->ksplit != 0 || !p->workspace_ready) return false;
  // the look-up takes a round per 64 segments: not for batches of mostly empty segments
  if (n_segs > kRowsMostSegments) return false;
  if (p->n_tokens <= 64) return true;
  // (rank 64 at 65 .. 128 rows: only at widths up to 4096 and where the tile kernel is out: Uniform
  // of 128 rows 15.3 against 44.5 us, one segment of 128 rows 12.8 against 17.4, 32 x 4 rows 17.6
  // against 19.6; with the tile kernel to choose from, 16 x 8 rows 16.6 against 15.5)
  if (p->n_tokens <= 128)
    return p->r <= 32 || (!tile && p->h_in <= 4096 && p->h_out <= 4096);
  if (p->n_tokens <= 256) return p->r <= 16 && (!tile || tile_slices < 8);
  //  * 257 .. 384 rows, ranks up to 16, inputs up to 4096 wide (two slices): only where the tile kernel
  //    is out or down to three slices (Skewed of 320 / 384 rows 11.0 / 11.9 against 19.8 / 18.4 us on the
  //    MFMA kernels, 96 x 4 rows 14.0 against 17.2 on the vector kernels; the tile kernel with four
  //    slices and more is ahead by 5-28 %, and at 512 rows, 1024 workgroups, nearly everything is)
  if (p->n_tokens <= 384) return p->r <= 16 && p->h_in <= 4096 && (!tile || tile_slices < 4);
  return false;
}

// The stand-alone expand of a small batch of longer segments (or of unknown length): a workgroup
// per row and column strip instead of per segment, as the add-on does (rows_apply); no workspace
// is involved.
bool expand_by_rows(const sgmv_problem* p, int n_segs) {
  if (p->path != SGMV_PATH_AUTO || p->max_seg_len == 1 || n_segs > kRowsMostSegments) return false;
  if (p->n_tokens <= 64) return true;
  if (p->n_tokens <= 128) return p->r <= 32;
  return p->n_tokens <= 384 && p->r <= 16;
}

// What sgmv_add_lora will launch for a checked problem: the single source of the path
// choice, shared by the entry points and by sgmv_plan_add_lora.
struct SinglePlan {
  int kernel;        // sgmv_kernel
  WholeArgs whole;   // SGMV_KERNEL_WHOLE
  TileArgs tile;     // SGMV_KERNEL_TILE
  FusedArgs fused;   // SGMV_KERNEL_FUSED
  int ksplit, kslice;  // SGMV_KERNEL_MATRIX / SGMV_KERNEL_VECTOR
  bool direct;         // SGMV_KERNEL_MATRIX: the expand adds the partial sums up itself
};

// pairs: whether rows may be taken two to an item (choose_add_on_pairs).
int plan_single(const sgmv_problem* p, int n_segs, SinglePlan* pl, bool pairs = true) {
  if (p->path == SGMV_PATH_WHOLE) {
    if (!choose_whole(p, n_segs, &pl->whole)) return SGMV_ERR_UNSUPPORTED;
    pl->kernel = SGMV_KERNEL_WHOLE;
    return SGMV_OK;
  }
  if (p->path == SGMV_PATH_ROWS) {
    if (!choose_fused(p, p->n_tokens, &pl->fused, true, true)) return SGMV_ERR_UNSUPPORTED;
    pl->kernel = SGMV_KERNEL_FUSED;
    return SGMV_OK;
  }
  const bool tile = (p->path == SGMV_PATH_AUTO || p->path == SGMV_PATH_FUSED) && p->max_seg_len != 1 &&
                    choose_tile(p, n_segs, &pl->tile);
  if (p->path == SGMV_PATH_AUTO && rows_apply(p, n_segs, tile, tile ? pl->tile.S : 0)) {
    // with an A_i of at most 64 KB the kernel without hand-off, as for one-row segments below
    if ((long long)p->h_in * p->r <= 32768 && p->n_tokens <= 512 && choose_whole(p, p->n_tokens, &pl->whole, true)) {
      pl->kernel = SGMV_KERNEL_WHOLE;
      return SGMV_OK;
    }
    if (choose_fused(p, p->n_tokens, &pl->fused, true, true) ||
        (pairs && choose_add_on_pairs(p, n_segs, tile ? pl->tile.S : 0, &pl->fused))) {
      pl->kernel = SGMV_KERNEL_FUSED;
      return SGMV_OK;
    }
  }
  if (tile) {
    pl->kernel = SGMV_KERNEL_TILE;
    return SGMV_OK;
  }
  if (p->path == SGMV_PATH_AUTO || p->path == SGMV_PATH_FUSED) {
    const bool fused = choose_fused(p, n_segs, &pl->fused);
    // One-row segments, measured on MI355X at h = 4096 (us per add-on, whole-shrink kernel
    // against the alternative): at rank 8, where A_i is small, it beats the kernel with the
    // hand-off at every batch (1 / 16 / 64 / 128 segments: 3.7 / 4.0 / 4.8 / 6.0 against 4.1 /
    // 4.7 / 5.2 / 6.2) and the launch-per-step kernels beyond (256: 9.5 against 12.4), but only
    // while A_i is small: at h_in = 8192 the hand-off kernel is 15-20 % ahead at every batch (64
    // segments: 6.2 against 7.4), at 5120 from 64 segments on (5.4 against 6.0; bfloat16 from 32 on); where the
    // hand-off kernel does not apply (no prepared workspace, or more segments than it takes) it
    // beats the launch-per-step kernels up to rank 16 and several hundred segments (192 / 256 /
    // 512: 13.5 / 16.4 / 28.8 against 16.2 / 18.6 / 29.9; 1024: 53.9 against 51.2), without a
    // workspace also at rank 32 (64 segments: 13.0 against 14.2; rank 64: 23.8 against 22.5).
    // For binary16 it is also ahead up to rank 16 where the input is so wide that the hand-off
    // kernel must take an odd number of slices and with them more workgroups than compute
    // units (h = 5120, three slices, 96 / 112 / 128 segments: 11.5 / 12.4 / 13.7 against 13.1 /
    // 13.7 / 14.6; bfloat16 at 128 segments: 15.2 against 14.8, so not there; 72 / 80 segments,
    // at most one workgroup per unit: 10.5 / 11.0 against 8.1 / 8.8, so not there either).
    // (the same wherever A_i is at most 64 KB, whatever the rank: h = 1024, rank 16, 1 / 8 / 32 / 64
    // segments 3.1 / 3.3 / 3.6 / 3.7 against 3.7 / 3.9 / 4.4 / 4.4; h = 2048, rank 16, 8 / 64 segments 4.0 /
    // 4.8 against 4.2 / 4.7; h = 1024, rank 32: 4.1 against 4.5; with 128 KB, h = 1024 at rank 64: 5.5 against 4.5)
    const bool small_a = (long long)p->h_in * p->r <= 32768;
    const bool odd_slices = fused && p->dtype == SGMV_F16 && (pl->fused.S & (pl->fused.S - 1)) != 0 &&
                            pl->fused.S * n_segs > limits().fused_workgroups;
    if (p->path == SGMV_PATH_AUTO && p->ksplit == 0 && choose_whole(p, n_segs, &pl->whole) &&
        (((p->r == 8 || small_a) && n_segs <= 512 && (!fused || p->h_in <= 4096 || small_a)) ||
         ((!fused || odd_slices) && n_segs <= 640 && p->r <= (p->workspace_ready ? 16 : 32)))) {
      pl->kernel = SGMV_KERNEL_WHOLE;
      return SGMV_OK;
    }
    if (fused) {
      pl->kernel = SGMV_KERNEL_FUSED;
      return SGMV_OK;
    }
    if (p->path == SGMV_PATH_FUSED) return SGMV_ERR_UNSUPPORTED;
  }
  if (use_matrix(p, n_segs)) {
    const MatrixSplit m = choose_split_matrix(p, n_segs, 1, false);
    pl->ksplit = m.ksplit;
    pl->kslice = m.kslice;
    pl->direct = m.direct;
    pl->kernel = SGMV_KERNEL_MATRIX;
    return SGMV_OK;
  }
  if (!choose_split(p, n_segs, &pl->ksplit, &pl->kslice)) return SGMV_ERR_UNSUPPORTED;
  pl->kernel = SGMV_KERNEL_VECTOR;
  return SGMV_OK;
}

// What sgmv_shrink launches: shared by the entry point and sgmv_plan_shrink.
struct ShrinkPlan {
  bool whole_by_rows;  // SGMV_KERNEL_WHOLE: a workgroup per row of the batch, not per segment
  int kernel;          // SGMV_KERNEL_FUSED (hand-off inside one launch), _MATRIX or _VECTOR (+ reduction launch)
  FusedArgs fused;     // SGMV_KERNEL_FUSED
  int ksplit, kslice;  // the others
};

int plan_shrink(const sgmv_problem* p, int n_segs, ShrinkPlan* pl) {
  // one-row segments with a prepared workspace: one launch, the partial sums handed over inside
  // it (measured at h = 4096, r = 16, 1 / 16 / 64 / 128 segments: 3.5 / 4.0 / 5.0 / 6.6 us against
  // 4.8 / 6.1 / 6.7 / 8.1 us for shrink + reduction; r = 64, 64 segments: 9.5 against 10.7)
  sgmv_problem shrink_only = *p;
  shrink_only.h_out = 0;  // the output width plays no part here (and need not be set by the caller)
  // one workgroup per one-row segment computes the whole product: no Split-K, no second launch
  const bool whole_shape = p->ksplit == 0 && p->h_in <= kWholeMaxHin && (long long)p->h_in * (p->r / 8) % 256 == 0;
  const bool whole_fits = p->max_seg_len == 1 && whole_shape;
  pl->whole_by_rows = false;
  if (p->path == SGMV_PATH_WHOLE) {
    if (!whole_shape) return SGMV_ERR_UNSUPPORTED;
    pl->whole_by_rows = p->max_seg_len != 1;  // longer segments (or unknown): per row of the batch
    pl->kernel = SGMV_KERNEL_WHOLE;
    return SGMV_OK;
  }
  // Measured on MI355X, us per call, against the launch with the hand-off (up to 128 segments) and
  // the two launches of the vector kernels (beyond): where A_i is at most 128 KB (h_in * r <= 65536)
  // it is ahead at every batch (h = 4096, rank 16, 1 / 32 / 64 / 128 / 256 / 512 segments: 3.4 / 3.9 /
  // 4.8 / 5.8 / 8.6 / 15.0 against 3.65 / 4.3 / 5.0 / 6.6 / 11.4 / 16.6; rank 8, 64 segments: 3.2
  // against 4.1); with a larger A_i only beyond the hand-off's batches (256 segments, rank 32:
  // 14.8 against 16.0; h = 8192: 15.3 against 16.6; but 64 segments at rank 64: 16.8 against 9.5);
  // from about 100 MB of weights on the Split-K kernels stream better (1024 segments at rank 16:
  // 27.8 against 26.9; 512 at rank 64: 48.1 against 46.5).
  // (an A_i of 64 .. 128 KB: only where all of it is in flight in at most two batches, and in bfloat16,
  // whose conversions this kernel does not hide as well, only from 96 segments on: h = 4096, rank 16,
  // 16 / 64 / 96 segments 4.2 / 5.3 / 6.0 against 3.8 / 4.8 / 6.7)
  const long long a_elems = (long long)p->h_in * p->r;
  const bool whole_small = a_elems <= 32768 || (a_elems <= 65536 && a_elems % (16 * 256 * 8) == 0 &&
                                                (p->dtype == SGMV_F16 || n_segs >= 96));
  const bool fused = p->path == SGMV_PATH_AUTO && p->ksplit == 0 && choose_fused(&shrink_only, n_segs, &pl->fused);
  if (p->path == SGMV_PATH_AUTO && whole_fits && (long long)n_segs * p->h_in * p->r <= kShrinkWholeMostElements &&
      (whole_small || (!fused && n_segs > 128))) {
    pl->kernel = SGMV_KERNEL_WHOLE;
    return SGMV_OK;
  }
  if (fused) {
    pl->kernel = SGMV_KERNEL_FUSED;
    return SGMV_OK;
  }
  // Small batches of longer segments (or of unknown length), per row of the batch.  With a small A_i
  // a workgroup per row without Split-K (measured at h = 4096, binary16, against the per-row launch
  // with the hand-off below, from 512 rows the MFMA kernels: rank 16, Uniform of 64 / 128 / 256 /
  // 384 / 512 rows 3.85 / 4.1 / 4.9 / 6.3 / 6.4 against 4.6 / 5.2 / 6.2 / 7.3 / 8.8 us, Identical of
  // 1024 rows 8.2 against 7.8; rank 8, Uniform of 64 rows 2.9 against 4.0; rank 32, where A_i is
  // 256 KB: 64 rows 6.6 against 5.5, 256 rows 7.2 against 9.3)
  const bool fused_rows = p->path == SGMV_PATH_AUTO && rows_apply(p, n_segs, false, 0) &&
                          (choose_fused(&shrink_only, p->n_tokens, &pl->fused, true, true) ||
                           choose_shrink_pairs(&shrink_only, n_segs, &pl->fused));
  {
    const bool small = a_elems <= 32768 || (a_elems <= 65536 && a_elems % (16 * 256 * 8) == 0 &&
                                            (p->dtype == SGMV_F16 || p->n_tokens >= 96));
    if (p->path == SGMV_PATH_AUTO && p->max_seg_len != 1 && whole_shape && n_segs <= kRowsMostSegments &&
        p->n_tokens <= 512 && (small || (!fused_rows && p->n_tokens > 128 && a_elems <= 131072))) {
      pl->whole_by_rows = true;
      pl->kernel = SGMV_KERNEL_WHOLE;
      return SGMV_OK;
    }
  }
  // else the launch with the hand-off per row of the
  // batch, as for the add-on (rows_apply; measured at h = 4096 against the better of the
  // launch-per-step kernels: rank 16, Uniform / Skewed / Identical of 64 rows 4.6 / 4.4 / 4.1 against
  // 7.7 / 7.3 / 6.7 us, of 256 rows 5.5 / 5.7 / 4.8 against 8.6 / 9.5 / 6.9; rank 64, 64 rows: 7.0 /
  // 6.5 / 5.6 against 10.5 / 10.9 / 9.8)
  if (fused_rows) {
    pl->kernel = SGMV_KERNEL_FUSED;
    return SGMV_OK;
  }
  if (use_matrix(p, n_segs)) {
    const MatrixSplit m = choose_split_matrix(&shrink_only, n_segs, 1, false);
    pl->ksplit = m.ksplit;
    pl->kslice = m.kslice;
    pl->kernel = SGMV_KERNEL_MATRIX;
    return SGMV_OK;
  }
  if (!choose_split(p, n_segs, &pl->ksplit, &pl->kslice)) return SGMV_ERR_UNSUPPORTED;
  pl->kernel = SGMV_KERNEL_VECTOR;
  return SGMV_OK;
}

// Multi-projection call: SGMV_KERNEL_MULTI_SIDE / _PIPELINED with the launch shape in *f (per
// segment, or per row of the batch when f->by_rows), SGMV_KERNEL_TILE with the shape in *t (groups
// of t->n_proj add-ons per launch), or SGMV_KERNEL_SEQUENCE (one sgmv_add_lora after the other).
int plan_multi(const sgmv_problem* p, int n_segs, int n_proj, FusedArgs* f, TileArgs* t) {
  const Limits lim = limits();
  const bool one_row = p->max_seg_len == 1;
  if (n_proj < 2) return SGMV_KERNEL_SEQUENCE;
  // Segments longer than a row in a small batch: where a single add-on runs the one-row kernel
  // per row of the batch (plan_single), so may the add-ons of this call, side by side
  bool per_row = false;
  if (!one_row && p->ksplit == 0 && (p->path == SGMV_PATH_AUTO || p->path == SGMV_PATH_ROWS)) {
    FusedArgs rows;
    TileArgs one;
    const bool tile_one = p->path == SGMV_PATH_AUTO && choose_tile(p, n_segs, &one);
    per_row = (p->path == SGMV_PATH_ROWS || rows_apply(p, n_segs, tile_one, tile_one ? one.S : 0)) &&
              choose_fused(p, p->n_tokens, &rows, true, true);
  }
  // The add-ons in one launch of the one-row kernels: one set of S workgroups per segment (or per
  // row of the batch) and add-on, side by side or, for one-row segments, walking the add-ons.
  auto joint_rows = [&]() -> int {
    if (!(p->path == SGMV_PATH_AUTO || p->path == SGMV_PATH_FUSED || per_row) || !(one_row || per_row)) return SGMV_KERNEL_SEQUENCE;
    const int items = per_row ? p->n_tokens : n_segs;  // what a set of S workgroups serves
    if (p->workspace == nullptr || !choose_fused(p, items, f, false, per_row) || f->S * n_proj > split_cap(p->n_tokens))
      return SGMV_KERNEL_SEQUENCE;
    f->r = p->r;
    // workgroups that hold segments count towards what must be resident; the grid, padded to
    // whole rows of segments, must leave every workgroup its own generation copy
    const long long grid = (long long)f->S * fused_grid_items(items) * n_proj;
    if ((long long)f->S * items * n_proj <= lim.multi_workgroups && grid <= kGenerationCopies)
      return SGMV_KERNEL_MULTI_SIDE;
    if (!per_row && fused_multi_fits(*f)) return SGMV_KERNEL_MULTI_PIPELINED;
    // slices too deep for the pipelined kernel's register sets (h_in = 5120 at four slices):
    // three workgroups per compute unit still beat one launch per add-on (measured, three
    // projections of 64 segments at h = 5120: 22.7 us against 24.8 us)
    // (ranks up to 16 only: the kernels of the higher ranks use more registers and fit two per unit)
    if (p->r <= 16 && (long long)f->S * items * n_proj <= lim.multi_workgroups_most && grid <= kGenerationCopies)
      return SGMV_KERNEL_MULTI_SIDE;
    return SGMV_KERNEL_SEQUENCE;
  };
  if (one_row) return joint_rows();
  // Measured at 4096 x 4096, binary16, us for two / three add-ons, per row side by side against
  // the joint tile launch below: rank 16, 64 rows: Uniform 8.1 / 11.0 against 12.6 / 20.5, Skewed
  // 7.2 / 9.1 against 10.0 / 13.7, Identical 6.2 / 7.4 against 7.7 / 8.0, 8 segments of 8 rows
  // 6.2 / 7.4 against 8.4 / 8.8; 128 rows: 16 x 8 rows 8.0 / 11.2 against 9.3 / 10.4, one segment 8.0 /
  // 11.2 against 8.5 / 9.0 (three add-ons of 128 rows are 768 workgroups at two slices); rank 64,
  // 64 rows, two add-ons: 8 x 8 rows 13.1 against 15.7, Identical 11.4 against 20.8.
  // (at rank 32, 128 rows, two add-ons, the tile launch is ahead: one segment 10.9 against 12.2,
  // 16 x 8 rows 11.2 against 14.5)
  // (and at rank 64 per row again, the tile kernel's hand-off being bound by its volume there: two
  // segments of 64 rows 16.8 against 21.2, 16 x 8 rows 23.0 against 31.1 in two tile launches)
  const bool rows_first = per_row && (p->n_tokens <= 64 || ((long long)n_proj * p->n_tokens <= 256 && p->r != 32));
  if (rows_first) {
    const int kernel = joint_rows();
    if (kernel != SGMV_KERNEL_SEQUENCE) return kernel;
  }
  // segments of a few rows: the add-ons side by side in one launch of the tile kernel while all
  // their workgroups are resident together (fewer slices each than a single add-on would get)
  // (t->n_proj: how many go into one launch; when not all of them fit, the call takes groups of
  // that many, and what is left over at the end in a smaller launch)
  bool tile = false;
  if ((p->path == SGMV_PATH_AUTO || p->path == SGMV_PATH_FUSED) && p->ksplit == 0) {
    for (int group = n_proj; group > 1 && !tile; --group) tile = choose_tile(p, n_segs, t, group);
  }
  // against add-ons that run per row side by side, the joint tile launch is ahead only as one
  // launch that keeps at least kTileMultiSlices slices (Skewed of 128 rows, three add-ons: three
  // slices 22.0 us against 11.5 per row; Uniform of 64 rows in two launches 20.5 against 11.0);
  // against add-ons per row one after the other it is ahead also in groups and with fewer slices
  // (four add-ons, rank 8: 32 x 2 rows in two launches 17.5 against 19.4, Skewed of 64 rows at
  // three slices 11.8 against 18.4; rank 32: 32 x 4 rows 30.4 against 40.6)
  // (The launch-per-step kernels, which take the add-ons side by side too, are asked at rank 64 in place of several tile launches,
  // multi_takes_matrix.  From 64 x 4 rows on they are ahead at ranks 16 / 32 too, three add-ons 24.4 / 33.7 against 31.3 / 42.3.)
  if (tile && (!per_row || (t->n_proj == n_proj && t->S >= kTileMultiSlices))) return SGMV_KERNEL_TILE;
  if (per_row && !rows_first) {
    const int kernel = joint_rows();
    if (kernel != SGMV_KERNEL_SEQUENCE) return kernel;
  }
  if (tile) return SGMV_KERNEL_TILE;
  return SGMV_KERNEL_SEQUENCE;
}

// Add-ons of rank 64 that plan_multi gives several launches (`kernel`, `t`): the MFMA kernels, three launches for three of them,
// from four rows per segment on.  Their second product then takes v as three 16-bit parts, all 24 bits of it, as the hand-off and vector
// kernels do, whose calls these mostly are (ExpandArgs::three_parts; two parts give y a relative error of 4.5e-3 in binary16 where v is about 2^-18).
// Measured, us, what was taken before / these, 24 to 400 rows, two to eight add-ons, 256 to 13824 wide, by the launches that were taken
// before (vector kernels two per add-on) to the groups of three:
//  * at least twice as many, 1055 points: 1.47 times as fast on average, six below 0.97, 0.90 at worst; four add-ons of the hand-off
//    kernel only from 50 rows on (45 rows of nine, 1736 -> 1024, 22.8 / 27.3);
//  * fewer, in groups of the tile kernel, 152 points: 0.84 times (four in two launches 0.83, five in two and three 0.82 and 1.08, eight in two,
//    three and four 0.60, 0.82 and 1.00: 4160 -> 2048, 30 rows of five, 21.5 / 52), so those stay.
// Two or three add-ons outside these limits would mostly gain too (8 to 23 rows 1.20 times as fast, down to 0.80; two and three rows per
// segment 1.35, down to 0.87; more than 400 rows 1.35, at two per segment down to 0.73) and are left where they are.
bool multi_takes_matrix(const sgmv_problem* p, int n_segs, int n_proj, int kernel, const TileArgs& t) {
  if (n_proj < 2 || p->path != SGMV_PATH_AUTO || p->ksplit != 0 || p->r != 64 || p->max_seg_len == 1) return false;
  if (p->n_tokens < 24 || p->n_tokens > 400 || p->n_tokens < 4LL * n_segs || p->workspace == nullptr ||
      p->workspace_bytes < sgmv_workspace_bytes_multi(p->n_tokens, p->r, n_proj))
    return false;
  int launches;
  if (kernel == SGMV_KERNEL_TILE) {
    launches = ceil_div(n_proj, t.n_proj);
  } else if (kernel == SGMV_KERNEL_SEQUENCE) {
    SinglePlan one;
    if (plan_single(p, n_segs, &one) != SGMV_OK || one.kernel == SGMV_KERNEL_MATRIX) return false;  // these it takes anyway
    if (one.kernel == SGMV_KERNEL_FUSED && n_proj == 4 && p->n_tokens < 50) return false;
    launches = one.kernel == SGMV_KERNEL_VECTOR ? 2 * n_proj : n_proj;
  } else {
    return false;
  }
  if (launches < 2 * ceil_div(n_proj, kSharedShrinkMost)) return false;
  // the third part of v lies behind the partial sums, half a slice of them: room for it in every group of add-ons
  const int cap = split_cap(p->n_tokens);
  for (int count = n_proj < kSharedShrinkMost ? n_proj : kSharedShrinkMost; count > 0; --count)
    if (choose_split_matrix(p, n_segs, count, true).ksplit >= cap || choose_split_matrix(p, n_segs, count, false).ksplit >= cap) return false;
  return true;
}

}  // namespace

extern "C" {

const char* sgmv_status_string(int status) {
  switch (status) {
    case SGMV_OK: return "ok";
    case SGMV_ERR_NULL: return "a required pointer is NULL";
    case SGMV_ERR_SHAPE: return "invalid size";
    case SGMV_ERR_UNSUPPORTED: return "unsupported dtype, rank, width or option";
    case SGMV_ERR_ALIGN: return "pointer not sufficiently aligned";
    case SGMV_ERR_WORKSPACE: return "workspace missing or too small";
    case SGMV_ERR_RANGE: return "layer_idx out of range";
    case SGMV_ERR_LAUNCH: return "kernel launch failed";
    case SGMV_ERR_TIMEOUT: return "a workgroup gave up waiting for partial sums";
    case SGMV_ERR_STATE: return "workspace not initialised or its launch accounting is inconsistent";
  }
  return "unknown status";
}

size_t sgmv_workspace_bytes(int32_t n_tokens, int32_t r) {
  if (n_tokens <= 0 || r <= 0) return 0;
  // header, fp32 split-K partials, 64-bit exchange words, 16-bit operand pairs of v
  return kWorkspaceHeader + 3 * partial_bytes(n_tokens, r) + operand_bytes(n_tokens, r);
}

size_t sgmv_workspace_bytes_multi(int32_t n_tokens, int32_t r, int32_t n_proj) {
  const size_t single = sgmv_workspace_bytes(n_tokens, r);
  if (single == 0 || n_proj < 2) return single;
  const int shared = n_proj < kSharedShrinkMost ? n_proj : kSharedShrinkMost;
  return single + (size_t)(shared - 1) * (partial_bytes(n_tokens, r) + operand_bytes(n_tokens, r));
}

int sgmv_workspace_init(void* workspace, size_t workspace_bytes, void* stream) {
  if (workspace == nullptr) return SGMV_ERR_NULL;
  if (!aligned(workspace, 256)) return SGMV_ERR_ALIGN;
  if (workspace_bytes < kWorkspaceHeader) return SGMV_ERR_WORKSPACE;
  if (launch_workspace_init(workspace, workspace_bytes, 0, static_cast<hipStream_t>(stream)) !=
      hipSuccess)
    return SGMV_ERR_LAUNCH;
  return SGMV_OK;
}

int sgmv_workspace_check(const void* workspace, void* stream) {
  if (workspace == nullptr) return SGMV_ERR_NULL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the generation copies and, right after them, the error word and the initialisation mark
  static_assert(kWorkspaceErrorOffset == (size_t)kGenerationCopies * 4, "error word follows the copies");
  uint32_t head[kGenerationCopies + 2];
  if (hipMemcpyAsync(head, workspace, sizeof head, hipMemcpyDeviceToHost, st) != hipSuccess)
    return SGMV_ERR_LAUNCH;
  if (hipStreamSynchronize(st) != hipSuccess) return SGMV_ERR_LAUNCH;
  // between launches all copies of the generation agree; anything else means the workspace was
  // never initialised, or a launch did not account for all of its workgroups and later launches
  // may disagree about their generation
  if (head[kGenerationCopies + 1] != kWorkspaceMagic) return SGMV_ERR_STATE;
  if (head[kGenerationCopies] != 0) return SGMV_ERR_TIMEOUT;
  if (head[0] == 0) return SGMV_ERR_STATE;
  for (int i = 1; i < kGenerationCopies; ++i)
    if (head[i] != head[0]) return SGMV_ERR_STATE;
  return SGMV_OK;
}

int sgmv_validate_segments(const int32_t* host_seg_starts, int32_t n_segs, int32_t n_tokens) {
  if (n_segs < 0 || n_tokens < 0) return SGMV_ERR_SHAPE;
  if (host_seg_starts == nullptr) return SGMV_ERR_NULL;
  if (host_seg_starts[0] != 0) return SGMV_ERR_SHAPE;
  for (int32_t i = 0; i < n_segs; ++i)
    if (host_seg_starts[i + 1] < host_seg_starts[i]) return SGMV_ERR_SHAPE;
  if (host_seg_starts[n_segs] != n_tokens) return SGMV_ERR_SHAPE;
  return SGMV_OK;
}

int sgmv_shrink(const sgmv_problem* p, float* v, const void* x, const void* const* A_ptrs,
                const int32_t* seg_starts, int32_t n_segs, int32_t layer_idx, void* stream) {
  int rc = check_common(p, seg_starts, n_segs, layer_idx, true, false);
  if (rc != SGMV_OK) return rc;
  if (n_segs == 0 || p->n_tokens == 0) return SGMV_OK;
  if (v == nullptr || x == nullptr || A_ptrs == nullptr) return SGMV_ERR_NULL;
  if (!aligned(v, 16) || !aligned(x, 16)) return SGMV_ERR_ALIGN;
  rc = check_workspace(p);
  if (rc != SGMV_OK) return rc;
  if (p->path == SGMV_PATH_FUSED || p->path == SGMV_PATH_ROWS) return SGMV_ERR_UNSUPPORTED;

  hipStream_t st = static_cast<hipStream_t>(stream);
  ShrinkPlan pl;
  rc = plan_shrink(p, n_segs, &pl);
  if (rc != SGMV_OK) return rc;
  if (pl.kernel == SGMV_KERNEL_WHOLE) {
    ShrinkArgs a = make_shrink(p, Scratch{}, x, A_ptrs, seg_starts, n_segs, layer_idx);
    a.by_rows = pl.whole_by_rows;
    return launch_shrink_whole(a, v, st) == hipSuccess ? SGMV_OK : SGMV_ERR_LAUNCH;
  }
  if (pl.kernel == SGMV_KERNEL_FUSED) {
    fill_fused(&pl.fused, p, caller_scratch(p), seg_starts, n_segs, layer_idx, 1.f);
    pl.fused.x = x;
    pl.fused.A_ptrs = A_ptrs;
    return launch_shrink_handoff(pl.fused, v, st) == hipSuccess ? SGMV_OK : SGMV_ERR_LAUNCH;
  }
  ShrinkArgs a = make_shrink(p, caller_scratch(p), x, A_ptrs, seg_starts, n_segs, layer_idx);
  a.ksplit = pl.ksplit;
  a.kslice = pl.kslice;
  if (pl.kernel == SGMV_KERNEL_MATRIX) {
    if (launch_shrink_matrix(a, st) != hipSuccess) return SGMV_ERR_LAUNCH;
  } else {
    if (launch_shrink_vector(a, st) != hipSuccess) return SGMV_ERR_LAUNCH;
  }
  if (launch_shrink_reduce(v, a, st) != hipSuccess) return SGMV_ERR_LAUNCH;
  return SGMV_OK;
}

int sgmv_expand(const sgmv_problem* p, void* y, const float* v, const void* const* B_ptrs,
                const int32_t* seg_starts, int32_t n_segs, int32_t layer_idx, float scale,
                void* stream) {
  int rc = check_common(p, seg_starts, n_segs, layer_idx, false, true);
  if (rc != SGMV_OK) return rc;
  if (n_segs == 0 || p->n_tokens == 0) return SGMV_OK;
  if (y == nullptr || v == nullptr || B_ptrs == nullptr) return SGMV_ERR_NULL;
  if (!aligned(v, 16) || !aligned(y, 16)) return SGMV_ERR_ALIGN;
  if (p->path == SGMV_PATH_FUSED || p->path == SGMV_PATH_WHOLE || p->path == SGMV_PATH_ROWS) return SGMV_ERR_UNSUPPORTED;

  hipStream_t st = static_cast<hipStream_t>(stream);
  ExpandArgs a = make_expand(p, y, v, 1, nullptr, B_ptrs, seg_starts, n_segs, layer_idx, scale);
  // the MFMA kernels keep v's 16-bit operand pairs in the workspace
  const bool have_ws = check_workspace(p) == SGMV_OK;
  if (p->path == SGMV_PATH_MATRIX && !have_ws) return check_workspace(p);
  const int strips_threads = expand_by_rows(p, n_segs) ? choose_expand_threads(p, p->n_tokens) : 0;
  if (strips_threads != 0) {
    a.by_rows = true;
    a.threads = strips_threads;
    if (launch_expand_vector(a, st) != hipSuccess) return SGMV_ERR_LAUNCH;
  } else if (have_ws && expand_use_matrix(p, n_segs)) {
    set_operands(&a, caller_scratch(p), p->n_tokens, p->r);
    if (launch_expand_matrix(&a, 1, false, st) != hipSuccess) return SGMV_ERR_LAUNCH;
  } else {
    if (launch_expand_vector(a, st) != hipSuccess) return SGMV_ERR_LAUNCH;
  }
  return SGMV_OK;
}

}  // extern "C"

namespace {

// Argument checks of the whole add-on that do not concern the scratch memory.
int check_add_lora(const sgmv_problem* p, const void* y, const void* x, const void* const* A_ptrs,
                   const void* const* B_ptrs, const int32_t* seg_starts, int32_t n_segs,
                   int32_t layer_idx, bool* nothing_to_do) {
  *nothing_to_do = false;
  const int rc = check_common(p, seg_starts, n_segs, layer_idx, true, true);
  if (rc != SGMV_OK) return rc;
  if (n_segs == 0 || p->n_tokens == 0) {
    *nothing_to_do = true;
    return SGMV_OK;
  }
  if (y == nullptr || x == nullptr || A_ptrs == nullptr || B_ptrs == nullptr) return SGMV_ERR_NULL;
  if (!aligned(y, 16) || !aligned(x, 16)) return SGMV_ERR_ALIGN;
  return SGMV_OK;
}

// The add-on on checked arguments, its intermediate results in `sc`.
int add_lora_launch(const sgmv_problem* p, const Scratch& sc, void* y, const void* x,
                    const void* const* A_ptrs, const void* const* B_ptrs,
                    const int32_t* seg_starts, int32_t n_segs, int32_t layer_idx, float scale,
                    hipStream_t st) {
  SinglePlan pl;
  const int rc = plan_single(p, n_segs, &pl);
  if (rc != SGMV_OK) return rc;
  switch (pl.kernel) {
    case SGMV_KERNEL_WHOLE: {
      WholeArgs& w = pl.whole;
      w.bf16 = p->dtype == SGMV_BF16;
      w.r = p->r;
      w.h_in = p->h_in;
      w.h_out = p->h_out;
      w.n_segs = n_segs;
      w.n_tokens = p->n_tokens;
      w.offA = (long long)layer_idx * p->h_in * p->r;
      w.offB = (long long)layer_idx * p->r * p->h_out;
      w.scale = scale;
      w.y = y;
      w.x = x;
      w.A_ptrs = A_ptrs;
      w.B_ptrs = B_ptrs;
      w.seg_starts = seg_starts;
      w.header = sc.header;
      return launch_add_lora_whole(w, st) == hipSuccess ? SGMV_OK : SGMV_ERR_LAUNCH;
    }
    case SGMV_KERNEL_TILE: {
      TileArgs& t = pl.tile;
      fill_tile(&t, p, sc, seg_starts, n_segs, layer_idx, scale);
      t.y = y;
      t.x = x;
      t.A_ptrs = A_ptrs;
      t.B_ptrs = B_ptrs;
      return launch_add_lora_tile(t, st) == hipSuccess ? SGMV_OK : SGMV_ERR_LAUNCH;
    }
    case SGMV_KERNEL_FUSED: {
      FusedArgs& f = pl.fused;
      fill_fused(&f, p, sc, seg_starts, n_segs, layer_idx, scale);
      f.y = y;
      f.x = x;
      f.A_ptrs = A_ptrs;
      f.B_ptrs = B_ptrs;
      return launch_add_lora_fused(f, st) == hipSuccess ? SGMV_OK : SGMV_ERR_LAUNCH;
    }
    case SGMV_KERNEL_MATRIX: {
      ShrinkArgs sa = make_shrink(p, sc, x, A_ptrs, seg_starts, n_segs, layer_idx);
      sa.ksplit = pl.ksplit;
      sa.kslice = pl.kslice;
      if (launch_shrink_matrix(sa, st) != hipSuccess) return SGMV_ERR_LAUNCH;
      ExpandArgs e = make_expand(p, y, sa.partials, sa.ksplit, A_ptrs, B_ptrs, seg_starts, n_segs,
                                 layer_idx, scale);
      set_operands(&e, sc, p->n_tokens, p->r);
      return launch_expand_matrix(&e, 1, pl.direct, st) == hipSuccess ? SGMV_OK : SGMV_ERR_LAUNCH;
    }
    default: {
      ShrinkArgs sa = make_shrink(p, sc, x, A_ptrs, seg_starts, n_segs, layer_idx);
      sa.ksplit = pl.ksplit;
      sa.kslice = pl.kslice;
      if (launch_shrink_vector(sa, st) != hipSuccess) return SGMV_ERR_LAUNCH;
      ExpandArgs e = make_expand(p, y, sa.partials, sa.ksplit, A_ptrs, B_ptrs, seg_starts, n_segs,
                                 layer_idx, scale);
      return launch_expand_vector(e, st) == hipSuccess ? SGMV_OK : SGMV_ERR_LAUNCH;
    }
  }
}

// The device address of this GPU's copy of `scratch`, prepared for the single-launch kernels
// the first time the GPU is seen: asked of the runtime once per device (every GPU holds its
// own copy at its own address), then header and exchange words are cleared and the generation set
// by a small kernel on `st`.  Calls no allocator.
int static_scratch(hipStream_t st, char** base) {
  static std::mutex mutex;
  static char* address[kMaxDevices];  // zero-initialised
  static bool ready[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return SGMV_ERR_LAUNCH;
  if (dev < 0 || dev >= kMaxDevices) return SGMV_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(mutex);
  if (address[dev] == nullptr) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return SGMV_ERR_LAUNCH;
    address[dev] = static_cast<char*>(ptr);
  }
  if (!ready[dev]) {
    // the clearing kernel must run once, not once per replay of a graph that captured it
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
      (void)hipGetLastError();
      return SGMV_ERR_STATE;
    }
    if (launch_workspace_init(address[dev], kStaticExchangeEnd, 0, st) != hipSuccess) return SGMV_ERR_LAUNCH;
    ready[dev] = true;
  }
  *base = address[dev];
  return SGMV_OK;
}

}  // namespace

extern "C" {

int sgmv_add_lora(const sgmv_problem* p, void* y, const void* x, const void* const* A_ptrs,
                  const void* const* B_ptrs, const int32_t* seg_starts, int32_t n_segs,
                  int32_t layer_idx, float scale, void* stream) {
  bool nothing = false;
  int rc = check_add_lora(p, y, x, A_ptrs, B_ptrs, seg_starts, n_segs, layer_idx, &nothing);
  if (rc != SGMV_OK || nothing) return rc;
  if (p->path == SGMV_PATH_WHOLE && p->workspace == nullptr)  // that kernel keeps nothing in memory
    return add_lora_launch(p, Scratch{nullptr, nullptr, nullptr, nullptr}, y, x, A_ptrs, B_ptrs, seg_starts,
                           n_segs, layer_idx, scale, static_cast<hipStream_t>(stream));
  rc = check_workspace(p);
  if (rc != SGMV_OK) return rc;
  return add_lora_launch(p, caller_scratch(p), y, x, A_ptrs, B_ptrs, seg_starts, n_segs, layer_idx,
                         scale, static_cast<hipStream_t>(stream));
}

int sgmv_add_lora_static(const sgmv_problem* p, void* y, const void* x, const void* const* A_ptrs,
                         const void* const* B_ptrs, const int32_t* seg_starts, int32_t n_segs,
                         int32_t layer_idx, float scale, void* stream) {
  bool nothing = false;
  int rc = check_add_lora(p, y, x, A_ptrs, B_ptrs, seg_starts, n_segs, layer_idx, &nothing);
  if (rc != SGMV_OK || nothing) return rc;
  if (sgmv_workspace_bytes(p->n_tokens, p->r) > SGMV_STATIC_MAX_WORKSPACE_BYTES) return SGMV_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* base = nullptr;
  rc = static_scratch(st, &base);
  if (rc != SGMV_OK) return rc;
  // within the size limit both regions of the array hold what this batch needs (exchange
  // words: twice the partial sums' bytes); checked all the same
  const size_t parts = partial_bytes(p->n_tokens, p->r);
  if (2 * parts > kStaticExchangeEnd - kWorkspaceHeader ||
      parts + operand_bytes(p->n_tokens, p->r) > kStaticBytes - kStaticExchangeEnd)
    return SGMV_ERR_WORKSPACE;
  sgmv_problem q = *p;
  q.workspace = base;
  q.workspace_bytes = kStaticBytes;
  q.workspace_ready = 1;
  const Scratch sc{reinterpret_cast<unsigned long long*>(base),
                   reinterpret_cast<float*>(base + kStaticExchangeEnd),
                   reinterpret_cast<unsigned long long*>(base + kWorkspaceHeader),
                   base + kStaticExchangeEnd + parts};
  return add_lora_launch(&q, sc, y, x, A_ptrs, B_ptrs, seg_starts, n_segs, layer_idx, scale, st);
}

int sgmv_add_lora_multi(const sgmv_problem* p, int32_t n_proj, void* const* ys,
                        const void* const* xs, const void* const* const* A_ptrs,
                        const void* const* const* B_ptrs, const int32_t* seg_starts, int32_t n_segs,
                        int32_t layer_idx, float scale, void* stream) {
  int rc = check_common(p, seg_starts, n_segs, layer_idx, true, true);
  if (rc != SGMV_OK) return rc;
  if (n_proj < 0 || n_proj > kMaxProjections) return SGMV_ERR_SHAPE;
  if (n_proj == 0 || n_segs == 0 || p->n_tokens == 0) return SGMV_OK;
  if (ys == nullptr || xs == nullptr || A_ptrs == nullptr || B_ptrs == nullptr) return SGMV_ERR_NULL;
  for (int i = 0; i < n_proj; ++i) {
    if (ys[i] == nullptr || xs[i] == nullptr || A_ptrs[i] == nullptr || B_ptrs[i] == nullptr)
      return SGMV_ERR_NULL;
    if (!aligned(ys[i], 16) || !aligned(xs[i], 16)) return SGMV_ERR_ALIGN;
    for (int j = 0; j < i; ++j)
      if (ys[i] == ys[j]) return SGMV_ERR_SHAPE;  // two add-ons into one y would race
  }
  rc = check_workspace(p);
  if (rc != SGMV_OK) return rc;

  hipStream_t st = static_cast<hipStream_t>(stream);
  FusedArgs f;
  TileArgs tile;
  int kernel = plan_multi(p, n_segs, n_proj, &f, &tile);
  const bool joint_matrix = multi_takes_matrix(p, n_segs, n_proj, kernel, tile);
  if (joint_matrix) kernel = SGMV_KERNEL_SEQUENCE;
  if (kernel == SGMV_KERNEL_TILE) {
    const Scratch sc = caller_scratch(p);
    const int group = tile.n_proj;
    for (int first = 0; first < n_proj; first += group) {
      const int count = n_proj - first < group ? n_proj - first : group;
      TileArgs t = tile;
      if (count == 1 || (count < group && !choose_tile(p, n_segs, &t, count))) {  // left over at the end
        for (int i = first; i < first + count; ++i) {
          rc = add_lora_launch(p, sc, ys[i], xs[i], A_ptrs[i], B_ptrs[i], seg_starts, n_segs, layer_idx, scale, st);
          if (rc != SGMV_OK) return rc;
        }
        break;
      }
      fill_tile(&t, p, sc, seg_starts, n_segs, layer_idx, scale);
      for (int i = 0; i < kMaxProjections; ++i) {
        t.table.x[i] = i < count ? xs[first + i] : nullptr;
        t.table.y[i] = i < count ? ys[first + i] : nullptr;
        t.table.A_ptrs[i] = i < count ? A_ptrs[first + i] : nullptr;
        t.table.B_ptrs[i] = i < count ? B_ptrs[first + i] : nullptr;
      }
      if (launch_add_lora_tile(t, st) != hipSuccess) return SGMV_ERR_LAUNCH;
    }
    return SGMV_OK;
  }
  if (kernel != SGMV_KERNEL_SEQUENCE) {
    fill_fused(&f, p, caller_scratch(p), seg_starts, n_segs, layer_idx, scale);
    f.n_proj = n_proj;
    for (int i = 0; i < kMaxProjections; ++i) {
      f.table.x[i] = i < n_proj ? xs[i] : nullptr;
      f.table.y[i] = i < n_proj ? ys[i] : nullptr;
      f.table.A_ptrs[i] = i < n_proj ? A_ptrs[i] : nullptr;
      f.table.B_ptrs[i] = i < n_proj ? B_ptrs[i] : nullptr;
    }
    // side by side while every workgroup of the launch is resident (two fit a compute
    // unit); beyond that one workgroup per (slice, segment) walks the projections in
    // turn, the next one's loads in flight
    f.Z = 1;
    const hipError_t err = kernel == SGMV_KERNEL_MULTI_SIDE ? launch_add_lora_fused(f, st)
                                                            : launch_add_lora_fused_multi(f, st);
    return err == hipSuccess ? SGMV_OK : SGMV_ERR_LAUNCH;
  }
  // Long segments on the MFMA kernels: up to three add-ons per launch of each kernel (one pass over x
  // where they read the same one).  Needs the larger workspace of sgmv_workspace_bytes_multi for the
  // partial sums and operands of the second and third add-on.
  // (Where a single add-on would take two rows to an item of the hand-off kernel, these launches together are ahead: two of
  // 250 rows of 37 adapters, 8192 wide, rank 16, 20.2 us against 35.9; three of 120 rows of 22, 13824 wide, rank 32, 37.7 / 66.1.)
  SinglePlan pl;
  if (n_proj >= 2 && (joint_matrix || (plan_single(p, n_segs, &pl, false) == SGMV_OK && pl.kernel == SGMV_KERNEL_MATRIX)) &&
      p->workspace_bytes >= sgmv_workspace_bytes_multi(p->n_tokens, p->r, n_proj)) {
    const Scratch sc = caller_scratch(p);
    // the first add-on's partial sums and operands where a single call keeps them, the others' behind the
    // single-call workspace (the exchange words in between are left alone: the single-launch kernels
    // rely on what their tags say)
    const size_t parts = partial_bytes(p->n_tokens, p->r), ops = operand_bytes(p->n_tokens, p->r);
    char* const extra = static_cast<char*>(p->workspace) + sgmv_workspace_bytes(p->n_tokens, p->r);
    for (int first = 0; first < n_proj; first += kSharedShrinkMost) {
      const int count = n_proj - first < kSharedShrinkMost ? n_proj - first : kSharedShrinkMost;
      ShrinkArgs sa = make_shrink(p, sc, xs[first], A_ptrs[first], seg_starts, n_segs, layer_idx);
      sa.n_proj = count;
      sa.same_x = true;
      for (int i = 0; i < count; ++i) {
        sa.same_x = sa.same_x && xs[first + i] == xs[first];
        sa.xs[i] = xs[first + i];
        sa.As[i] = A_ptrs[first + i];
        if (i > 0) sa.partials_of[i] = reinterpret_cast<float*>(extra + (size_t)(i - 1) * (parts + ops));
      }
      MatrixSplit m = choose_split_matrix(p, n_segs, count, sa.same_x);
      // two launches or three as sgmv_plan_add_lora tells, which does not see the inputs (slices of inputs of their own are fewer: what
      // the expand adds up of one x it can add up of several)
      if (!sa.same_x) m.direct = choose_split_matrix(p, n_segs, count, true).direct;
      sa.ksplit = m.ksplit;
      sa.kslice = m.kslice;
      if (launch_shrink_matrix(sa, st) != hipSuccess) return SGMV_ERR_LAUNCH;
      ExpandArgs es[kSharedShrinkMost];
      for (int i = 0; i < count; ++i) {
        es[i] = make_expand(p, ys[first + i], sa.partials_of[i], sa.ksplit, A_ptrs[first + i], B_ptrs[first + i], seg_starts,
                            n_segs, layer_idx, scale);
        Scratch own = sc;
        if (i > 0) own.operands = extra + (size_t)(i - 1) * (parts + ops) + parts;
        set_operands(&es[i], own, p->n_tokens, p->r);
        es[i].three_parts = joint_matrix;
      }
      if (launch_expand_matrix(es, count, m.direct, st) != hipSuccess) return SGMV_ERR_LAUNCH;
    }
    return SGMV_OK;
  }
  // any other shape: one add-on after the other
  for (int i = 0; i < n_proj; ++i) {
    rc = sgmv_add_lora(p, ys[i], xs[i], A_ptrs[i], B_ptrs[i], seg_starts, n_segs, layer_idx, scale,
                       stream);
    if (rc != SGMV_OK) return rc;
  }
  return SGMV_OK;
}

int sgmv_plan_shrink(const sgmv_problem* p, int32_t n_segs, sgmv_plan* plan) {
  if (plan == nullptr) return SGMV_ERR_NULL;
  *plan = sgmv_plan{};
  static const int32_t no_segments[2] = {0, 0};  // only tested for being non-NULL
  int rc = check_common(p, no_segments, n_segs, 0, true, false);
  if (rc != SGMV_OK) return rc;
  if (n_segs == 0 || p->n_tokens == 0) return SGMV_OK;  // nothing is launched
  rc = check_workspace(p);
  if (rc != SGMV_OK) return rc;
  if (p->path == SGMV_PATH_FUSED || p->path == SGMV_PATH_ROWS) return SGMV_ERR_UNSUPPORTED;
  ShrinkPlan pl;
  rc = plan_shrink(p, n_segs, &pl);
  if (rc != SGMV_OK) return rc;
  plan->kernel = pl.kernel;
  if (pl.kernel == SGMV_KERNEL_WHOLE) {
    plan->launches = 1;
    plan->slices = 1;
    plan->workgroups = pl.whole_by_rows ? ceil_div(p->n_tokens, 8) * 8 : n_segs;
  } else if (pl.kernel == SGMV_KERNEL_FUSED) {
    plan->launches = 1;
    plan->slices = pl.fused.S;
    plan->workgroups = pl.fused.S * (int)fused_grid_items(pl.fused.items);
  } else {
    plan->launches = 2;
    plan->slices = pl.ksplit;
  }
  return SGMV_OK;
}

int sgmv_plan_expand(const sgmv_problem* p, int32_t n_segs, sgmv_plan* plan) {
  if (plan == nullptr) return SGMV_ERR_NULL;
  *plan = sgmv_plan{};
  static const int32_t no_segments[2] = {0, 0};  // only tested for being non-NULL
  const int rc = check_common(p, no_segments, n_segs, 0, false, true);
  if (rc != SGMV_OK) return rc;
  if (n_segs == 0 || p->n_tokens == 0) return SGMV_OK;  // nothing is launched
  if (p->path == SGMV_PATH_FUSED || p->path == SGMV_PATH_WHOLE || p->path == SGMV_PATH_ROWS) return SGMV_ERR_UNSUPPORTED;
  const bool have_ws = check_workspace(p) == SGMV_OK;
  if (p->path == SGMV_PATH_MATRIX && !have_ws) return check_workspace(p);
  if (!expand_by_rows(p, n_segs) && have_ws && expand_use_matrix(p, n_segs)) {
    plan->kernel = SGMV_KERNEL_MATRIX;
    plan->launches = 2;  // operand preparation, expand
    return SGMV_OK;
  }
  const bool by_rows = expand_by_rows(p, n_segs);
  const int threads = choose_expand_threads(p, by_rows ? p->n_tokens : n_segs);
  plan->kernel = SGMV_KERNEL_VECTOR;
  plan->launches = 1;
  plan->slices = ceil_div(p->h_out, threads == kExpandSplit ? 512 : threads * 8);  // column strips
  // v of the rows of a pass, and in the kernel whose waves divide the weight rows the partial sums of three waves
  const int rows_per_pass = by_rows ? 1 : 4;
  plan->lds_bytes = rows_per_pass * p->r * 4 + (threads == kExpandSplit ? 3 * rows_per_pass * 512 * 4 : 0);
  plan->workgroups = plan->slices * (by_rows ? ceil_div(p->n_tokens, 8) * 8 : n_segs);
  return SGMV_OK;
}

int sgmv_plan_add_lora(const sgmv_problem* p, int32_t n_segs, int32_t n_proj, sgmv_plan* plan) {
  if (plan == nullptr) return SGMV_ERR_NULL;
  *plan = sgmv_plan{};
  static const int32_t no_segments[2] = {0, 0};  // only tested for being non-NULL
  int rc = check_common(p, no_segments, n_segs, 0, true, true);
  if (rc != SGMV_OK) return rc;
  if (n_proj < 1 || n_proj > kMaxProjections) return SGMV_ERR_SHAPE;
  if (n_segs == 0 || p->n_tokens == 0) return SGMV_OK;  // nothing is launched
  if (!(p->path == SGMV_PATH_WHOLE && p->workspace == nullptr && n_proj == 1)) {
    rc = check_workspace(p);
    if (rc != SGMV_OK) return rc;
  }
  bool joint_matrix = false;
  if (n_proj > 1) {
    FusedArgs f;
    TileArgs tile;
    int kernel = plan_multi(p, n_segs, n_proj, &f, &tile);
    joint_matrix = multi_takes_matrix(p, n_segs, n_proj, kernel, tile);
    if (joint_matrix) kernel = SGMV_KERNEL_SEQUENCE;
    if (kernel == SGMV_KERNEL_TILE) {  // groups of tile.n_proj add-ons; slices and workgroups of the first launch
      plan->kernel = kernel;
      plan->launches = (n_proj + tile.n_proj - 1) / tile.n_proj;
      plan->slices = tile.S;
      plan->workgroups = tile.S * n_segs * tile.n_proj * tile.Z;
      plan->lds_bytes = (int32_t)tile.lds_bytes;
      return SGMV_OK;
    }
    if (kernel != SGMV_KERNEL_SEQUENCE) {
      plan->kernel = kernel;
      plan->launches = 1;
      plan->slices = f.S;
      plan->workgroups = f.S * (int)fused_grid_items(f.items) * (kernel == SGMV_KERNEL_MULTI_SIDE ? n_proj : 1);
      return SGMV_OK;
    }
  }
  SinglePlan pl;
  rc = plan_single(p, n_segs, &pl, n_proj < 2);
  if (rc == SGMV_OK && n_proj >= 2 &&
      (pl.kernel != SGMV_KERNEL_MATRIX || p->workspace_bytes < sgmv_workspace_bytes_multi(p->n_tokens, p->r, n_proj)))
    rc = plan_single(p, n_segs, &pl);  // one after the other
  if (joint_matrix) {
    rc = SGMV_OK;
    pl.kernel = SGMV_KERNEL_MATRIX;
    pl.direct = false;
  }
  if (rc != SGMV_OK) return rc;
  plan->kernel = pl.kernel;
  switch (pl.kernel) {
    case SGMV_KERNEL_WHOLE:
      plan->launches = 1;
      plan->slices = pl.whole.S;
      plan->workgroups = 8 * pl.whole.S * ceil_div(pl.whole.by_rows ? p->n_tokens : n_segs, 8);
      plan->lds_bytes = 0;
      break;
    case SGMV_KERNEL_TILE:
      plan->launches = 1;
      plan->slices = pl.tile.S;
      plan->workgroups = pl.tile.S * n_segs * pl.tile.Z;
      plan->lds_bytes = (int32_t)pl.tile.lds_bytes;
      break;
    case SGMV_KERNEL_FUSED:
      plan->launches = 1;
      plan->slices = pl.fused.S;
      plan->workgroups = pl.fused.S * (int)fused_grid_items(pl.fused.items);
      break;
    case SGMV_KERNEL_MATRIX:
      plan->launches = pl.direct ? 2 : 3;  // shrink, operand preparation, expand
      plan->slices = pl.ksplit;
      break;
    default:
      plan->launches = 2;
      plan->slices = pl.ksplit;
      plan->workgroups = pl.ksplit * n_segs;
      break;
  }
  if (pl.kernel == SGMV_KERNEL_MATRIX && n_proj > 1 &&
      p->workspace_bytes >= sgmv_workspace_bytes_multi(p->n_tokens, p->r, n_proj)) {
    // as for add-ons on one x, which a caller of several projections usually has
    plan->launches = 0;
    for (int first = 0; first < n_proj; first += kSharedShrinkMost) {
      const MatrixSplit m = choose_split_matrix(p, n_segs, n_proj - first < kSharedShrinkMost ? n_proj - first : kSharedShrinkMost, true);
      plan->launches += m.direct ? 2 : 3;
      if (first == 0) plan->slices = m.ksplit;
    }
  } else
    plan->launches *= n_proj;  // a multi-projection call that is not batched runs them in turn
  return SGMV_OK;
}

}  // extern "C"
