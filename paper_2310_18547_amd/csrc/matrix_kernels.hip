// MFMA path of SGMV for long (prefill-shaped) segments, gfx950.
//
// When a segment holds hundreds of rows, the per-segment product really is a
// dense contraction -- the reason the paper gives for grouping the requests of
// one adapter (section "Segmented Gather Matrix-Vector Multiplication", kernel
// schedule paragraph: higher operational intensity, matrix units) -- and at
// ranks up to 64 the vector ALUs can no longer keep up with HBM: the shrink
// needs r FLOP per byte of x and the expand r/2 FLOP per byte of y.  All
// kernels here are still bound by HBM (x is read once, y is read and written
// once); the matrix cores only have to be fast enough not to matter, so the
// code is organised around how x and y stream, not around MFMA utilisation.
//
// The kernels use v_mfma_f32_16x16x32_{f16,bf16}.  Its operands want eight
// consecutive k per lane: lane l of a wave holds row (l % 16), k = 8 (l / 16) ..
// +7 of the first operand and column (l % 16), same k, of the second; it
// receives D[4 (l / 16) + i][l % 16], i = 0..3.  x and v are k-contiguous in
// memory, the weights A_i [h_in][r] and B_i [r][h_out] are not, so weight tiles
// are transposed once per workgroup through LDS (pairs of k packed into a dword
// on the way in, so the LDS writes are conflict-free dword writes) and are then
// reused for every row tile of the workgroup.
//
//   shrink_stream_kernel   workgroup = (k-slice, block of rows, group of add-ons that read the same x);
//           Split-K partial sums.
//   finalize_v_kernel      sums the partial sums in ascending order and writes v as a high and a
//           low 16-bit part (16 significant bits for bfloat16, 22 for binary16) plus a range
//           factor per row (binary16).  v stays fp32 in the workspace until then.
//   expand_matrix_kernel   workgroup = (strip of columns, block of rows or short segment, add-on).
//
// Up to three add-ons of a call go into one launch of each kernel.  4814 rows of eight segments, bfloat16: 8192 ->
// 8192 at rank 16 61.4 -> 53.3 us, 8192 -> 28672 at rank 64 167 -> 144; three projections of 4096 -> 4096, 41 decode
// rows beside three prompts of 1152 rows, rank 16: 69.5 -> 33.1; of 3272 -> 4096, 3254 rows, rank 64: 119 -> 62.8.
#include <type_traits>

#include "device_common.h"
#include "launch.h"
#include "mfma.h"
#include "trace.h"


namespace sgmv {

constexpr int kExpandCols = 256;   // columns of a block item of the expand
constexpr int kExpandRows = 64;    // its rows

// ---------------------------------------------------------------- row blocks
//
// The work of a launch is the list of row blocks of all segments: segment 0's blocks of ROWS rows,
// then segment 1's, and so on.  A workgroup is handed an index into that list and finds its block
// itself, so the grid has no more workgroups than there can be blocks (n_tokens / ROWS + n_segs,
// those that find none leave at once) whatever the lengths are -- a grid of (longest
// segment) x (segments) is mostly empty when a few prompts run beside the decode rows of everybody
// else (44 segments, 3 of them long: 352 blocks for 61).
//
// Up to kDenseSegments a wave looks at all of them in one round of loads (from 65 on, four per lane) and adds
// up the list, which has no gaps.  Beyond that segment i's part starts at block (seg_starts[i] + i (ROWS - 1)) / ROWS,
// which needs no sum over the segments before it and leaves room for its ceil(rows / ROWS) blocks: a
// workgroup looks among the 64 segments around the place that equal lengths would give, and if its own is not
// among them searches sixty-four ways, three rounds at most for 65535 segments.  (Adding the blocks up from segment 0
// took a round per 64 segments in front of every workgroup: 256 / 1024 / 4096 / 16384 segments of 8 rows, 4096 -> 4096 at
// rank 16, 34.7 / 149 / 1044 / 12376 us against 29.9 / 82.9 / 314 / 1232.  The search from 65 segments on: 3 prompts beside
// 125 one-row segments at rank 64 51.4 against 42.7 us, because workgroups that find nothing stand between the others,
// not behind them; 200 segments of 8 rows at rank 16 29.0 against 29.8.)
struct Found {
  int seg, lo, hi;   // segment and its rows; seg < 0: nothing at this place
  int index;         // place in the segment's part of the list
};
constexpr int kDensePerLane = 4, kDenseSegments = 64 * kDensePerLane;

// Inclusive prefix sum over the wave by data-parallel-primitive moves.
__device__ __forceinline__ int prefix_sum(int sum) {
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x111, 0xF, 0xF, false);  // row_shr 1
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x112, 0xF, 0xF, false);  // row_shr 2
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x114, 0xF, 0xF, false);  // row_shr 4
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x118, 0xF, 0xF, false);  // row_shr 8
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x142, 0xA, 0xF, false);  // row_bcast 15 into rows 1 and 3
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x143, 0xC, 0xF, false);  // row_bcast 31 into rows 2 and 3
  return sum;
}

// Called by whole waves.  A segment of that many rows (at least one) has count(rows) items, per_block for each of its
// blocks or, if it has a single one, fewer.  item: the place in the list, or beyond kDenseSegments, place `item
// % per_block` of block `item / per_block`.  turn: the items of a segment that has fewer.  guess: segments per block on average.
template <int ROWS, class Count>
__device__ __forceinline__ Found find_item(const int32_t* __restrict__ seg_starts, int n_segs, unsigned item, int per_block,
                                           int turn, float guess, int lane, Count count) {
  int base = 0;
  int lo, hi;
  auto look = [&]() {  // lane l: segment base + l
    const int i = min(base + lane, n_segs - 1);
    lo = seg_starts[i];
    hi = seg_starts[i + 1];
  };
  auto take = [&](int at) {
    lo = __builtin_amdgcn_readlane(lo, at);
    hi = __builtin_amdgcn_readlane(hi, at);
  };
  // told to be wave-uniform, what is derived from these stays in scalar registers
  auto found = [&](int seg, int index) {
    return Found{__builtin_amdgcn_readfirstlane(seg), __builtin_amdgcn_readfirstlane(lo), __builtin_amdgcn_readfirstlane(hi),
                 __builtin_amdgcn_readfirstlane(index)};
  };
  if (n_segs <= 64) {
    look();
    const int items = lane < n_segs && hi > lo ? count(hi - lo) : 0, sum = prefix_sum(items);
    const int index = (int)item;
    if (index >= __builtin_amdgcn_readlane(sum, 63)) return Found{-1, 0, 0, 0};
    const int at = __builtin_ctzll(__ballot(sum > index));
    take(at);
    return found(at, index - __builtin_amdgcn_readlane(sum, at) + __builtin_amdgcn_readlane(items, at));
  }
  if (n_segs <= kDenseSegments) {  // lane l: segments 4 l .. 4 l + 3, those past the end empty
    int start[kDensePerLane + 1], items[kDensePerLane], mine_all = 0;
#pragma unroll
    for (int k = 0; k <= kDensePerLane; ++k) start[k] = seg_starts[min(kDensePerLane * lane + k, n_segs)];
#pragma unroll
    for (int k = 0; k < kDensePerLane; ++k) {
      items[k] = start[k + 1] > start[k] ? count(start[k + 1] - start[k]) : 0;
      mine_all += items[k];
    }
    const int sum = prefix_sum(mine_all);
    int index = (int)item;
    if (index >= __builtin_amdgcn_readlane(sum, 63)) return Found{-1, 0, 0, 0};
    const int at = __builtin_ctzll(__ballot(sum > index));
    index -= __builtin_amdgcn_readlane(sum, at) - __builtin_amdgcn_readlane(mine_all, at);
    int seg = kDensePerLane * at;
    lo = __builtin_amdgcn_readlane(start[0], at);
    hi = __builtin_amdgcn_readlane(start[1], at);
    int before = __builtin_amdgcn_readlane(items[0], at);  // items of the lane's segments up to `seg`
#pragma unroll
    for (int k = 1; k < kDensePerLane; ++k) {
      const int more = __builtin_amdgcn_readlane(items[k], at);
      const int next = __builtin_amdgcn_readlane(start[k + 1], at);
      if (index >= before) {
        index -= before;
        before = more;
        seg = kDensePerLane * at + k;
        lo = hi;
        hi = next;
      }
    }
    return found(seg, index);
  }
  // first block of segment i (n_tokens + 65535 * 127 fits 32 bits)
  auto first_of = [](int start, int i) { return ((unsigned)start + (unsigned)i * (ROWS - 1)) / ROWS; };
  const unsigned block = item / (unsigned)per_block;
  // the last segment whose part starts at or before the block
  base = min(max((int)((float)block * guess) - 32, 0), n_segs - 64);
  look();
  int at = __popcll(__ballot(first_of(lo, base + lane) <= block)) - 1;
  if (at < 0 || (at == 63 && base + 64 < n_segs && first_of(__builtin_amdgcn_readlane(hi, 63), base + 64) <= block)) {
    int from = at < 0 ? 0 : base + 64, to = at < 0 ? base : n_segs;  // among these, and `from` starts at or before
    while (to - from > 64) {
      const int step = (to - from + 63) / 64, i = from + lane * step;
      const bool before = i < to && first_of(seg_starts[min(i, n_segs)], i) <= block;
      from += (__popcll(__ballot(before)) - 1) * step;
      to = min(to, from + step);
    }
    base = from;
    look();
    at = __popcll(__ballot(base + lane < to && first_of(lo, base + lane) <= block)) - 1;
  }
  take(at);
  // a segment with fewer items than places takes other places in every block: workgroup ids go round the eight
  // XCDs, so that always the first places of a multiple of eight would be always the same XCDs
  int part = (int)(item - block * (unsigned)per_block) + (int)(block * (unsigned)turn % (unsigned)per_block);
  if (part >= per_block) part -= per_block;
  const int index = (int)(block - first_of(lo, base + at)) * per_block + part;
  return found(hi > lo && index < count(hi - lo) ? base + at : -1, index);
}
// Length of the list at most; `guess` for find_item.
static long long most_blocks(int n_tokens, int n_segs, int rows) {
  const long long b = ((long long)n_tokens + (long long)n_segs * (rows - 1)) / rows;
  return n_segs <= kDenseSegments && b > n_tokens ? n_tokens : b;
}
static float segments_per_block(int n_segs, long long blocks) { return (float)n_segs / (float)blocks; }

// Binary16 has a narrow range, so a row of v whose largest |v|, amax, reaches 2^14 is scaled down by an exact power of
// two, the result, and `undo` restores the fp32 result (both 1 otherwise).  As three parts (BOTH) a smaller row is scaled up
// likewise, so that its parts keep all bits.
template <bool BOTH = false>
__device__ __forceinline__ float range_factor(float amax, float& undo) {
  const int above = (int)((__float_as_uint(amax) >> 23) & 0xFF) - 127 - 13;  // amax * 2^-above is in 2^13 .. 2^14
  const int e = amax >= 3.0e38f ? 0 : amax >= 16384.f ? above : BOTH ? max(above, -100) : 0;
  undo = __uint_as_float((uint32_t)(127 + e) << 23);
  return __uint_as_float((uint32_t)(127 - e) << 23);
}

// v of a row at four consecutive k as the MFMA expand's PARTS 16-bit operand parts (two, or three: all 24 bits) and, for binary16,
// the row's range factor.  The R / 4 lanes that hold a row are consecutive lanes of a wave, and every lane of the wave calls this
// (live or not; what a lane that is not live holds is of no consequence).
template <class DT, int R, int PARTS>
__device__ __forceinline__ void split_quad(const float4& sum, uint2 (&part)[PARTS], float& undo) {
  constexpr int GPR = R / 4;  // lanes per row
  float f[4] = {sum.x, sum.y, sum.z, sum.w};
  undo = 1.f;
  if (std::is_same<DT, F16>::value) {
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) amax = fmaxf(amax, PARTS == 3 && !(fabsf(f[i]) < 3.0e38f) ? 0.f : fabsf(f[i]));
#pragma unroll
    for (int msk = 1; msk < GPR; msk <<= 1) amax = fmaxf(amax, __shfl_xor(amax, msk, 64));
    const float down = range_factor<PARTS == 3>(amax, undo);
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] *= down;
  }
  uint32_t h[PARTS][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (PARTS == 3)
      split16<DT>(f[i], h[0][i], h[1][i], h[2][i]);
    else
      split16<DT>(f[i], h[0][i], h[1][i]);
  }
#pragma unroll
  for (int q = 0; q < PARTS; ++q) part[q] = make_uint2(h[q][0] | (h[q][1] << 16), h[q][2] | (h[q][3] << 16));
}

// A lane's part of the split-K partial sums, four consecutive k, of up to N slices in flight together (load(i) gives those
// of slice i), added up in ascending order.
template <int N>
struct PartialSums {
  float4 q[N];
  template <class Load>
  __device__ __forceinline__ void load(int from, int slices, Load slice) {
#pragma unroll
    for (int i = 0; i < N; ++i) q[i] = slice(min(from + i, slices - 1));
  }
  __device__ __forceinline__ void add_to(float4& sum, int from, int slices) const {
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (from + i < slices) {
        sum.x += q[i].x; sum.y += q[i].y; sum.z += q[i].z; sum.w += q[i].w;
      }
  }
};

// ---------------------------------------------------------------- shrink
//
// P add-ons on the same x side by side (P = 1: one): P slices of A_i in LDS, P sets of partial sums, one
// pass over x, which is most of a shrink's bytes.
//
// Workgroup = (k-slice, row block, group of P add-ons).  Each wave owns
// sixteen rows.  The slice is walked in chunks of KC: while the matrix cores work on a chunk, the
// loads of the next one -- the wave's x operands (KC / 32 128-bit loads per lane) and the
// workgroup's share of A_i -- are in flight; A_i passes through registers into the other of two LDS
// buffers, transposed, so one LDS-only barrier per chunk suffices and no load is ever drained at
// one.  The first operand is A_i^T, so a lane ends with four consecutive columns of one row and the
// partial sums leave as 128-bit stores.
template <int R, int P>
struct ShrinkShape {
  static constexpr int kTiles = (R + 15) / 16;              // 16-column tiles of one add-on
  static constexpr int kColumns = P * R;
  static constexpr int kWaves = kColumns > 32 ? 8 : 4;      // more waves to share a larger chunk of A_i
  // k per LDS buffer: 128.  Two chunks' operands of x and one chunk of A_i are in registers at a time, 88 registers at
  // rank 64; with 256 they pass the 128 of four waves per SIMD and 29 go to scratch memory (4814 rows of 8192: 44 us
  // against 26; with 64: 28)
  static constexpr int kChunk = 128;
  static constexpr int kBlk = kTiles * 16 + 1;              // 16-byte slots {8 k of one column} per 8 k; the odd pitch spreads the banks
  static constexpr int kRows = 16 * kWaves;
  static constexpr size_t kLds = (size_t)2 * P * (kChunk / 8) * kBlk * 16;
};

struct ShrinkTable {
  const uint16_t* x[kSharedShrinkMost];
  const uint16_t* const* A_ptrs[kSharedShrinkMost];
  float* partials[kSharedShrinkMost];  // [slices][n_tokens][R]
};

template <class DT, int R, int P>
__global__ __launch_bounds__((64 * ShrinkShape<R, P>::kWaves), 4) void shrink_stream_kernel(
    const int32_t* __restrict__ seg_starts, int n_segs, float guess, int slices, int groups, int h_in, int kslice,
    int n_tokens, long long layer_off, unsigned long long* header, ShrinkTable tab) {
  using Shape = ShrinkShape<R, P>;
  constexpr int NT = 64 * Shape::kWaves;
  constexpr int NTILE = Shape::kTiles;
  constexpr int RPAD = NTILE * 16;
  constexpr int CG = R / 8;
  constexpr int KC = Shape::kChunk;
  constexpr int XB = KC / 32;
  constexpr int BLK = Shape::kBlk;
  constexpr int PAIRS = (KC / 2) * CG;                // (pair of k, eight columns) items of one add-on's chunk
  constexpr int ITEMS = (PAIRS * P + NT - 1) / NT;    // per thread
  static_assert(PAIRS % NT == 0 || NT % PAIRS == 0 || P == 1, "an item row of the block belongs to one add-on");
  __shared__ __align__(16) uint32_t at[2][P * (KC / 8) * BLK * 4];

  const int tid = threadIdx.x, lane = tid & 63;
  // told to be wave-uniform, the wave index keeps the base of the wave's x buffer in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  SGMV_TRACE_DECL
  SGMV_TRACE_POINT(0);
  // eight (slice, block) pairs, one per XCD, times the groups of add-ons: the groups that read the same
  // part of x run on one XCD at the same time and find it in its L2
  unsigned id = blockIdx.x;
  if (blockIdx.y != 0) id += blockIdx.y * gridDim.x;  // (reading the grid's size costs a memory latency)
  const unsigned row_of_eight = id / (8 * (unsigned)groups), in_row = id - row_of_eight * 8 * (unsigned)groups;
  const unsigned pair = row_of_eight * 8 + in_row % 8;
  const int s = pair % (unsigned)slices;
  const Found at_seg = find_item<Shape::kRows>(seg_starts, n_segs, pair / (unsigned)slices, 1, 0, guess, lane,
                                               [](int rows) { return (rows + Shape::kRows - 1) / Shape::kRows; });
  if (at_seg.seg < 0) return;
  const int block_row = at_seg.lo + at_seg.index * Shape::kRows;
  const int p0 = (int)(in_row / 8) * P;
  const uint16_t* A[P];
  bool any = false;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    A[p] = tab.A_ptrs[p0 + p][at_seg.seg];
    any = any || A[p] != nullptr;
  }
  if (!any) return;
  const int k0 = s * kslice;
  const int klen = min(h_in, k0 + kslice) - k0;
  if (klen <= 0) return;
  SGMV_TRACE_POINT(8);
  const int m = lane & 15, g = lane >> 4;

  const int row0 = block_row + wave * 16;
  const int rows = max(0, min(16, at_seg.hi - row0));  // rows past the segment read as zeros
  const __amdgpu_buffer_rsrc_t rX = make_uniform_buffer(
      tab.x[p0] + (long long)(rows > 0 ? row0 : block_row) * h_in + k0, rows > 0 ? (uint32_t)((rows - 1) * h_in + klen) * 2u : 0u);
  const uint32_t x_lane = (uint32_t)(m * h_in + g * 8) * 2u;
  const int k_end = m < rows ? klen - g * 8 : 0;
  auto load_x = [&](uint4 (&q)[XB], int c) {
#pragma unroll
    for (int i = 0; i < XB; ++i) {
      const int k = c * KC + i * 32;
      q[i] = buffer_load128(rX, k < k_end ? x_lane + (uint32_t)k * 2u : kOutOfRange);
    }
  };
  __amdgpu_buffer_rsrc_t rA[P];  // an add-on without an adapter for this segment: an empty buffer, zeros
#pragma unroll
  for (int p = 0; p < P; ++p)
    rA[p] = make_uniform_buffer(A[p] != nullptr ? A[p] + layer_off + (long long)k0 * R : tab.x[p0],
                        A[p] != nullptr ? (uint32_t)klen * R * 2u : 0u);
  uint4 a0[ITEMS], a1[ITEMS];
  auto load_a = [&](int c) {
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      // item = kp * CG + cg of one add-on -> rows 2 kp, 2 kp + 1, columns 8 cg .. +7
      const int all = u * NT + tid, item = P == 1 ? all : all % PAIRS;
      const uint32_t o = P * PAIRS % NT == 0 || all < P * PAIRS
                             ? (uint32_t)(c * KC * R + (2 * item - item % CG) * 8) * 2u : kOutOfRange;
      if constexpr (P == 1) {
        a0[u] = buffer_load128(rA[0], o);
        a1[u] = buffer_load128(rA[0], o + (uint32_t)R * 2u);
      } else if constexpr (PAIRS % NT == 0) {  // all lanes at the same add-on
        a0[u] = buffer_load128(rA[u / (PAIRS / NT)], o);
        a1[u] = buffer_load128(rA[u / (PAIRS / NT)], o + (uint32_t)R * 2u);
      } else {  // several add-ons in one row of items, whole waves each
        const int mine = __builtin_amdgcn_readfirstlane(all / PAIRS);
#pragma unroll
        for (int p = 0; p < P; ++p)
          if (mine == p) {
            a0[u] = buffer_load128(rA[p], o);
            a1[u] = buffer_load128(rA[p], o + (uint32_t)R * 2u);
          }
      }
    }
  };
  auto place_a = [&](uint32_t* buf) {
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int all = u * NT + tid, item = P == 1 ? all : all % PAIRS;
      if (P * PAIRS % NT == 0 || all < P * PAIRS) {
        const int cg = item % CG, kp = item / CG;
        const uint32_t w0[4] = {a0[u].x, a0[u].y, a0[u].z, a0[u].w};
        const uint32_t w1[4] = {a1[u].x, a1[u].y, a1[u].z, a1[u].w};
        uint32_t* to = &buf[((P == 1 ? 0 : all / PAIRS) * (KC / 8) + (kp >> 2)) * BLK * 4 + (kp & 3)];  // k block, dword of the k pair
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // columns 8 cg + 2 i and + 2 i + 1, column n in slot n
          to[(8 * cg + 2 * i) * 4] = (w0[i] & 0xFFFFu) | (w1[i] << 16);
          to[(8 * cg + 2 * i + 1) * 4] = (w0[i] >> 16) | (w1[i] & 0xFFFF0000u);
        }
      }
    }
  };

  uint4 q0[XB], q1[XB];
  load_a(0);
  load_x(q0, 0);
  if (R < RPAD) {  // slots no column of A_i fills
    constexpr int PER = (RPAD - R) * 4;
    for (int i = tid; i < 2 * P * (KC / 8) * PER; i += NT) (&at[0][0])[(i / PER * BLK + R) * 4 + i % PER] = 0u;
  }
  f32x4 acc[P][NTILE];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int t = 0; t < NTILE; ++t) acc[p][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto consume = [&](const uint4 (&q)[XB], const uint32_t* buf) {
#pragma unroll
    for (int i = 0; i < XB; ++i) {
      asm volatile("" ::: "memory");  // a step's LDS reads stay in the step: hoisted together they would spill
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int t = 0; t < NTILE; ++t) {
          // A_i^T first: D[column 16 t + 4 g + i][token m]
          const uint4 w = *reinterpret_cast<const uint4*>(&buf[((p * (KC / 8) + i * 4 + g) * BLK + t * 16 + m) * 4]);
          acc[p][t] = mfma16x16x32<DT>(w, q[i], acc[p][t]);
        }
    }
  };
  const int chunks = (klen + KC - 1) / KC;
  SGMV_TRACE_POINT(1);
  for (int c = 0;; c += 2) {
    place_a(at[0]);
    load_a(c + 1);      // past the slice: out of range, no memory traffic
    load_x(q1, c + 1);
    lds_barrier();      // LDS only: the loads stay in flight
    consume(q0, at[0]);
    if (c + 1 >= chunks) break;
    place_a(at[1]);
    load_a(c + 2);
    load_x(q0, c + 2);
    lds_barrier();
    consume(q1, at[1]);
    if (c + 2 >= chunks) break;
  }
  SGMV_TRACE_POINT(2);
  // lane (m, g): row m of the tile, columns 16 t + 4 g .. + 3 of every column tile
  if (m < rows) {
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int t = 0; t < NTILE; ++t) {
        const int n = t * 16 + 4 * g;
        if (n < R)
          *reinterpret_cast<float4*>(tab.partials[p0 + p] + ((long long)s * n_tokens + row0 + m) * R + n) =
              make_float4(acc[p][t][0], acc[p][t][1], acc[p][t][2], acc[p][t][3]);
      }
  }
  SGMV_TRACE_POINT(6);
#ifdef SGMV_TRACE
  if (header != nullptr) {
    SGMV_TRACE_FLUSH(tid == 0, 0, 2);
    SGMV_TRACE_FLUSH(tid == 0, 6, 6);
    SGMV_TRACE_FLUSH(tid == 0, 8, 8);
  }
#endif
}

// ---------------------------------------------------------------- expand

// v[row][k] = sum over the split-K parts (ascending), written out as the two or three 16-bit
// operands the expand kernel feeds to the matrix cores: vh, vl [n_tokens][R] 16-bit, the third likewise behind
// the partial sums (third_part), undo [n_tokens] fp32 (split_quad).  One thread handles four consecutive k of a row;
// the kernel is one memory latency long.
// blockIdx.y is the add-on.
struct FinalizeTable {
  const float* v_parts[kSharedShrinkMost];
  uint16_t* vh[kSharedShrinkMost];
  uint16_t* vl[kSharedShrinkMost];
  float* undo[kSharedShrinkMost];
};
// (A pointer of its own in the kernels' arguments moves others to another cache line, which every workgroup waits for: 4814
// rows, rank 16, four calls of 8192 -> 8192 204.2 -> 205.4 us.)
template <int R>
__device__ __forceinline__ uint16_t* third_part(const float* v_parts, int nparts, int n_tokens) {
  return reinterpret_cast<uint16_t*>(const_cast<float*>(v_parts + nparts * ((long long)n_tokens * R)));
}
template <class DT, int R, int PARTS>
__global__ __launch_bounds__(256) void finalize_v_kernel(int nparts, int n_tokens, FinalizeTable tab) {
  constexpr int GPR = R / 4;  // threads per row
  const int z = blockIdx.y;
  const long long item = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long total = (long long)n_tokens * GPR;
  const bool live = item < total;
  const long long it = live ? item : total - 1;
  const long long e0 = it * 4;  // first element (row * R + k)
  float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add_parts = [&](auto n_tag) {
    PartialSums<decltype(n_tag)::value> parts;
    for (int from = 0; from < nparts; from += decltype(n_tag)::value) {
      parts.load(from, nparts, [&](int i) {
        return *reinterpret_cast<const float4*>(tab.v_parts[z] + e0 + i * ((long long)n_tokens * R));
      });
      parts.add_to(sum, from, nparts);
    }
  };
  if (nparts <= 4)
    add_parts(std::integral_constant<int, 4>{});
  else if (nparts <= 8)
    add_parts(std::integral_constant<int, 8>{});
  else
    add_parts(std::integral_constant<int, 16>{});
  uint2 part[PARTS];
  float undo;
  split_quad<DT, R>(sum, part, undo);
  if (live) {
    *reinterpret_cast<uint2*>(tab.vh[z] + e0) = part[0];
    *reinterpret_cast<uint2*>(tab.vl[z] + e0) = part[1];
    if constexpr (PARTS == 3) *reinterpret_cast<uint2*>(third_part<R>(tab.v_parts[z], nparts, n_tokens) + e0) = part[2];
    if (it % GPR == 0) tab.undo[z][it / GPR] = undo;
  }
}

// How the expand adds the partial sums of a block's v up itself (DIRECT, ranks up to 16): a thread has four consecutive k
// of a row, kParts slices of them in flight together.
template <int R>
struct DirectShape {
  static constexpr int kPerRow = R / 4;
  static constexpr int kQuads = kExpandRows * kPerRow;
  static constexpr int kParts = 8;
  static constexpr int kPitch = R + 8;  // 16-bit elements of a row in LDS
};

// What the expand of one add-on reads and writes.
struct ExpandTable {
  uint16_t* y[kSharedShrinkMost];
  const uint16_t* vh[kSharedShrinkMost];
  const uint16_t* vl[kSharedShrinkMost];
  const float* undo[kSharedShrinkMost];
  const uint16_t* const* A_ptrs[kSharedShrinkMost];  // may be nullptr
  const uint16_t* const* B_ptrs[kSharedShrinkMost];
  const float* v_parts[kSharedShrinkMost];  // DIRECT; else vh, vl and undo, which finalize_v_kernel made of them
};

// grid = (items, add-ons, further items); v comes as the partial sums (DIRECT) or as finalize_v_kernel's operands.  The list of items: for a segment
// of more than few_rows rows its 64-row blocks x strips of 256 columns, for a shorter one its strips of 2048
// columns.
//
// Block items.  The product is taken as D = v B_i with the token rows in the first operand: lane
// (n = l % 16, g = l / 16) receives D[row 4 g + i][column slot n] of every 16-column tile.  Tile t of a
// group of 64 columns holds its columns 4 n + t, so a lane ends up with four consecutive columns
// (8 bytes) of rows 4 g .. 4 g + 3, and each of its four 64-bit accesses of y covers four rows x 128
// contiguous bytes across the wave: whole cache lines in both directions.  (Measured on plain
// read-modify-write kernels of this shape: 5.9 TB/s with the non-temporal hint on both sides,
// 5.1 without or with one of them, against 3.3 TB/s for 128-bit accesses that cover sixteen rows x 64 bytes, the layout the transposed product
// D = B_i^T v^T would give.)  A wave owns sixteen rows and walks the strip's four column groups (with one
// or two tiles of rows in the block, one or two groups): its v operands stay in registers, the strip of
// B_i, transposed through LDS once, is shared by the four waves, and all of the wave's loads of y are in
// flight at once, requested before the strip is placed.  Workgroups are short-lived on purpose:
// the launch has more than fit the chip at once, and the hardware hands the next one to
// whichever compute unit comes free.
//
// What bounds it besides HBM is the vector ALU, which a wave keeps busy for 4 cycles per
// instruction: y is rounded two values at a time by the conversion instruction, the rows of a
// block are cut off by the buffer's range check instead of a compare per access, a thread
// transposes up to eight weight rows in registers so that it writes LDS 128 bits at a time, and at ranks
// up to 16 the two parts of v share one 32-deep step.  (4814 rows, bfloat16: 8192 -> 28672 at rank 64 117 -> 108 us,
// 8192 -> 8192 at rank 16 32 -> 29 us.)
//
// Strip items (one or two rows, where there are enough of them: launch_expand_matrix_t): nothing to reuse, a row
// of B_i is streamed to the vector ALUs, eight columns per lane, eight rows of it in flight (three projections of
// 4096 -> 4096, 41 decode rows beside three prompts of 1152 rows, rank 16: 22.5 -> 17.0 us).  Three and four rows are
// taken in pairs, each pair reading B_i again, and cost up to twice as much as blocks (expand to 13824 at rank 64
// of 8 / 40 / 100 segments of three rows 21.6 / 33.3 / 68.3 us against 8.7 / 21.9 / 47.6) -- except at rank 8, where B_i is one
// batch of loads, and where they are many (expand to 13824 of 100, 700 items, 15.0 against 19.0; add-on 4096 -> 4096 of 100,
// 200 items, 17.0 against 18.3, of 40, 80 items, 13.7 against 13.0).
constexpr int kFewCols = 2048;

// y[0 .. 3] of one row: y + scale * sum
template <class DT>
__device__ __forceinline__ uint2 add4(const uint2& y, float scale, const f32x4 (&acc)[4], int i) {
  float f[4];
  unpack2<DT>(y.x, f[0], f[1]);
  unpack2<DT>(y.y, f[2], f[3]);
#pragma unroll
  for (int t = 0; t < 4; ++t) f[t] = fmaf(scale, acc[t][i], f[t]);
  return make_uint2(pack2<DT>(f[0], f[1]), pack2<DT>(f[2], f[3]));
}

// (three parts of v at rank 64: 137 registers)
template <class DT, int R, bool DIRECT, int PARTS>
__global__ __launch_bounds__(256, PARTS == 3 ? 3 : 4) void expand_matrix_kernel(
    const int32_t* __restrict__ seg_starts, int n_segs, float guess, int strips, int few_rows, int few_strips, int h_out,
    long long layer_off, float scale, unsigned long long* header, ExpandTable tab, int nparts, int n_tokens) {
  constexpr int NC = kExpandCols;        // columns of a strip
  constexpr int CT = 4;                  // 16-column tiles (and columns per lane) of a group
  constexpr int NG = NC / (16 * CT);     // column groups of the strip
  constexpr int KSTEPS = R <= 32 ? 1 : R / 32;
  constexpr bool PAIRED = R <= 16;       // the high and the low part of v side by side in one 32-deep step
  constexpr int KB = R / 8;              // blocks of eight weight rows
  constexpr int KR = R >= 64 ? 8 : R >= 32 ? 4 : 2;  // weight rows a thread transposes
  static_assert(!DIRECT || (PAIRED && DirectShape<R>::kQuads <= 256), "a thread has at most one quad of v");
  constexpr int ITEMS = (R / KR) * (NC / 8);
  static_assert(ITEMS <= 256, "one item per thread");
  static_assert(PARTS == 2 || (PARTS == 3 && !PAIRED), "v as two parts or three");
  // B_i strip, transposed, as 16-byte slots {8 consecutive k of one column}, k block by k block; column c of
  // the strip sits in slot (c % 8) * PITCH + c / 8: consecutive lanes of the staging write
  // consecutive slots, and the sixteen lanes of an operand read (columns 4 n + t) read two runs
  // of eight slots that lie in different halves of the banks
  constexpr int PITCH = 34, BLK = 8 * PITCH;
  __shared__ __align__(16) uint32_t bt[KB * BLK * 4];
  using Direct = DirectShape<R>;
  // the operands of the block's v, high and low part, and its rows' range factors
  __shared__ __align__(16) uint16_t vs[2][DIRECT ? kExpandRows * Direct::kPitch : 8];
  __shared__ float undo_s[DIRECT ? kExpandRows : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int z = blockIdx.y;
  uint16_t* const y = tab.y[z];
  const float* const v_parts = tab.v_parts[z];
  const long long v_stride = (long long)n_tokens * R;  // from one part to the next
  const uint16_t *const vh = tab.vh[z], *const vl = tab.vl[z];
  const uint16_t* const vr = PARTS == 3 ? third_part<R>(v_parts, nparts, n_tokens) : nullptr;
  const float* const undo = tab.undo[z];
  SGMV_TRACE_DECL
  SGMV_TRACE_POINT(0);

  unsigned index = blockIdx.x;
  if (blockIdx.z != 0) index += blockIdx.z * gridDim.x;
  const Found it = find_item<kExpandRows>(seg_starts, n_segs, index, strips, few_strips, guess, lane, [=](int rows) {
    return rows <= few_rows ? few_strips : (rows + kExpandRows - 1) / kExpandRows * strips;
  });
  if (it.seg < 0) return;
  const uint16_t* B = tab.B_ptrs[z][it.seg];
  if (B == nullptr) return;
  if (tab.A_ptrs[z] != nullptr && tab.A_ptrs[z][it.seg] == nullptr) return;
  SGMV_TRACE_POINT(8);
  {
    if (it.hi - it.lo <= few_rows) {
      const int c = it.index * kFewCols + tid * 8;
      const uint32_t off = c < h_out ? (uint32_t)c * 2u : kOutOfRange;
      constexpr int JC = 8;  // weight rows in flight
      const __amdgpu_buffer_rsrc_t rB = make_uniform_buffer(B + layer_off, (uint32_t)((long long)R * h_out * 2));
      for (int row = it.lo; row < it.hi; row += 2) {
        const bool two = row + 1 < it.hi;
        // lane j: v[row][j], v[row + 1][j]
        const int vj = min(lane, R - 1), second = two ? R : 0;
        constexpr int PB = 8;  // partial sums of a row in flight together
        float p0[PB], p1[PB], sum0 = 0.f, sum1 = 0.f;
        int part = 0;
        auto load_parts = [&]() {
#pragma unroll
          for (int i = 0; i < PB; ++i) {
            const float* const at = v_parts + min(part + i, nparts - 1) * v_stride + (long long)row * R + vj;
            p0[i] = at[0];
            p1[i] = at[second];
          }
        };
        auto add_parts = [&]() {
#pragma unroll
          for (int i = 0; i < PB; ++i)
            if (part + i < nparts) {
              sum0 += p0[i];
              sum1 += p1[i];
            }
        };
        if constexpr (DIRECT) {
          for (; part + PB < nparts; part += PB) {
            load_parts();
            add_parts();
          }
          load_parts();
        }
        uint4 b[JC];
#pragma unroll
        for (int j = 0; j < JC; ++j) b[j] = buffer_load128<kNonTemporal>(rB, off + (uint32_t)(j * h_out) * 2u);
        const __amdgpu_buffer_rsrc_t rY = make_uniform_buffer(y + (long long)row * h_out, (uint32_t)(two ? 2 : 1) * h_out * 2u);
        const uint4 y0 = buffer_load128<kNonTemporal>(rY, off);
        const uint4 y1 = buffer_load128<kNonTemporal>(rY, off + (uint32_t)h_out * 2u);
        int v0, v1;
        if constexpr (DIRECT) {
          add_parts();
          v0 = __float_as_int(sum0 * scale);
          v1 = __float_as_int(sum1 * scale);
        } else {
          const uint16_t *const h = vh + (long long)row * R + vj, *const l = vl + (long long)row * R + vj;
          const float u0 = std::is_same<DT, F16>::value ? undo[row] : 1.f;
          const float u1 = std::is_same<DT, F16>::value ? undo[two ? row + 1 : row] : 1.f;
          float l0 = decode1<DT>(l[0]), l1 = decode1<DT>(l[second]);
          if constexpr (PARTS == 3) {
            const uint16_t* const r = vr + (long long)row * R + vj;
            l0 += decode1<DT>(r[0]);
            l1 += decode1<DT>(r[second]);
          }
          v0 = __float_as_int((decode1<DT>(h[0]) + l0) * (scale * u0));
          v1 = __float_as_int((decode1<DT>(h[second]) + l1) * (scale * u1));
        }
        float s0[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, s1[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int jc = 0; jc < R; jc += JC) {
#pragma unroll
          for (int j = 0; j < JC; ++j) {
            // one row at a time: the compiler would widen all of them to fp32 first, and spill
            asm volatile("" : "+v"(b[j].x), "+v"(b[j].y), "+v"(b[j].z), "+v"(b[j].w), "+v"(s0[7]), "+v"(s1[7]));
            float w[8];
            unpack8<DT>(b[j], w);
            // its register takes the row that follows eight later (none: past the end of the buffer): the
            // loads in flight never run dry
            if (R > JC) b[j] = buffer_load128<kNonTemporal>(rB, off + (uint32_t)((jc + JC + j) * h_out) * 2u);
            const float f0 = __int_as_float(__builtin_amdgcn_readlane(v0, jc + j));
            const float f1 = __int_as_float(__builtin_amdgcn_readlane(v1, jc + j));
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              s0[e] = fmaf(f0, w[e], s0[e]);
              s1[e] = fmaf(f1, w[e], s1[e]);
            }
          }
        }
        auto put = [&](const uint4& q, const float (&sum)[8], uint32_t at) {
          float f[8];
          unpack8<DT>(q, f);
          buffer_store128<kNonTemporal>(rY, at, make_uint4(pack2<DT>(f[0] + sum[0], f[1] + sum[1]), pack2<DT>(f[2] + sum[2], f[3] + sum[3]),
                                                           pack2<DT>(f[4] + sum[4], f[5] + sum[5]), pack2<DT>(f[6] + sum[6], f[7] + sum[7])));
        };
        put(y0, s0, off);
        if (two) put(y1, s1, off + (uint32_t)h_out * 2u);
        if (R > 8) break;  // two rows at most
      }
    } else {
      const int block = it.index / strips, strip = it.index - block * strips;
      const int row0 = it.lo + block * kExpandRows, left = it.hi - row0;
      const int tiles = left > 32 ? 4 : left > 16 ? 2 : 1;  // sixteen-row tiles the waves are dealt to
      const int tile = wave & (tiles - 1), group0 = wave / tiles * tiles;  // this wave's rows, its first column group
      const int r0 = row0 + tile * 16, rows = max(0, min(16, it.hi - r0));
      const int c0 = strip * NC, ncols = min(NC, h_out - c0);
      const int n = lane & 15, g = lane >> 4;

      // ---- the strip's loads first (L2 hits mostly), so that placing it does not wait for y
      const int cg = tid % (NC / 8), kq = tid / (NC / 8);
      const bool stages = (ITEMS == 256 || tid < ITEMS);
      const __amdgpu_buffer_rsrc_t rB = make_uniform_buffer(B + layer_off + c0, (uint32_t)((long long)(R - 1) * h_out + ncols) * 2u);
      uint4 w[KR];
#pragma unroll
      for (int i = 0; i < KR; ++i)
        w[i] = buffer_load128(rB, stages && cg * 8 < ncols ? (uint32_t)((kq * KR + i) * h_out + cg * 8) * 2u : kOutOfRange);

      // ---- v: row n of the tile; rows past the segment read as zeros
      uint4 v_hi[KSTEPS], v_lo[KSTEPS], v_rest[KSTEPS];
      float un[4];
      // DIRECT: thread `tid` has quad `tid` of the block, whose partial sums are requested here, in front of y (the loads of
      // a wave return in order), and added up behind y's requests
      PartialSums<Direct::kParts> parts;
      float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
      int part = 0;
      const int quad_row = tid / Direct::kPerRow;
      if constexpr (DIRECT) {
        // rows past the segment read as zeros
        const __amdgpu_buffer_rsrc_t rV = make_uniform_buffer(v_parts + (long long)row0 * R, (uint32_t)((nparts - 1) * v_stride + left * R) * 4u);
        const uint32_t quad_at = tid < Direct::kQuads && quad_row < left ? (uint32_t)tid * 16u : kOutOfRange;
        auto load_parts = [&]() {
          parts.load(part, nparts, [&](int p) {
            return __builtin_bit_cast(float4, buffer_load128_at(rV, quad_at, (uint32_t)(p * v_stride * 4)));
          });
        };
        for (; part + Direct::kParts < nparts; part += Direct::kParts) {
          load_parts();
          parts.add_to(sum, part, nparts);
        }
        load_parts();
      } else {
        const __amdgpu_buffer_rsrc_t rH = make_uniform_buffer(vh + (long long)r0 * R, (uint32_t)(rows * R) * 2u);
        const __amdgpu_buffer_rsrc_t rL = make_uniform_buffer(vl + (long long)r0 * R, (uint32_t)(rows * R) * 2u);
        if constexpr (PAIRED) {  // k blocks 0 .. KB - 1 the high part, KB .. 2 KB - 1 the low one
          v_hi[0] = buffer_load128(rH, g < KB ? (uint32_t)(n * R + g * 8) * 2u : kOutOfRange);
          v_lo[0] = buffer_load128(rL, g >= KB && g < 2 * KB ? (uint32_t)(n * R + (g - KB) * 8) * 2u : kOutOfRange);
        } else {
#pragma unroll
          for (int ks = 0; ks < KSTEPS; ++ks) {
            v_hi[ks] = buffer_load128(rH, (uint32_t)(n * R + ks * 32 + g * 8) * 2u);
            v_lo[ks] = buffer_load128(rL, (uint32_t)(n * R + ks * 32 + g * 8) * 2u);
            if constexpr (PARTS == 3) {
              const __amdgpu_buffer_rsrc_t rR = make_uniform_buffer(vr + (long long)r0 * R, (uint32_t)(rows * R) * 2u);
              v_rest[ks] = buffer_load128(rR, (uint32_t)(n * R + ks * 32 + g * 8) * 2u);
            }
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
          un[i] = std::is_same<DT, F16>::value && rows > 0 ? undo[r0 + min(4 * g + i, rows - 1)] : 1.f;
      }
      auto place_v = [&]() {
        parts.add_to(sum, part, nparts);
        uint2 operand[2];
        float factor;
        split_quad<DT, R>(sum, operand, factor);
        if (tid < Direct::kQuads) {
          const int k = tid % Direct::kPerRow * 4;
          *reinterpret_cast<uint2*>(&vs[0][quad_row * Direct::kPitch + k]) = operand[0];
          *reinterpret_cast<uint2*>(&vs[1][quad_row * Direct::kPitch + k]) = operand[1];
          if (std::is_same<DT, F16>::value && k == 0) undo_s[quad_row] = factor;
        }
      };
      auto fetch_v = [&]() {
        const int row = (tile * 16 + n) * Direct::kPitch;
        const uint4 none = make_uint4(0, 0, 0, 0);
        v_hi[0] = g < 2 * KB ? *reinterpret_cast<const uint4*>(&vs[g < KB ? 0 : 1][row + g % KB * 8]) : none;
        v_lo[0] = none;
#pragma unroll
        for (int i = 0; i < 4; ++i) un[i] = std::is_same<DT, F16>::value ? undo_s[tile * 16 + 4 * g + i] : 1.f;
      };

      // FULL: every column of the strip is inside h_out.  GROUPS: the most column groups this wave takes, so that
      // only their part of y is loaded and held.  (Loads from an empty buffer for the groups that other waves take cost
      // their issue all the same: expand to 13824 of 40 / 200 segments of 8 rows, rank 16, 15.9 / 62.1 -> 12.4 / 45.7 us.
      // One code for all counts kept up to nine registers of rank 64 in scratch memory: 8192 -> 28672, 4800 rows,
      // 134.6 -> 131.6 us.)
      auto rest = [&](auto full_tag, auto groups_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        constexpr int GROUPS = decltype(groups_tag)::value;
        auto mine = [&](int j) { return GROUPS == NG || j < tiles; };
        // rows past the segment lie past the end of the buffer
        uint2 yq[GROUPS][4];
        uint32_t yoff[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) yoff[i] = (uint32_t)((4 * g + i) * h_out + c0 + group0 * (16 * CT) + n * CT) * 2u;
        const uint32_t y_bytes = (uint32_t)(rows * h_out) * 2u;
        uint16_t* const y_at = y + (long long)(rows > 0 ? r0 : row0) * h_out;
        auto in_strip = [&](int j) { return FULL || (group0 + j) * (16 * CT) + n * CT < ncols; };
#pragma unroll
        for (int j = 0; j < GROUPS; ++j) {
          const __amdgpu_buffer_rsrc_t rY = make_uniform_buffer(y_at, y_bytes);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (mine(j)) yq[j][i] = buffer_load64_at<kNonTemporal>(rY, in_strip(j) ? yoff[i] : kOutOfRange, (uint32_t)j * (16 * CT * 2));
        }

        // ---- place the strip: dword d of a slot holds rows 2 d and 2 d + 1 of the k block
        if (stages) {
          const uint16_t* e[KR];
#pragma unroll
          for (int i = 0; i < KR; ++i) e[i] = reinterpret_cast<const uint16_t*>(&w[i]);
          uint32_t* const to = &bt[((kq * KR / 8) * BLK + cg) * 4 + kq * KR % 8 / 2];
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            uint32_t d[KR / 2];
#pragma unroll
            for (int k = 0; k < KR / 2; ++k) d[k] = (uint32_t)e[2 * k][c] | ((uint32_t)e[2 * k + 1][c] << 16);
            uint32_t* const at = to + c * PITCH * 4;
            if constexpr (KR == 8)
              *reinterpret_cast<uint4*>(at) = make_uint4(d[0], d[1], d[2], d[3]);
            else if constexpr (KR == 4)
              *reinterpret_cast<uint2*>(at) = make_uint2(d[0], d[1]);
            else
              *at = d[0];
          }
        }
        if constexpr (DIRECT) {
          __builtin_amdgcn_sched_barrier(0);  // the strip's registers are free by now
          place_v();
        }
        SGMV_TRACE_POINT(1);
        lds_barrier();  // LDS only: the loads of y stay in flight
        if constexpr (DIRECT) fetch_v();
        SGMV_TRACE_POINT(2);

        // second operands: column 64 (group0 + j) + 4 n + t of the strip
        auto operand = [&](int j, int block_of_k, int t) {
          const int slot = (4 * (n & 1) + t) * PITCH + 8 * (group0 + j) + (n >> 1);
          return *reinterpret_cast<const uint4*>(&bt[(block_of_k * BLK + slot) * 4]);
        };
        const uint4 v_pair = make_uint4(v_hi[0].x | v_lo[0].x, v_hi[0].y | v_lo[0].y, v_hi[0].z | v_lo[0].z, v_hi[0].w | v_lo[0].w);
#pragma unroll
        for (int j = 0; j < GROUPS; ++j) {
          if (mine(j)) {
            asm volatile("" ::: "memory");  // a group's operands are read where they are used: together they would spill
            f32x4 acc[CT];
#pragma unroll
            for (int t = 0; t < CT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (PAIRED) {
#pragma unroll
              for (int t = 0; t < CT; ++t) {
                uint4 bop = operand(j, g % KB, t);
                if (2 * KB < 4 && g >= 2 * KB) bop = make_uint4(0, 0, 0, 0);  // k blocks neither part of v fills
                acc[t] = mfma16x16x32<DT>(v_pair, bop, acc[t]);
              }
            } else {
#pragma unroll
              for (int ks = 0; ks < KSTEPS; ++ks) {
                uint4 bop[CT];
#pragma unroll
                for (int t = 0; t < CT; ++t) bop[t] = operand(j, ks * 4 + g, t);
                if constexpr (PARTS == 3) {
#pragma unroll
                  for (int t = 0; t < CT; ++t) acc[t] = mfma16x16x32<DT>(v_rest[ks], bop[t], acc[t]);
                }
#pragma unroll
                for (int t = 0; t < CT; ++t) acc[t] = mfma16x16x32<DT>(v_lo[ks], bop[t], acc[t]);
#pragma unroll
                for (int t = 0; t < CT; ++t) acc[t] = mfma16x16x32<DT>(v_hi[ks], bop[t], acc[t]);
              }
            }
            // acc[t][i] is column 64 (group0 + j) + 4 n + t of row 4 g + i
            const __amdgpu_buffer_rsrc_t rY = make_uniform_buffer(y_at, y_bytes);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              buffer_store64_at<kNonTemporal>(rY, in_strip(j) ? yoff[i] : kOutOfRange, (uint32_t)j * (16 * CT * 2),
                                              add4<DT>(yq[j][i], scale * un[i], acc, i));
          }
        }
      };
      auto by_columns = [&](auto groups_tag) {
        if (ncols == NC)
          rest(std::true_type{}, groups_tag);
        else
          rest(std::false_type{}, groups_tag);
      };
      static_assert(NG == 4, "a wave takes four, two or one of the column groups");
      if (tiles == 4)
        by_columns(std::integral_constant<int, 4>{});
      else
        by_columns(std::integral_constant<int, 2>{});
    }
  }
  SGMV_TRACE_POINT(6);
#ifdef SGMV_TRACE
  if (header != nullptr) {
    SGMV_TRACE_FLUSH(tid == 0, 0, 2);
    SGMV_TRACE_FLUSH(tid == 0, 6, 6);
    SGMV_TRACE_FLUSH(tid == 0, 8, 8);
  }
#endif
}

// ---------------------------------------------------------------- launchers

// Along one dimension of a grid, which holds fewer than 2^32 threads (512 per workgroup here at most); a longer list
// goes on in the next dimension.
constexpr long long kMostWorkgroups = 1 << 22;

// Whether one pass over x serves n add-ons (their chunks of A_i side by side in LDS).
bool shrink_shared_fits(int r, int n_shared) { return n_shared == 1 || (n_shared >= 2 && n_shared <= kSharedShrinkMost && r <= 32); }

// Rows per workgroup of the shrink, for the split-K rule.
int shrink_stream_rows(int r, int n_shared) { return 16 * (r * (shrink_shared_fits(r, n_shared) ? n_shared : 1) > 32 ? 8 : 4); }

template <class DT, int R, int P>
static hipError_t launch_shrink_matrix_p(const ShrinkArgs& a, hipStream_t st) {
  using Shape = ShrinkShape<R, P>;
  static_assert(Shape::kLds <= 80 * 1024, "two workgroups per compute unit");
  ShrinkTable tab;
  for (int i = 0; i < kSharedShrinkMost; ++i) {
    const int k = i < a.n_proj ? i : 0;
    tab.x[i] = (const uint16_t*)a.xs[k];
    tab.A_ptrs[i] = (const uint16_t* const*)a.As[k];
    tab.partials[i] = a.partials_of[k];
  }
  const int groups = a.n_proj / P;
  const long long blocks = most_blocks(a.n_tokens, a.n_segs, Shape::kRows);
  const long long wgs = (a.ksplit * blocks + 7) / 8 * 8 * groups;
  const dim3 grid((unsigned)(wgs < kMostWorkgroups ? wgs : kMostWorkgroups), (unsigned)((wgs + kMostWorkgroups - 1) / kMostWorkgroups));
  hipLaunchKernelGGL((shrink_stream_kernel<DT, R, P>), grid, dim3(64 * Shape::kWaves), 0, st, a.seg_starts, a.n_segs,
                     segments_per_block(a.n_segs, blocks), a.ksplit, groups, a.h_in, a.kslice, a.n_tokens, a.layer_off, a.header, tab);
  return hipGetLastError();
}

template <class DT, int R>
static hipError_t launch_shrink_matrix_t(const ShrinkArgs& a, hipStream_t st) {
  if constexpr (R <= 32) {
    if (a.same_x && a.n_proj == 2) return launch_shrink_matrix_p<DT, R, 2>(a, st);
    if (a.same_x && a.n_proj == 3) return launch_shrink_matrix_p<DT, R, 3>(a, st);
  }
  return launch_shrink_matrix_p<DT, R, 1>(a, st);
}

template <class DT>
static hipError_t launch_shrink_matrix_r(const ShrinkArgs& a, hipStream_t st) {
  switch (a.r) {
    case 8: return launch_shrink_matrix_t<DT, 8>(a, st);
    case 16: return launch_shrink_matrix_t<DT, 16>(a, st);
    case 32: return launch_shrink_matrix_t<DT, 32>(a, st);
    case 64: return launch_shrink_matrix_t<DT, 64>(a, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_shrink_matrix(const ShrinkArgs& a, hipStream_t st) {
  if (a.n_proj < 1 || a.n_proj > kSharedShrinkMost) return hipErrorInvalidValue;
  return a.bf16 ? launch_shrink_matrix_r<BF16>(a, st) : launch_shrink_matrix_r<F16>(a, st);
}

// The expands of n add-ons in one launch, in front of it the one that makes operands of their v.
template <class DT, int R>
static hipError_t launch_expand_matrix_t(const ExpandArgs* es, int n, bool direct, hipStream_t st) {
  const ExpandArgs& a = es[0];
  FinalizeTable fin;
  ExpandTable tab;
  for (int i = 0; i < kSharedShrinkMost; ++i) {
    const ExpandArgs& e = es[i < n ? i : 0];
    tab.v_parts[i] = fin.v_parts[i] = e.v_parts;
    tab.vh[i] = fin.vh[i] = e.vh;
    tab.vl[i] = fin.vl[i] = e.vl;
    tab.undo[i] = fin.undo[i] = e.undo;
    tab.y[i] = (uint16_t*)e.y;
    tab.A_ptrs[i] = (const uint16_t* const*)e.A_ptrs;
    tab.B_ptrs[i] = (const uint16_t* const*)e.B_ptrs;
  }
  if (a.three_parts && R != 64) return hipErrorInvalidValue;
  if (!direct) {
    const long long quads = (long long)a.n_tokens * (R / 4);
    const auto finalize = [&](auto parts_tag) {
      hipLaunchKernelGGL((finalize_v_kernel<DT, R, decltype(parts_tag)::value>), dim3((unsigned)((quads + 255) / 256), (unsigned)n),
                         dim3(256), 0, st, a.nparts, a.n_tokens, fin);
    };
    if constexpr (R == 64) {
      if (a.three_parts) finalize(std::integral_constant<int, 3>{});
    }
    if (!a.three_parts) finalize(std::integral_constant<int, 2>{});
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  const int strips = (a.h_out + kExpandCols - 1) / kExpandCols;
  // Strip items only where there can be enough of them: each walks its R weight rows in R / 8 batches of loads, one
  // after the other, so the higher the rank, the more of the chip they have to fill to be ahead of the blocks, which
  // request all of them at once.  Measured, one-row segments, weights from HBM, as strips / as blocks, us: the
  // whole add-on 4096 -> 4096 of 8 of them (16 items) 10.4 / 10.2, 11.2 / 10.2, 13.1 / 9.7 and 19.7 / 13.7 at ranks 8, 16, 32
  // and 64, of 40 (80 items) 12.1 / 13.8, 14.5 / 15.2, 17.3 / 16.3 and 26.8 / 24.3; the expand to 13824 of 40 (280
  // items) 6.5 / 12.6, 8.4 / 13.3, 12.1 / 15.4 and 18.8 / 21.0.
  int few = (a.h_out + kFewCols - 1) / kFewCols;
  const long long items = (long long)a.n_segs * few * n;
  const int few_rows = items < 4 * R ? 0 : R == 8 && items >= 200 ? 4 : 2;
  const long long blocks = most_blocks(a.n_tokens, a.n_segs, kExpandRows);
  const long long wgs = strips * blocks;
  const dim3 grid((unsigned)(wgs < kMostWorkgroups ? wgs : kMostWorkgroups), (unsigned)n,
                  (unsigned)((wgs + kMostWorkgroups - 1) / kMostWorkgroups));
  const auto launch = [&](auto direct_tag, auto parts_tag) {
    hipLaunchKernelGGL((expand_matrix_kernel<DT, R, decltype(direct_tag)::value, decltype(parts_tag)::value>), grid, dim3(256), 0, st, a.seg_starts, a.n_segs,
                       segments_per_block(a.n_segs, blocks), strips, few_rows, few, a.h_out, a.layer_off, a.scale, a.header,
                       tab, a.nparts, a.n_tokens);
  };
  if constexpr (R <= 16) {
    if (direct) {
      launch(std::true_type{}, std::integral_constant<int, 2>{});
      return hipGetLastError();
    }
  }
  if constexpr (R == 64) {
    if (a.three_parts) {
      launch(std::false_type{}, std::integral_constant<int, 3>{});
      return hipGetLastError();
    }
  }
  launch(std::false_type{}, std::integral_constant<int, 2>{});
  return hipGetLastError();
}

template <class DT>
static hipError_t launch_expand_matrix_r(const ExpandArgs* es, int n, bool direct, hipStream_t st) {
  switch (es[0].r) {
    case 8: return launch_expand_matrix_t<DT, 8>(es, n, direct, st);
    case 16: return launch_expand_matrix_t<DT, 16>(es, n, direct, st);
    case 32: return launch_expand_matrix_t<DT, 32>(es, n, direct, st);
    case 64: return launch_expand_matrix_t<DT, 64>(es, n, direct, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_expand_matrix(const ExpandArgs* es, int n, bool direct, hipStream_t st) {
  if (n < 1 || n > kSharedShrinkMost || (direct && es[0].r > 16)) return hipErrorInvalidValue;
  return es[0].bf16 ? launch_expand_matrix_r<BF16>(es, n, direct, st) : launch_expand_matrix_r<F16>(es, n, direct, st);
}

}  // namespace sgmv
