// Chunked prefill attention over a cached prefix.
//
// "Compute Analysis": chunked prefill is largely compute-bound, and an SWA
// layer only needs the keys inside its window, so tiles outside the window are
// never visited. Keys below the prefix length P come from the paged cache (FULL:
// the block table; SWA: the ring), keys from P on come from the chunk's own
// k_new / v_new (the chunk is appended to the cache only after this kernel).
//
// Work unit: one workgroup (8 waves, two per SIMD) per (tile of 256 query rows,
// KV head, sequence). A query row is a (position, query head) pair of the KV
// head's GQA group, so one K/V tile in LDS serves every query head that shares
// it. Each wave owns 32 rows (two 16-column MFMA groups). Per 64-key tile:
//   S^T[key][row]  = K[key][:] . Q[row][:]          (bf16 MFMA, fp32 accumulate)
//   online softmax per row in fp32 (exp2, scale*log2(e) folded in); the running
//   maximum is only raised when a score exceeds it by more than 2^8 in exp2
//   units, so the output rescale is rare (exact: numerator and denominator share
//   the stale maximum)
//   O^T[d][row]   += V^T[d][key] . P^T[key][row]    (bf16 MFMA)
// The two waves of a SIMD play ping-pong: while one runs its matrix products
// (QK^T of one tile, PV of the previous one) the other runs its softmax and
// stages tiles, and workgroup barriers swap the roles, so the matrix cores and
// the vector ALUs work at the same time.
// LDS holds the tiles in MFMA operand order (every operand read is one
// contiguous, conflict-free 1 KiB); four tile buffers let two tiles be read
// while a third is stored, and the global loads of a fourth are in flight.
// Keys outside the workgroup's range are staged as zeros, so NaN or stale data
// in unused cache slots never reaches an accumulator; per-element masks are
// applied only on tiles that cross the causal diagonal, the window edge or the
// range ends. Workgroups are mapped so that each XCD works through the query
// tiles of a few (sequence, KV head) pairs at a time and shares their K/V in L2.
// A call with few tiles (or few in its last round) leaves compute units idle:
// given a workspace, its key tiles are cut into equal spans instead, one per
// workgroup, and prefill_merge_kernel combines the pieces of a tile (295 tokens
// over 22.5K cached, 80 tiles: 498 -> 209 us). Whether that gains depends on the
// lengths, which only the device has: the host rules calls out by what the block
// table can hold, and the kernel decides (split_gains); where it does not gain
// the kernel works as the unsplit one. A span walks its tiles in a loop
// around the same code; what the tile loop does not need is kept out of its
// registers (walk state in LDS, parameters and lane addresses formed anew per
// tile), which a plain loop spilled at +5% per key tile.
#include <algorithm>
#include <cfloat>
#include <climits>
#include <cmath>
#include <type_traits>

#include "hswa_common.h"
#include "hswa_launch.h"

namespace hswa {
namespace {

constexpr int kThreads = 512;
constexpr int kKT = 64;     // keys per tile
constexpr int kXcds = 8;
constexpr int kBufs = 4;  // LDS tile buffers (a power of two): two being read, one stored, one loading
static_assert((kBufs & (kBufs - 1)) == 0, "buffer indices are taken modulo kBufs with a mask");
// a lane's share (16 probabilities) of a row sum above which the running
// maximum is raised
constexpr float kLaneSumLimit = 4096.f;
constexpr int kSplitSpans = 256;  // spans of the split order: one workgroup per CU
constexpr int kTileCost = 5;      // what a query tile costs besides its key tiles, in key tiles
constexpr int kSplitGain = 14;    // key tiles a split has to gain (its partials, their merge, its own order)
constexpr int kCutCost = 13;      // the same once its kernels are launched
constexpr int kMinSpan = 8;       // least worth of a span
// LDS operand reads in flight ahead of the matrix products (8: +0.6%, 10: +1.6%,
// 6: +0.3% on 4 x 2048 over 8192)
constexpr int kAhead = 4;
// LDS holds each tile in MFMA operand order: every operand a wave reads (K: 16
// keys x 32 dims of a QK^T step; V^T: 16 dims x 32 keys of a PV step) is a
// contiguous 1 KiB block with lane l's 16 bytes at 16 l, so each operand read
// is one conflict-free ds_read_b128 at a per-lane base plus a constant.
//   K tile: block (h, ab, t) at ((2 h + ab) * 4 + t) KiB holds, for lane
//     r + 16 q, dims 32 t + 8 q .. +7 of tile key 32 h + 8 (r >> 2) + 4 ab + (r & 3):
//     MFMA row r of the QK^T step of half h, block ab, dim slab t. This is the
//     pool's K block layout, so an interior tile is a straight copy.
//   V^T tile: block (h, dt) at 16 KiB + (8 h + dt) KiB holds, for lane r + 16 q,
//     keys 32 h + 8 q .. +7 of dim 16 dt + r.
constexpr int kKTileBytes = kKT * kHeadDim * 2;
// Fourth word of a gfx9 buffer resource for raw (untyped) loads: 32-bit data
// format, no swizzle, no index stride.
constexpr int kBufferWord3 = 0x00020000;
constexpr int kBufBytes = 2 * kKTileBytes;

// LDS byte offset (within a buffer) of keys 32 h + 8 q .. +7 of dim d (V^T).
__device__ __forceinline__ uint32_t v_lds_off(int h, int q, int d) {
  return (uint32_t)(kKTileBytes + ((8 * h + (d >> 4)) * 64 + (d & 15) + 16 * q) * 16);
}

constexpr int kStage = kKT * kHeadDim / 8 / kThreads;  // 16-byte pieces per thread per tile (K or V)
static_assert(kStage == 2 && kKT == 64, "V staging maps piece i of a thread to 32-key block i");

// Staging maps every wave's 16-byte LDS stores onto one contiguous 1 KiB
// operand block (lane l at 16 l), so the stores are free of bank conflicts;
// thread tid (lane l of wave w) stores piece i at byte 16 tid + 8 KiB i of the
// K tile and of the V^T tile.
// V^T piece i of thread tid: dim 16 w + l % 16, keys 8 (4 i + l / 16) .. +7 of
// the tile, i.e. piece l / 16 of dim row 16 w + l % 16 of the pool's 32-key V
// block i (a wave reads one contiguous 1 KiB of the block).
// K tile pieces in pool order: piece idx (0 .. 1023) is 16-byte piece idx & 511
// of the tile's 32-key block idx >> 9 (half (idx >> 8) & 1, slab (idx >> 6) & 3,
// dim piece (idx >> 4) & 3, row idx & 15 of the block's K layout). LDS holds it
// at byte 16 idx.
__device__ __forceinline__ int v_piece_dim(int tid) { return 16 * (tid >> 6) + (tid & 15); }

struct Stage {
  u32x4 k[kStage], v[kStage];
  bool vrow;  // chunk tile: k[] holds key rows, v[] pieces follow the chunk mapping
};

// Valid tokens of sequence b (never past q / k_new / v_new / out, whatever the
// device offsets say; none for offsets out of range).
template <typename Params>
__device__ __forceinline__ int chunk_len(const Params &p, int b) {
  const int tok = p.cu_seqlens[b];
  const int n = min(min(p.cu_seqlens[b + 1], p.total_tokens) - tok, p.max_chunk_len);
  return tok < 0 || p.prefix_lens[b] < 0 ? 0 : n;
}
// Key tiles of query tile t (npos positions) of a sequence with chunk length c
// and prefix length pre, under window w (0: none).
__device__ __forceinline__ int key_tiles(int t, int npos, int c, int pre, int w) {
  const int last = min(c, (t + 1) * npos) - 1;  // its last position, from pre on
  if (t * npos > last) return 0;
  const int lo = w > 0 ? max(0, pre + t * npos - w + 1) : 0;
  const int cached = lo < pre ? ((pre - 1) >> 6) - (lo >> 6) + 1 : 0;
  return cached + (last >> 6) - ((max(lo, pre) - pre) >> 6) + 1;
}

// A workgroup's place in the split order (kept in LDS: the tile loop leaves no
// scalar registers for it).
struct Walk {
  int64_t one;    // worth of the query tiles of one KV head
  int64_t per;    // worth of a span
  int64_t u0;     // this span's start
  int64_t u, u1;  // its rest [u, u1)
  int64_t next;   // where the query tile at u ends (u1 if the span ends in it)
};

// Inclusive scan over the wave's lanes with `op` (`none`: its identity) by data
// movement inside the vector ALU; lane 63 ends up with the result of all lanes.
template <int kCtrl, int kRows, typename T>
__device__ __forceinline__ T lane_move(T none, T x) {
  if constexpr (sizeof(T) == 8) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x), o = __builtin_bit_cast(uint64_t, none);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)o, (int)u, kCtrl, kRows, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(o >> 32), (int)(u >> 32), kCtrl, kRows, 0xf, false);
    return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
  } else {
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, none), __builtin_bit_cast(int, x),
                                                             kCtrl, kRows, 0xf, false));
  }
}
template <typename T, typename Op>
__device__ __forceinline__ T wave_scan(T x, T none, Op op) {
  x = op(x, lane_move<0x111, 0xf>(none, x));  // from 1, 2, 4, 8 lanes down in a row of 16
  x = op(x, lane_move<0x112, 0xf>(none, x));
  x = op(x, lane_move<0x114, 0xf>(none, x));
  x = op(x, lane_move<0x118, 0xf>(none, x));
  x = op(x, lane_move<0x142, 0xa>(none, x));  // a row's last lane to the next row (rows 1 and 3)
  x = op(x, lane_move<0x143, 0xc>(none, x));  // lane 31 to the upper rows
  return x;
}
__device__ __forceinline__ float last_lane(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), kWave - 1));
}

// Whether cutting the call into spans gains, by its lengths (lane b holds
// sequence b; every wave finds it by itself). In key tiles, a query tile worth
// its key tiles plus kTileCost, the unsplit call takes the largest of: the load
// of the fullest XCD (sequences taken as alike); its rounds of the shortest
// tiles; and, for a sequence whose last (sequence, KV head) pair comes after
// others on its XCD, the time until a compute unit is free for it and then its
// longest tile. Each round also takes this decision anew (about 1.3 us, a
// unit), and the merge is launched either way. The split one takes the average
// over all compute units and kCutCost. us per call unsplit by hswa_prefill / whole
// tiles here / cut, with the gain by this rule and the 13 it is held against (the
// block table 128K positions wide, 64 / 8 heads, except where other heads are given):
//   300 tokens over none             16.9 / 20.2 / -       3
//   600 over none                    24.5 / 28.2 / 34.5    8
//   1500 over none                   48.0 / 52.5 / 66.3    5
//   4 x 600 over none                47.2 / 52.8 / 60.3    6
//   8 x 64 over 1000                 34.4 / 38.4 / 40.0   12
//   1000 over none, 16 / 16          35.9 / 40.0 / 36.6   14
//   20 - 780 over 100, 20 of them,
//     PG 16, 32 / 8                 106.7 / 116.6 / 107.7  13.5
//   64 over 1000                     32.6 /  -   / 30.6   15
//   446 - 1471 over 463 - 2957,
//     4 of them, PG 16, 32 / 8      139   /  -   / 119    33
//   600 over 4000                   111   /  -   / 95.7   35
//   295 over 22.5K                  494   /  -   / 212   250
// A table as wide as the context is long takes the same decisions. (By table
// width alone 600 and 1500 tokens over none were cut: 34.5 and 66.3 us.)
__device__ __forceinline__ bool split_gains(const PrefillParams &p, int npos, int lane) {
  constexpr float kXcdCus = kSplitSpans / kXcds;
  const auto add = [](float a, float b) { return a + b; };
  const auto most = [](float a, float b) { return fmaxf(a, b); };
  const auto least = [](float a, float b) { return fminf(a, b); };
  const float heads = (float)p.hkv * (1.f / kXcds), others = fmaxf(heads - 1.f, 0.f);  // pairs of a sequence on an XCD
  float count = 0.f, sum = 0.f, late = 0.f, shortest = FLT_MAX;
  for (int b0 = 0; b0 < p.ns; b0 += kWave) {
    const int b = b0 + lane;
    const int c = b < p.ns ? chunk_len(p, b) : 0;
    float n = 0.f, s = 0.f, first = 0.f, longest = 0.f;  // query tiles, their worth, the first's and the last's
    if (c > 0) {
      const int pre = p.prefix_lens[b];
      const int cached = kTileCost + (pre > 0 ? ((pre - 1) >> 6) + 1 : 0);
      n = (float)((c + npos - 1) >> __builtin_ctz(npos));  // (npos is a power of two)
      first = (float)(cached + ((min(npos, c) - 1) >> 6) + 1);
      longest = (float)(cached + ((c - 1) >> 6) + 1);
      s = n * .5f * (first + longest);
    }
    const float cn = wave_scan(n, 0.f, add), cs = wave_scan(s, 0.f, add);
    const float bn = heads * (count + cn - n) + others * n, bs = heads * (sum + cs - s) + others * s;  // before the last pair
    if (c > 0) {
      late = fmaxf(late, longest + (bn >= kXcdCus ? bs * (1.f / kXcdCus - .5f * __builtin_amdgcn_rcpf(bn)) : 0.f));
      shortest = fminf(shortest, first);
    }
    count += last_lane(cn);
    sum += last_lane(cs);
  }
  late = last_lane(wave_scan(late, 0.f, most));
  shortest = last_lane(wave_scan(shortest, FLT_MAX, least));
  const float share = (float)((p.ns * p.hkv + kXcds - 1) / kXcds) * __builtin_amdgcn_rcpf((float)p.ns * kXcdCus);
  const float unsplit = fmaxf(late, fmaxf(sum * share, ceilf(count * share) * shortest));
  const float rounds = ceilf(count * (float)p.hkv * (1.f / kSplitSpans));
  const float spans = fmaxf((float)kMinSpan, sum * (float)p.hkv * (1.f / kSplitSpans));
  return __builtin_amdgcn_readfirstlane((int)(count > 0.f && unsplit + rounds - spans >= (float)kCutCost)) != 0;
}

typedef __attribute__((address_space(4))) const PrefillParams KernArgs;

// LDS of a workgroup: kBufs tile buffers, each a K tile then a V^T tile (byte
// offsets below).
struct __attribute__((aligned(16))) TileBufs {
  unsigned char b[kBufs * kBufBytes];
};
// And of a span: key tiles up to and including each (sequence, query tile) of
// one KV head, their per-wave parts, the walk, the current query tile.
struct SpanLds {
  int64_t cum[kThreads], wave[kThreads / kWave];
  Walk walk;
  int tile[3];
};

// One query tile (tq of sequence b, KV head g), or with kSplit the query tiles
// of a span. kCG: 16-column MFMA groups per wave, 128 kCG query rows per
// workgroup. kPage: keys of a page, 64 standing for 64 and more.
template <int kCG, int kPage, bool kSplit>
__device__ __forceinline__ void prefill_tiles(const PrefillParams &p0, TileBufs &bufs, [[maybe_unused]] SpanLds *sl,
                                              [[maybe_unused]] int span, int b, int g, int tq) {
  constexpr int kRows = 8 * 16 * kCG;
  unsigned char *const s_lds = bufs.b;
  for (;;) {
  int tid = threadIdx.x;
  // opaque, so that the lane addresses below are formed anew for each query
  // tile and not kept (and spilled) across them
  if constexpr (kSplit) asm volatile("" : "+v"(tid));
  // likewise the parameters: read again from the kernel's argument segment
  const KernArgs *args = (const KernArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if constexpr (kSplit) asm volatile("" : "+s"(args));
  const auto &p = [&]() -> const auto & {
    if constexpr (kSplit) return *args;
    else return p0;
  }();
  const auto &pv = p.pool;
  const int G = p.group;
  const int npos = kRows / G;  // positions per workgroup
  const int ntq = (p.max_chunk_len + npos - 1) / npos;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);  // uniform in a wave
  const int r = lane & 15, q = lane >> 4;
  const int hkv = p.hkv, hq = p.hq;
  const int shift = pv.pg_shift, pg = 1 << shift;
  const float c2 = p.scale_log2;

  int j0 = 0, j1 = INT_MAX;  // key tiles [j0, j1) of the query tile
  if constexpr (kSplit) {
    // the query tile that holds unit u
    __syncthreads();
    const int64_t gl = sl->walk.u / sl->walk.one;
    const int64_t rem = sl->walk.u - gl * sl->walk.one;
    const int64_t lo = tid > 0 ? sl->cum[tid - 1] : 0, hi = sl->cum[tid];
    if (lo <= rem && rem < hi) {
      sl->tile[0] = tid;
      const int64_t left = min(hi - rem, sl->walk.u1 - sl->walk.u);
      sl->tile[1] = (int)max((int64_t)0, rem - lo - kTileCost);
      sl->tile[2] = (int)(rem + left - lo - kTileCost);
      sl->walk.next = sl->walk.u + left;
    }
    __syncthreads();
    g = __builtin_amdgcn_readfirstlane((int)gl);
    const int tile = __builtin_amdgcn_readfirstlane(sl->tile[0]);
    b = tile / ntq;
    tq = tile - b * ntq;
    j0 = __builtin_amdgcn_readfirstlane(sl->tile[1]);
    j1 = __builtin_amdgcn_readfirstlane(sl->tile[2]);
    if (j1 <= 0) {  // the span ends before the tile's first key tile
      if (tid == 0 && sl->walk.u == sl->walk.u0) p.ws_desc[span].pieces = 0;
      return;
    }
  }

  const int tok0 = p.cu_seqlens[b];
  const int C = chunk_len(p, b);
  const int P = p.prefix_lens[b];
  const int q0 = tq * npos;
  const int q1 = min(C, q0 + npos) - 1;
  const int pfirst = P + q0, plast = P + q1;
  const int W = pv.window;
  const int klo = W > 0 ? max(0, pfirst - W + 1) : 0;
  const int khi = plast;

  // Q^T operands and the position of each of this lane's columns.
  u32x4 qf[kCG][4];
  int cpos[kCG], clo[kCG];
  bool cval[kCG];
#pragma unroll
  for (int cg = 0; cg < kCG; ++cg) {
    const int row = wave * (16 * kCG) + cg * 16 + r;
    const int po = row / G, head = row - po * G;
    cval[cg] = q0 + po <= q1;
    cpos[cg] = P + q0 + po;
    clo[cg] = W > 0 ? max(0, cpos[cg] - W + 1) : 0;
    const int64_t tok = tok0 + q0 + (cval[cg] ? po : 0);
    const uint16_t *qrow = p.q + (tok * hq + (int64_t)g * G + head) * kHeadDim;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const u32x4 v = ldg128(qrow + 32 * t + 8 * q);
      const u32x4 z = {0u, 0u, 0u, 0u};
      qf[cg][t] = cval[cg] ? v : z;
    }
  }

  // ---- the key range in tiles ----
  // Cut at P: tiles of cached keys, aligned to 64 absolute positions (so that a
  // tile is whole pool blocks), then tiles of the chunk's own keys, aligned to
  // P. No tile holds both kinds; a tile at an end of its range is partly masked.
  const int nlo = max(klo, P);  // first new key in range
  const int nall = key_tiles(tq, npos, C, P, W);
  // this workgroup's tiles, numbered from j0 on (ncached <= 0: no cached one)
  const int ntiles = kSplit ? min(j1, nall) - j0 : nall;
  const int ncached = (klo < P ? ((P - 1) >> 6) - (klo >> 6) + 1 : 0) - j0;
  const int kt0 = (klo & ~(kKT - 1)) + kKT * j0;
  const int ktn = P + ((nlo - P) & ~(kKT - 1)) - kKT * ncached;  // tile j >= ncached starts at ktn + 64 j
  auto tile_key = [&](int j) { return kKT * j + (j < ncached ? kt0 : ktn); };

  // ---- staging: global -> registers -> LDS ----
  // Chunk tile: every key is one of this chunk's own (key >= P). K and V rows
  // are 256-byte runs of k_new / v_new, loaded as 16-byte pieces of a row. K
  // piece i of lane l of wave w is MFMA row l % 16 of K block (h = i,
  // ab = w / 4, slab w % 4), dims 32 (w % 4) + 8 (l / 16) .. +7, so it lands at
  // the same LDS byte as a pool piece. V piece i of lane l of wave w is key
  // 8 w + 4 i + l / 16, dims 8 (l % 16) .. +7; the store transposes those into
  // V^T (store_tile).
  auto load_tile_chunk = [&](int kt, Stage &st) __attribute__((always_inline)) {
    const u32x4 z = {0u, 0u, 0u, 0u};
    const int r = lane & 15, ab = wave >> 2;
#pragma unroll
    for (int i = 0; i < kStage; ++i) {
      const int j = kt + 32 * i + 8 * (r >> 2) + 4 * ab + (r & 3);
      const bool in = j >= nlo && j <= khi;
      const int c = 4 * (wave & 3) + (lane >> 4);
      const int64_t off = ((int64_t)(tok0 + (in ? j - P : 0)) * hkv + g) * kHeadDim + c * 8;
      st.k[i] = in ? ldg128(p.k_new + off) : z;
    }
#pragma unroll
    for (int i = 0; i < kStage; ++i) {
      const int j = kt + 8 * wave + 4 * i + (lane >> 4);
      const bool in = j >= nlo && j <= khi;
      const int64_t off = ((int64_t)(tok0 + (in ? j - P : 0)) * hkv + g) * kHeadDim + (lane & 15) * 8;
      st.v[i] = in ? ldg128(p.v_new + off) : z;
    }
    st.vrow = true;
  };
  // Full chunk tile: every key is the chunk's own and inside [klo, khi]. The
  // tile's 64 rows of k_new / v_new start at a wave-uniform address and each
  // lane's pieces sit at fixed byte offsets from it (rows of Hkv D 2 bytes), so
  // the loads are buffer loads from a scalar resource with those offsets: no
  // per-tile vector address arithmetic and no per-lane range checks.
  const uint32_t row_bytes = (uint32_t)hkv * (kHeadDim * 2);
  const bool chunk_buf = (uint64_t)hkv * (kHeadDim * 2) * kKT <= 0x7fffffffull;
  uint32_t ch_koff[kStage], ch_voff[kStage];
  {
    const int r = lane & 15, ab = wave >> 2, c = 4 * (wave & 3) + (lane >> 4);
#pragma unroll
    for (int i = 0; i < kStage; ++i) {
      ch_koff[i] = (uint32_t)(32 * i + 8 * (r >> 2) + 4 * ab + (r & 3)) * row_bytes + (uint32_t)c * 16u;
      ch_voff[i] = (uint32_t)(8 * wave + 4 * i + (lane >> 4)) * row_bytes + (uint32_t)(lane & 15) * 16u;
    }
  }
  auto load_tile_chunk_full = [&](int kt, Stage &st) __attribute__((always_inline)) {
    const int64_t row0 = ((int64_t)(tok0 + kt - P) * hkv + g) * kHeadDim;
    const __amdgpu_buffer_rsrc_t krs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.k_new + row0), 0, kKT * row_bytes, kBufferWord3);
    const __amdgpu_buffer_rsrc_t vrs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.v_new + row0), 0, kKT * row_bytes, kBufferWord3);
#pragma unroll
    for (int i = 0; i < kStage; ++i) {
      st.k[i] = __builtin_amdgcn_raw_buffer_load_b128(krs, (int)ch_koff[i], 0, 0);
      st.v[i] = __builtin_amdgcn_raw_buffer_load_b128(vrs, (int)ch_voff[i], 0, 0);
    }
    st.vrow = true;
  };
  // Page ids of cached tiles come from a per-wave window of the block table:
  // lane i holds the entry of logical page tab_lp0 + i, and a tile's ids are
  // read with v_readlane. The next window is loaded when one is entered, 16 to
  // 64 tiles before its first use, so no tile waits for the table. (Entries are
  // checked where they are used; -1 past the cached pages.)
  int tab_page = -1, tab_next = -1, tab_lp0 = kt0 >> shift;
  auto load_tab = [&](int lp0) {
    const int lp = lp0 + lane;
    int v = -1;
    if (lp <= ((P - 1) >> shift) && P > 0) {
      const int e = pv.ring > 0 ? lp % pv.ring : lp;
      if (e < pv.stride) v = pv.table[(int64_t)b * pv.stride + e];
    }
    return v;
  };
  if (ncached > 0) {
    tab_page = load_tab(tab_lp0);
    tab_next = load_tab(tab_lp0 + kWave);
  }
  auto page_at = [&](int lp) {  // -1: not a valid page
    const int v = __builtin_amdgcn_readlane(tab_page, lp - tab_lp0);
    return v >= 0 && v < pv.num_pages ? v : -1;
  };
  // Cached tile: the K tile is two 8 KiB K blocks and the V tile two [D][32]
  // blocks of 8 KiB (16-key pages: four 4 KiB blocks each), contiguous in the
  // pools. The base addresses are wave-uniform (scalar registers) and each load
  // adds a fixed 32-bit per-lane byte offset (buffer loads), so a tile's loads
  // need no vector address arithmetic; with 16-key pages a lane chooses one of
  // a block's two pages (three vector instructions a load). Looking a page up
  // per key instead, with 2-byte V loads where a piece crossed a range end, took
  // a PG 16 call of 4 ragged chunks (3263 tokens over 463-2957 cached, 32 / 8
  // heads) 232 us against 150, and 4 x 2048 over 8192 (64 / 8) 3239 against
  // 2104 (1965 with PG 64).
  // (The empty asm keeps the offsets opaque: the compiler would otherwise fold
  // the constant 8 KiB step between a thread's two pieces into arithmetic of
  // its own.)
  constexpr int kPages = kKT / kPage;  // pages of a tile
  const int vq = (tid >> 4) & 3;       // V^T piece: keys 8 vq .. +7 of its 32-key block
  uint32_t pg_koff[kStage], pg_voff[kStage];
#pragma unroll
  for (int i = 0; i < kStage; ++i) {
    if constexpr (kPage == 16) {
      pg_koff[i] = (uint32_t)((tid >> 4) * 128 + (tid & 7) * 16);  // 8-row slabs
      pg_voff[i] = (uint32_t)(v_piece_dim(tid) * 32 + (vq & 1) * 16);
    } else {
      const uint32_t blk = kPage == 32 ? 0u : 8192u * i;  // PG >= 64: both blocks from one base
      pg_koff[i] = blk + (uint32_t)tid * 16u;
      pg_voff[i] = blk + (uint32_t)(v_piece_dim(tid) * 32 + vq * 8) * 2u;
    }
    asm volatile("" : "+v"(pg_koff[i]), "+v"(pg_voff[i]));
  }
  // Both pools put a page-head at the same byte offset, page * (Hkv PG D 2) +
  // g * (PG D 2), and its 32-key blocks 8 KiB apart: one scalar offset serves
  // the K and the V loads.
  const uint32_t page_bytes = (uint32_t)hkv << (shift + kHeadDimShift + 1);
  const uint64_t head_bytes = (uint64_t)g << (shift + kHeadDimShift + 1);
  auto page_off = [&](int kt, int page) {
    uint64_t o = (uint64_t)(uint32_t)max(page, 0) * page_bytes + head_bytes;
    if constexpr (kPage == 64) o += (uint64_t)(((uint32_t)kt & (uint32_t)(pg - 1)) >> 5) * 8192u;
    return o;
  };
  auto buf_load = [&](uint16_t *pool, uint64_t o, int bytes, uint32_t off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
        __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char *>(pool) + o, 0, bytes, kBufferWord3), (int)off, 0, 0));
  };
  auto load_tile_cached = [&](int kt, Stage &st) __attribute__((always_inline)) {
    const int lp = kt >> shift;
    if (lp - tab_lp0 >= kWave) {
      tab_lp0 += kWave;
      tab_page = tab_next;
      tab_next = load_tab(tab_lp0 + kWave);
    }
    int page[kPages];
    bool whole = kt >= klo && kt + kKT <= P;
#pragma unroll
    for (int n = 0; n < kPages; ++n) {
      page[n] = page_at(lp + n);
      whole = whole && page[n] >= 0;
    }
    st.vrow = false;
    // 16-key pages: the page of this lane's K rows (8 (r >> 3) ..) and V keys
    const bool ksel = kPage == 16 && (tid & 8), vsel = kPage == 16 && (vq & 2);
    if (whole) {
#pragma unroll
      for (int i = 0; i < kStage; ++i) {
        if constexpr (kPage == 16) {
          const uint64_t o0 = page_off(kt, page[2 * i]), o1 = page_off(kt, page[2 * i + 1]);
          st.k[i] = ldg128_global(reinterpret_cast<const char *>(pv.k_pool) + (ksel ? o1 : o0) + pg_koff[i]);
          st.v[i] = ldg128_global(reinterpret_cast<const char *>(pv.v_pool) + (vsel ? o1 : o0) + pg_voff[i]);
        } else {
          const uint64_t o = page_off(kt, page[kPage == 32 ? i : 0]);
          st.k[i] = buf_load(pv.k_pool, o, kKTileBytes, pg_koff[i]);
          st.v[i] = buf_load(pv.v_pool, o, kKTileBytes, pg_voff[i]);
        }
      }
      return;
    }
    // A tile that crosses an end of the cached range (its out-of-range V is
    // zeroed: those slots may hold anything, NaN included, and meet probability
    // 0; their K only reaches masked scores) or meets an invalid page (a zero
    // key and value).
#pragma unroll
    for (int i = 0; i < kStage; ++i) {
      const int n0 = kPage == 16 ? 2 * i : kPage == 32 ? i : 0, n1 = kPage == 16 ? 2 * i + 1 : n0;
      const int kpage = ksel ? page[n1] : page[n0], vpage = vsel ? page[n1] : page[n0];
      u32x4 k = {0u, 0u, 0u, 0u}, v = k;
      if (kpage >= 0) k = ldg128(reinterpret_cast<const char *>(pv.k_pool) + page_off(kt, kpage) + pg_koff[i]);
      if (vpage >= 0) v = ldg128(reinterpret_cast<const char *>(pv.v_pool) + page_off(kt, vpage) + pg_voff[i]);
      st.k[i] = k;
      st.v[i] = keep_bf16x8(v, key_range_bits(kt + 32 * i + 8 * vq, klo, P - 1));
    }
  };
  // LDS addresses are a per-lane byte offset (fixed for the kernel) plus the
  // buffer's byte offset (a scalar), with everything else in the instruction's
  // immediate offset field.
  auto buf_off = [&](int buf) { return (uint32_t)__builtin_amdgcn_readfirstlane(buf * kBufBytes); };
  auto lds128 = [&](uint32_t off) { return reinterpret_cast<u32x4 *>(s_lds + off); };
  // LDS offsets of this thread's pieces: piece 1 is 8 KiB after piece 0, except
  // for the V^T pieces of a chunk tile, dims 8 (l % 16) + 2 m and + 1
  // (m = l / 16) of keys 8 w .. +7, which are 16 bytes apart.
  const uint32_t st_k0 = tid * 16;
  const uint32_t st_v0 = kKTileBytes + tid * 16;
  const uint32_t st_vrow0 = v_lds_off(wave >> 2, wave & 3, 8 * (lane & 15) + 2 * (lane >> 4));
  // 4 x 4 transpose of dwords across the lanes l, l ^ 16, l ^ 32, l ^ 48: the
  // lane in 16-lane row m enters with dword j of its row m in t[j] and leaves
  // with dword m of rows 0..3 in w[0..3] (a swap with l ^ 32, then with l ^ 16).
  auto transpose4 = [&](const u32x4 &t, uint32_t (&w)[4]) {
    const auto a = __builtin_amdgcn_permlane32_swap(t[0], t[2], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(t[1], t[3], false, false);
    const auto c = __builtin_amdgcn_permlane16_swap((uint32_t)a[0], (uint32_t)b[0], false, false);
    const auto d = __builtin_amdgcn_permlane16_swap((uint32_t)a[1], (uint32_t)b[1], false, false);
    w[0] = (uint32_t)c[0];
    w[1] = (uint32_t)c[1];
    w[2] = (uint32_t)d[0];
    w[3] = (uint32_t)d[1];
  };
  auto store_tile = [&](int buf, Stage &st) __attribute__((always_inline)) {
    static_assert(kStage == 2, "two pieces per thread");
    const uint32_t bo = buf_off(buf);
    *lds128(bo + st_k0) = st.k[0];
    *lds128(bo + st_k0 + kKTileBytes / 2) = st.k[1];
    if (st.vrow) {
      // The lanes l % 16 + 16 m (m = 0..3) of a wave hold an 8 x 8 block: keys
      // 8 w + 4 i + m (piece i) x dims 8 (l % 16) .. +7. After the transposes
      // lane m holds dims 2 m, 2 m + 1 of keys 8 w .. +7 (w[k]); byte permutes
      // split them into one V^T piece per dim, which replace the pieces in
      // place (so both kinds of tile store the same registers and the stores
      // need no copies).
      uint32_t w[8];
      transpose4(st.v[0], *reinterpret_cast<uint32_t(*)[4]>(&w[0]));
      transpose4(st.v[1], *reinterpret_cast<uint32_t(*)[4]>(&w[4]));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        st.v[0][j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x05040100u);
        st.v[1][j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x07060302u);
      }
    }
    // V^T pieces: a pool tile's two pieces sit 8 KiB apart at st_v0, a chunk
    // tile's 16 bytes apart at st_vrow0
    const uint32_t va = bo + (st.vrow ? st_vrow0 : st_v0);
    *lds128(va) = st.v[0];
    *lds128(va + (uint32_t)__builtin_amdgcn_readfirstlane(st.vrow ? 16 : kKTileBytes / 2)) = st.v[1];
  };

  float m[kCG], lsum[kCG];  // m: running maximum in exp2 units
  f32x4 acc[kCG][8];
#pragma unroll
  for (int cg = 0; cg < kCG; ++cg) {
    m[cg] = -FLT_MAX;
    lsum[cg] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[cg][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  auto fetch = [&](int j, Stage &st) __attribute__((always_inline)) {
    const int kt = tile_key(j);
    if (j < ncached) load_tile_cached(kt, st);
    else if (chunk_buf && kt >= nlo && kt + kKT - 1 <= khi) load_tile_chunk_full(kt, st);
    else load_tile_chunk(kt, st);
  };

  // QK^T of one half tile: S^T for keys kt + 32h .. +31.
  const uint32_t op_lane = lane * 16;
  auto qk_half = [&](int buf, int h, f32x4 (&sc)[2][kCG]) {
    const uint32_t a = buf_off(buf) + op_lane + h * (kKTileBytes / 2);
#pragma unroll
    for (int cg = 0; cg < kCG; ++cg) {
      sc[0][cg] = f32x4{0.f, 0.f, 0.f, 0.f};
      sc[1][cg] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const u32x4 ka = *lds128(a + 1024 * t);
      const u32x4 kb = *lds128(a + 4096 + 1024 * t);
#pragma unroll
      for (int cg = 0; cg < kCG; ++cg) {
        sc[0][cg] = mfma16x16x32(ka, qf[cg][t], sc[0][cg]);
        sc[1][cg] = mfma16x16x32(kb, qf[cg][t], sc[1][cg]);
      }
    }
  };
  // Per-element mask of a half tile on the diagonal, window edge or range ends
  // (kend: the last key of the tile's kind, P - 1 or khi).
  auto mask_half = [&](int kt, int kend, int h, f32x4 (&sc)[2][kCG]) {
    // this lane's 8 keys are kt + 32h + 8q + e, e = 4 ab + i; allowed e form
    // the interval [lo_e, hi_e] of the column's visible keys
    // kt laundered: the per-lane bounds below are then formed here, in the
    // masked tiles only, not carried through the loop as vector induction
    // variables that every tile would update
    int ktl = kt;
    asm volatile("" : "+s"(ktl));
    const int j0 = ktl + 32 * h + 8 * q;
#pragma unroll
    for (int cg = 0; cg < kCG; ++cg) {
      const int lo_e = max(clo[cg] - j0, 0);
      const int hi_e = min(min(cpos[cg], kend) - j0, 7);
      const uint32_t bits = hi_e < lo_e ? 0u : ((2u << hi_e) - 1u) & ~((1u << lo_e) - 1u);
#pragma unroll
      for (int ab = 0; ab < 2; ++ab)
#pragma unroll
        for (int i = 0; i < 4; ++i) sc[ab][cg][i] = (bits >> (4 * ab + i)) & 1u ? sc[ab][cg][i] : -INFINITY;
    }
  };
  auto needs_mask = [&](int j, int kt) {
    return kt + kKT > (j < ncached ? P : pfirst + 1) || (W > 0 && kt < plast - W + 1);
  };
  // Lazy raise of the running maximum, checked after the fact. The
  // exponentials of a tile are taken against the running maximum m as it
  // stands, and each lane adds up its 16 probabilities of a column (its share
  // of the row sum). Only if some lane's share exceeds 2^12 (a ballot; an
  // infinite sum counts) is the exact column maximum formed across the 4 lanes
  // that share a column, m raised to it, the output and the row sum rescaled,
  // and the tile's exponentials taken again. Otherwise every probability is
  // below 2^12 and m stays: the result is the same either way, because
  // numerator and denominator share m, and the 2^12 bound keeps both far
  // inside the fp32 and bf16 ranges. The running maximum is kept in exp2
  // units (score * scale * log2 e) and starts at -FLT_MAX, a finite value
  // whatever the scale: exp2 of a masked score (-inf) is then 0 with no NaN
  // from (-inf) - (-inf), and the first finite score always raises it (its
  // probability overflows to infinity; alpha = exp2(-huge) = 0).
  // The exponentials give the bf16 P^T operands; the row sums use the same
  // bf16-rounded probabilities as the PV product.
  auto tile_exp = [&](f32x4 (&sc)[2][2][kCG], u32x4 (&pf)[2][kCG], float (&ts)[kCG]) {
#pragma unroll
    for (int cg = 0; cg < kCG; ++cg) {
      const float mc = m[cg];
      ts[cg] = 0.f;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float pr[8];
#pragma unroll
        for (int ab = 0; ab < 2; ++ab)
#pragma unroll
          for (int i = 0; i < 4; ++i) pr[4 * ab + i] = fast_exp2(fmaf(sc[h][ab][cg][i], c2, -mc));
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) pf[h][cg][jj] = pack_bf16x2(pr[2 * jj], pr[2 * jj + 1]);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) ts[cg] = dot2_bf16_ones(pf[h][cg][jj], ts[cg]);
      }
    }
  };
  auto softmax_tile = [&](f32x4 (&sc)[2][2][kCG], u32x4 (&pf)[2][kCG]) {
    float ts[kCG];
    tile_exp(sc, pf, ts);
    bool raise = false;
#pragma unroll
    for (int cg = 0; cg < kCG; ++cg) raise = raise || !(ts[cg] <= kLaneSumLimit);
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {
#pragma unroll
      for (int cg = 0; cg < kCG; ++cg) {
        const float a8[8] = {sc[0][0][cg][0], sc[0][0][cg][1], sc[0][0][cg][2], sc[0][0][cg][3],
                             sc[0][1][cg][0], sc[0][1][cg][1], sc[0][1][cg][2], sc[0][1][cg][3]};
        const float b8[8] = {sc[1][0][cg][0], sc[1][0][cg][1], sc[1][0][cg][2], sc[1][0][cg][3],
                             sc[1][1][cg][0], sc[1][1][cg][1], sc[1][1][cg][2], sc[1][1][cg][3]};
        const float cmax = max_xor32(max_xor16(max2(max8(a8), max8(b8)))) * c2;
        const bool up = cmax > m[cg];
        const float alpha = up ? fast_exp2(m[cg] - cmax) : 1.f;
        m[cg] = up ? cmax : m[cg];
        lsum[cg] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) acc[cg][dt] *= alpha;
      }
      tile_exp(sc, pf, ts);
    }
#pragma unroll
    for (int cg = 0; cg < kCG; ++cg) lsum[cg] += ts[cg];
  };
  // O^T += V^T P^T for one half tile.
  auto load_v = [&](int buf, int h, u32x4 (&vf)[8]) {
    const uint32_t a = buf_off(buf) + kKTileBytes + op_lane + h * (kKTileBytes / 2);  // keys 32h + 8q .. +7
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) vf[dt] = *lds128(a + 1024 * dt);
  };
  auto pv_ops = [&](const u32x4 (&vf)[8], const u32x4 (&pf)[kCG]) {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
      for (int cg = 0; cg < kCG; ++cg) acc[cg][dt] = mfma16x16x32(vf[dt], pf[cg], acc[cg][dt]);
  };

  // ---- tile loop ----
  // The waves form two groups, A (waves 0-3) and B (waves 4-7), one wave of
  // each on every SIMD. A tile is processed in two phases: a matrix phase
  // (QK^T of tile j and PV of tile j-1, both on MFMA with operands from LDS)
  // and a softmax phase (VALU: mask, exponentials, row sums, plus this
  // thread's share of the tile staging: LDS stores, global loads, address
  // arithmetic). Group B runs its phases offset from group A's (see the loop),
  // so that on every SIMD one wave's matrix products overlap the other wave's
  // softmax, and the two matrix phases overlap in part. Each thread stores its
  // share of a tile two (group A) or one (group B) barrier intervals before
  // the tile is first read; the global loads of a tile go out one tile before
  // its store.
  auto pv_tile = [&](int buf, const u32x4 (&pf)[2][kCG]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 vf[8];
      load_v(buf, h, vf);
      pv_ops(vf, pf[h]);
    }
  };

  // the first three tiles' loads go out together (no accumulator is live yet),
  // those that exist: one tile loaded three times took 34 tokens over none 9.4 us
  // instead of 8.8
  Stage st;
  {
    Stage s0, s1;
    fetch(0, s0);
    if (ntiles > 1) {
      fetch(1, s1);
      if (ntiles > 2) fetch(2, st);
      store_tile(0, s0);
      store_tile(1, s1);
    } else {
      store_tile(0, s0);
    }
  }
  __syncthreads();
  const bool lag = wave >= kThreads / kWave / 2;  // group B

  f32x4 sc[2][2][kCG];
  u32x4 pf[2][kCG];
  // matrix phase: PV of tile jt-1, QK^T of tile jt, at raised issue priority
  // so that the other wave's softmax takes the issue slots the matrix
  // products leave free. One software pipeline through both: draining it
  // between PV and QK^T cost 1.0-1.5% (4 x 2048 over 8192 cached: 1965 -> 1947
  // us) and 3% with one workgroup per compute unit at work (295 tokens over
  // 22.5K: 517 -> 502 us).
  auto matrix_phase = [&](int jt, auto first_tag) __attribute__((always_inline)) {
    constexpr bool kFirst = decltype(first_tag)::value;
    constexpr int kReads = kFirst ? 16 : 32;
    const int buf = jt & (kBufs - 1);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(2);
    if constexpr (!kFirst) pv_tile((jt + kBufs - 1) & (kBufs - 1), pf);
    qk_half(buf, 0, sc[0]);
    qk_half(buf, 1, sc[1]);
    // operand reads run kAhead reads ahead of the products that use them, from
    // the PV products on into the QK^T ones
    __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
    for (int i = 0; i < kReads - kAhead; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, kCG, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kCG * kAhead, 0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
  };
  // softmax phase of tile jt, with this thread's share of the staging: tile
  // jt+2 from registers to LDS, tile jt+3's global loads
  auto softmax_phase = [&](int jt) __attribute__((always_inline)) {
    const int kt = tile_key(jt);
    if (jt + 2 < ntiles) store_tile((jt + 2) & (kBufs - 1), st);
    if (jt + 3 < ntiles) fetch(jt + 3, st);
    if (needs_mask(jt, kt)) {
      const int kend = jt < ncached ? P - 1 : khi;
      mask_half(kt, kend, 0, sc[0]);
      mask_half(kt, kend, 1, sc[1]);
    }
    softmax_tile(sc, pf);
  };
  // One barrier per tile. Between barriers t and t+1 group A runs the matrix
  // phase of tile t, then its softmax phase; group B first the softmax phase
  // of tile t-1, then the matrix phase of tile t. A wave of B thus starts its
  // matrix products while its SIMD partner is still in its own, and the
  // partner's softmax runs under the rest of them. Between those barriers the
  // tiles read are t (K) and t-1 (V); the stores go to tile t+2 (group A) and
  // t+1 (group B), whose buffers were last read (as tiles t-2 and t-3) before
  // barrier t, and a stored tile is first read after a further barrier.
  auto tile_barrier = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::true_type kFirstTile{};
  constexpr std::false_type kNextTile{};
  if (!lag) {
    matrix_phase(0, kFirstTile);
    softmax_phase(0);
    tile_barrier();
    for (int jt = 1; jt < ntiles; ++jt) {
      matrix_phase(jt, kNextTile);
      softmax_phase(jt);
      tile_barrier();
    }
  } else {
    matrix_phase(0, kFirstTile);
    tile_barrier();
    for (int jt = 1; jt < ntiles; ++jt) {
      softmax_phase(jt - 1);
      matrix_phase(jt, kNextTile);
      tile_barrier();
    }
    softmax_phase(ntiles - 1);
  }
  pv_tile((ntiles + kBufs - 1) & (kBufs - 1), pf);

  // ---- normalise and write ----
  bool last = !kSplit;
  if constexpr (kSplit) {
    const int64_t u = sl->walk.u, per = sl->walk.per;
    const bool whole = ntiles == nall;
    if (tid == 0 && u == sl->walk.u0) {
      // the span's first query tile, for the merge: it takes up a tile at the
      // second of its spans
      const int64_t k0 = u - j0, first = k0 / per;  // k0: the place of the tile's first key tile, if j0 > 0
      PrefillDesc d;
      d.pieces = j0 > 0 && first + 1 == span ? (int)((k0 + nall - 1) / per - first) + 1 : 0;
      d.tok = tok0 + q0;
      d.positions = q1 - q0 + 1;
      d.head = g;
      p.ws_desc[span] = d;
    }
    if (!whole) {
      // a piece of the query tile: slot 2 span + 1 for its first key tiles,
      // slot 2 span for later ones (the span's last and first piece);
      // accumulators in register order (1 KiB runs)
      const int64_t base = ((int64_t)(2 * span + (j0 == 0 ? 1 : 0)) * 8 + wave) * kCG;
#pragma unroll
      for (int cg = 0; cg < kCG; ++cg) {
        const float l = sum_xor32(sum_xor16(lsum[cg]));
        // a row that sees no key of this piece: o = 0, log-sum-exp -inf
        const float inv = l != 0.f ? 1.f / l : 0.f;
        f32x4 *dst = reinterpret_cast<f32x4 *>(p.ws_o) + (base + cg) * 8 * kWave + lane;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) dst[dt * kWave] = acc[cg][dt] * inv;
        if (q == 0) p.ws_lse[(base + cg) * 16 + r] = m[cg] + __log2f(l);
      }
    }
    const int64_t unext = sl->walk.next;
    const bool done = unext >= sl->walk.u1;
    __syncthreads();  // every wave has read sl->walk and the tile buffers
    if (tid == 0) sl->walk.u = unext;
    if (!whole) {
      if (done) return;
      continue;
    }
    if (done) last = true;
  }
#pragma unroll
  for (int cg = 0; cg < kCG; ++cg) {
    const float l = sum_xor32(sum_xor16(lsum[cg]));
    const float inv = 1.f / l;
    const int row = wave * (16 * kCG) + cg * 16 + r;
    const int po = row / G, head = row - po * G;
    uint16_t *orow = p.out + ((int64_t)(tok0 + q0 + (cval[cg] ? po : 0)) * hq + (int64_t)g * G + head) * kHeadDim;
    u32x2 w[8];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      w[dt][0] = pack_bf16x2(acc[cg][dt][0] * inv, acc[cg][dt][1] * inv);
      w[dt][1] = pack_bf16x2(acc[cg][dt][2] * inv, acc[cg][dt][3] * inv);
    }
    store_out_row(orow, w, q, cval[cg]);
  }
  if (last) break;
  }
}

// kSplit: a call that may be cut into equal spans of key tiles, one per
// workgroup.
template <int kCG, int kPage, bool kSplit>
__global__ __launch_bounds__(kThreads) void prefill_kernel(PrefillParams p) {
  constexpr int kRows = 8 * 16 * kCG;
  __shared__ TileBufs bufs;
  const int npos = kRows / p.group, ntq = (p.max_chunk_len + npos - 1) / npos;
  // XCD-aware order of whole query tiles. Workgroup ids are dealt to the XCDs
  // round-robin; the (sequence, KV head) pairs are dealt the same way, pair
  // x + 8k to XCD x, so every query tile of a pair runs on one XCD and shares
  // its K/V in that L2, while pairs of unequal length (different prefixes)
  // spread over all XCDs. Within a pair the longest query tiles (the last ones)
  // go first. False: no tile for this workgroup.
  int b = 0, g = 0, tq = 0;
  auto take_whole = [&]() {
    const int npairs = p.ns * p.hkv;
    const int xcd = (int)(blockIdx.x % kXcds);
    const int local = (int)(blockIdx.x / kXcds);
    const int k = local / ntq;
    tq = ntq - 1 - (local - k * ntq);
    const int pair = xcd + kXcds * k;
    if (pair >= npairs) return false;
    b = pair / p.hkv;
    g = pair - b * p.hkv;
    return tq * npos < chunk_len(p, b);
  };
  if constexpr (kSplit) {
    __shared__ SpanLds sl;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const bool extra = blockIdx.x >= kSplitSpans;  // whole tiles only
    if (extra && !take_whole()) return;
    if (!split_gains(p, npos, lane)) {
      // No gain: a whole query tile each, as in the unsplit call, and nothing to
      // merge. (The same code as there: deciding inside the walk of the spans
      // took both of them 2% more.)
      if (tid == 0 && !extra) p.ws_desc[blockIdx.x].pieces = 0;
      if (extra || take_whole()) prefill_tiles<kCG, kPage, false>(p, bufs, nullptr, 0, b, g, tq);
      return;
    }
    if (extra) return;
    // Split order: the query tiles of every KV head, sequence and position, in
    // that order, each worth its key tiles plus kTileCost, are cut into equal
    // spans of `per`, one span per workgroup (workgroup ids go to the XCDs
    // round-robin, so an XCD gets consecutive spans: with 8 KV heads, one
    // head). A query tile met by several spans gets a partial result from
    // each, merged by prefill_merge_kernel.
    const int span = (int)(blockIdx.x % kXcds) * (kSplitSpans / kXcds) + (int)(blockIdx.x / kXcds);
    const int idx = tid;  // (sequence, query tile) pairs: at most one per thread (checked on the host)
    const int bb = idx / ntq;
    int64_t n = bb < p.ns ? key_tiles(idx - bb * ntq, npos, chunk_len(p, bb), p.prefix_lens[bb], p.pool.window) : 0;
    n += n > 0 ? kTileCost : 0;
    n = wave_scan(n, (int64_t)0, [](int64_t x, int64_t y) { return x + y; });
    if (lane == kWave - 1) sl.wave[wave] = n;
    __syncthreads();
    int64_t one = 0;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) {
      if (w == wave) n += one;
      one += sl.wave[w];
    }
    sl.cum[tid] = n;
    const int64_t total = one * p.hkv, per = max((int64_t)kMinSpan, (total + kSplitSpans - 1) / kSplitSpans);
    const int64_t u = span * per;
    if (tid == 0) sl.walk = Walk{one, per, u, u, min(total, u + per), 0};
    if (u >= total) {
      if (tid == 0) p.ws_desc[span].pieces = 0;
      return;
    }
    prefill_tiles<kCG, kPage, true>(p, bufs, &sl, span, 0, 0, 0);
  } else {
    if (!take_whole()) return;
    prefill_tiles<kCG, kPage, false>(p, bufs, nullptr, 0, b, g, tq);
  }
}

// Log-sum-exp merge of the query tiles that several spans met. One workgroup
// per 16 rows of the tile that the first boundary of a span cuts; wave pp
// merges dims 32 pp .. +31 (the accumulator vectors 2 pp and 2 pp + 1).
template <int kCG>
__global__ __launch_bounds__(4 * kWave) void prefill_merge_kernel(PrefillParams p) {
  constexpr int kParts = 8 * kCG;  // 16-row groups of a tile
  const int span = 1 + (int)(blockIdx.x / kParts), part = (int)(blockIdx.x % kParts);
  const PrefillDesc d = p.ws_desc[span];
  if (d.pieces == 0) return;
  const int lane = threadIdx.x & (kWave - 1), pp = threadIdx.x / kWave;
  const int r = lane & 15, q = lane >> 4;
  // piece 0 lies in slot 2 (span - 1) + 1, piece i in slot 2 (span - 1 + i)
  auto group_of = [&](int i) { return (int64_t)(2 * (span - 1 + i) + (i == 0 ? 1 : 0)) * kParts + part; };
  float mx = -INFINITY;
#pragma unroll 4
  for (int i = 0; i < d.pieces; ++i) mx = fmaxf(mx, p.ws_lse[group_of(i) * 16 + r]);
  const f32x4 *src = reinterpret_cast<const f32x4 *>(p.ws_o) + 2 * pp * kWave + lane;
  float wsum = 0.f;
  f32x4 o0 = {0.f, 0.f, 0.f, 0.f}, o1 = o0;
#pragma unroll 4
  for (int i = 0; i < d.pieces; ++i) {
    const int64_t gi = group_of(i);
    const float w = fast_exp2(p.ws_lse[gi * 16 + r] - mx);
    wsum += w;
    o0 += w * src[gi * 8 * kWave];
    o1 += w * src[gi * 8 * kWave + kWave];
  }
  const float inv = 1.f / wsum;
  const u32x2 w0 = {pack_bf16x2(o0[0] * inv, o0[1] * inv), pack_bf16x2(o0[2] * inv, o0[3] * inv)};
  const u32x2 w1 = {pack_bf16x2(o1[0] * inv, o1[1] * inv), pack_bf16x2(o1[2] * inv, o1[3] * inv)};
  const u32x4 v = out_row_piece(w0, w1);
  const int row = part * 16 + r;
  const int po = row / p.group, head = row - po * p.group;
  if (po >= d.positions) return;
  uint16_t *orow = p.out + ((int64_t)(d.tok + po) * p.hq + (int64_t)d.head * p.group + head) * kHeadDim;
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(orow + 32 * pp + 16 * (q & 1) + 8 * (q >> 1)));
}

}  // namespace

constexpr int kRowGroups = 2;  // 16-column MFMA groups per wave: 256 query rows per workgroup

template <bool kSplit>
hipError_t launch_prefill_rows(const PrefillParams &p, dim3 grid, hipStream_t stream) {
  const dim3 block(kThreads);
  switch (p.pool.pg_shift) {
    case 4: return launch_kernel(prefill_kernel<kRowGroups, 16, kSplit>, grid, block, stream, p);
    case 5: return launch_kernel(prefill_kernel<kRowGroups, 32, kSplit>, grid, block, stream, p);
    default: return launch_kernel(prefill_kernel<kRowGroups, 64, kSplit>, grid, block, stream, p);
  }
}

// Whether a FULL call can gain from a cut into spans of key tiles. The host knows
// the chunk lengths only by their largest and their sum, and the prefix lengths
// only as what the block table can hold; in key tiles it takes the unsplit call
// as the largest of its longest tile, its rounds of the shortest tiles and its
// average load on the fullest XCD, and the split one as the average over all
// compute units. Calls that fill the device whatever their contexts stay
// unsplit here (4 x 2048 over 8192, gain 0: 1915 us, cut 2150); for the others the
// kernel decides by the lengths themselves (split_gains), which costs a call that
// is then not cut 3 to 5 us. With a context as long as the table, the line of
// kSplitGain is where both measured the same: with 64 / 8 heads, 64 tokens over
// 1000 (14) 32 us unsplit and 30 split, 8 x 64 over 1000 (11) 34 and 40.
bool prefill_split_fits(const PrefillParams &p) {
  if (p.pool.window > 0 || p.ns <= 0 || p.max_chunk_len <= 0 || p.total_tokens <= 0) return false;
  const int npos = 128 * kRowGroups / p.group;
  const int64_t ntq = (p.max_chunk_len + npos - 1) / npos;
  if (ntq * p.ns > kThreads) return false;  // one (sequence, query tile) pair per thread
  const double keys = (double)(((int64_t)p.pool.stride << p.pool.pg_shift) / kKT);
  const double chunk = std::min<double>(keys, (double)p.max_chunk_len / kKT);
  const double longest = keys + kTileCost, average = longest - chunk / 2, shortest = longest - chunk;
  const double tiles = (double)(std::min<int64_t>(ntq * p.ns, p.total_tokens / npos + p.ns) * p.hkv) / kSplitSpans;
  const int64_t pairs = (int64_t)p.ns * p.hkv;
  const double load = (double)((pairs + kXcds - 1) / kXcds * ntq) / (kSplitSpans / kXcds);  // tiles per CU
  const double unsplit = std::max({longest, std::ceil(load) * shortest, load * average});
  return unsplit - std::max((double)kMinSpan, tiles * average) >= kSplitGain;
}

// fp32 partials, their log-sum-exps and a descriptor per span.
constexpr size_t kSplitOBytes = (size_t)2 * kSplitSpans * 128 * kRowGroups * kHeadDim * 4;
constexpr size_t kSplitLseBytes = (size_t)2 * kSplitSpans * 128 * kRowGroups * 4;

size_t prefill_split_bytes() { return kSplitOBytes + kSplitLseBytes + kSplitSpans * sizeof(PrefillDesc); }

hipError_t launch_prefill_split(const PrefillParams &p0, void *workspace, hipStream_t stream) {
  PrefillParams p = p0;
  char *ws = static_cast<char *>(workspace);
  p.ws_o = reinterpret_cast<float *>(ws);
  p.ws_lse = reinterpret_cast<float *>(ws + kSplitOBytes);
  p.ws_desc = reinterpret_cast<PrefillDesc *>(ws + kSplitOBytes + kSplitLseBytes);
  // a workgroup per span, and one per query tile should the lengths show no gain
  const int npos = 128 * kRowGroups / p.group;
  const int64_t ntq = (p.max_chunk_len + npos - 1) / npos;
  const int64_t pairs_per_xcd = ((int64_t)p.ns * p.hkv + kXcds - 1) / kXcds;
  const int64_t grid = std::max<int64_t>(kSplitSpans, pairs_per_xcd * ntq * kXcds);
  const hipError_t e = launch_prefill_rows<true>(p, dim3((unsigned)grid), stream);
  if (e != hipSuccess) return e;
  return launch_kernel(prefill_merge_kernel<kRowGroups>, dim3((kSplitSpans - 1) * 8 * kRowGroups), dim3(4 * kWave),
                       stream, p);
}

hipError_t launch_prefill(const PrefillParams &p, hipStream_t stream) {
  if (p.ns <= 0 || p.max_chunk_len <= 0 || p.total_tokens <= 0) return hipSuccess;
  if (p.pool.window > 0 && prefill_run_fits(p)) return launch_prefill_run(p, stream);
  if (p.pool.window > 0 && p.pool.window <= kPrefillWindowMax) return launch_prefill_window(p, stream);
  const int npos = 128 * kRowGroups / p.group;
  const int64_t ntq = (p.max_chunk_len + npos - 1) / npos;
  const int64_t pairs_per_xcd = ((int64_t)p.ns * p.hkv + kXcds - 1) / kXcds;
  return launch_prefill_rows<false>(p, dim3((unsigned)(pairs_per_xcd * ntq * kXcds)), stream);
}

}  // namespace hswa
