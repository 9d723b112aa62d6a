// KV append: slot mapping and scatter of new K/V rows into the paged pools.
//
// Dual-pool layout ("KVCache Dual-Pool Design"): a FULL layer keeps every
// position; an SWA layer keeps a ring of R = ceil(W/PG)+1 pages per sequence,
// and the ring overwrite is the out-of-window eviction that follows every chunk
// and every decode step ("SWA-Aware Prefix Cache Tree").
//
// Bound by moving the rows: every row is read once and written once. What
// decides the rate is the width of the V stores, since a V block is transposed
// ([D][B] keys) and a token's column in it is 128 scattered 2-byte elements.
// Long sequences are therefore cut along the pool's blocks, not along the batch:
// for each aligned run of 32 positions of one sequence and KV head, one
// workgroup reads its rows (64-byte runs of 16 rows per load instruction),
// transposes V in registers with lane swaps, and writes whole 16-byte pieces,
// the K block as contiguous 1 KiB runs and V as full 64-byte rows, whatever the
// sequences' alignment in the batch; only the first and last 8 keys of such an
// append can be partial pieces (2-byte stores).
// 12.3K tokens in 8 sequences at unaligned positions, 8 heads, PG 64 (101 MB
// read and written): 92 us cut at 8 tokens of the batch, 25 by runs, 4.0 TB/s
// (a large device copy: 4.9).
// Sequences of fewer than 8 new tokens of a batch of longer ones are scattered
// token by token. Calls of few tokens a sequence take 8-token tiles, which
// scatter them too, except that eight tokens on 8 aligned slots in a row go out
// as one 16-byte V store a dim (see append_tile for which call takes which tile).
#include "append_grid.h"
#include "hswa_common.h"
#include "hswa_launch.h"

namespace hswa {
namespace {

constexpr int kThreads = kAppendThreads;
constexpr int kLdsSeqs = 4096;  // batches up to this size search cu_seqlens in LDS
constexpr int kRun = 32;        // positions of an aligned run

// Sequence of flattened token t: the b with cu(b) <= t < cu(b + 1) (-1 if none).
template <typename Cu>
__device__ __forceinline__ int find_seq(Cu cu, int ns, int t) {
  int lo = 0, hi = ns;  // answer in [0, ns)
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (cu(mid) <= t) lo = mid; else hi = mid;
  }
  return t >= cu(lo) && t < cu(lo + 1) ? lo : -1;
}

// Physical page of logical page lp >= 0 of sequence b, -1 if the table has none.
__device__ __forceinline__ int64_t page_of(const PoolView &pv, int b, int64_t lp) {
  if (pv.ring > 0) lp = (uint32_t)lp % (uint32_t)pv.ring;  // lp < 2^33 / 16
  if (lp >= pv.stride) return -1;
  const int64_t page = pv.table[int64_t(b) * pv.stride + lp];
  return page >= 0 && page < pv.num_pages ? page : -1;
}

// The same for a wave-uniform b and lp, read through the scalar cache (the
// kernel writes no table).
__device__ __forceinline__ int uniform_page(const PoolView &pv, int b, int lp) {
  if (pv.ring > 0) lp %= pv.ring;
  if (lp >= pv.stride) return -1;
  typedef __attribute__((address_space(4))) const int32_t const_i32;
  const int page = ((const_i32 *)pv.table)[(int64_t)b * pv.stride + lp];
  return page >= 0 && page < pv.num_pages ? page : -1;
}

// Lane l's v (l wave-uniform), as a scalar.
__device__ __forceinline__ int64_t lane64(int64_t v, int l) {
  return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32) |
                   (uint32_t)__builtin_amdgcn_readlane((int)v, l));
}

// 4 x 4 transpose of dwords across the lanes l, l ^ 16, l ^ 32, l ^ 48: the
// lane in 16-lane row m enters with dword j of its row m in t[j] and leaves
// with dword m of rows 0..3 in w[0..3].
__device__ __forceinline__ void transpose4(const u32x4 &t, uint32_t *w) {
  const auto a = __builtin_amdgcn_permlane32_swap(t[0], t[2], false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(t[1], t[3], false, false);
  const auto c = __builtin_amdgcn_permlane16_swap((uint32_t)a[0], (uint32_t)b[0], false, false);
  const auto d = __builtin_amdgcn_permlane16_swap((uint32_t)a[1], (uint32_t)b[1], false, false);
  w[0] = (uint32_t)c[0];
  w[1] = (uint32_t)c[1];
  w[2] = (uint32_t)d[0];
  w[3] = (uint32_t)d[1];
}

// One workgroup per (tile of kTok consecutive tokens of the flattened batch, KV
// head). It scatters the tile's tokens of short sequences, and writes every
// aligned run of a long sequence whose first appended token lies in the tile
// (the run's other tokens may lie past it; no other workgroup writes them).
// 8-token tiles scatter every sequence.
template <int kTok>
__global__ __launch_bounds__(kThreads) void kv_append_kernel(AppendParams p) {
  // sequences of at least this many new tokens are written by runs (8 against
  // 16: 4096 + 64 x 12 tokens 11.0 us against 14.1)
  constexpr int kLong = kTok == 8 ? INT32_MAX : 8;
  __shared__ int32_t s_cu[kLdsSeqs + 1];
  const PoolView &pv = p.pool;
  const int hkv = p.hkv;
  const int tile = (int)(blockIdx.x / (unsigned)hkv);
  const int g = (int)(blockIdx.x - (unsigned)tile * (unsigned)hkv);  // heads of a token next to each other: whole rows
  const int t0 = tile * kTok;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int pg = 1 << pv.pg_shift;

  // An 8-token tile loads its rows at once, next to the lengths and the table,
  // so that only the stores wait for the slots: waves 0 and 1 a 16-byte piece
  // of a K row a thread, waves 2 and 3 one dim of all 8 V rows.
  constexpr bool kTile8 = kTok == 8;
  constexpr int kSK = (kTok * 16 + kThreads - 1) / kThreads, kSV = kTok * kHeadDim / kThreads;  // pieces a thread
  [[maybe_unused]] u32x4 ek = {0u, 0u, 0u, 0u};
  [[maybe_unused]] uint16_t ev[8] = {};
  if constexpr (kTile8) {
    if (wave < 2) {
      const int tk = min(t0 + (tid >> 4), p.total_tokens - 1);
      ek = ldg128(p.k_new + ((int64_t)tk * hkv + g) * kHeadDim + (tid & 15) * 8);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int tk = min(t0 + i, p.total_tokens - 1);
        ev[i] = p.v_new[((int64_t)tk * hkv + g) * kHeadDim + tid - kHeadDim];
      }
    }
  }

  // Lane i < kTok of every wave holds token t0 + i: its sequence b, the
  // sequence's first token tb, its end te and the position of its first token.
  // The lengths are read once, coalesced, instead of by a chain of dependent
  // loads in the binary search: up to 63 sequences in the lanes (with their
  // start positions), larger batches in LDS.
  const int t = t0 + lane;
  const bool tok_ok = lane < kTok && t < p.total_tokens;
  int b = -1, tb = 0, te = 0;
  int64_t start = 0;
  if (p.ctx_lens) {  // decode step: token t is sequence t's
    if (tok_ok) {
      b = t;
      tb = t;
      te = t + 1;
      start = (int64_t)min(p.ctx_lens[b], p.max_ctx) - 1;
    }
  } else if (p.ns < kWave) {
    const int cul = p.cu_seqlens[min(lane, p.ns)];
    const int spl = p.start_pos[min(lane, p.ns - 1)];
    int lo = 0;  // the last b with cu[b] <= t, by halving (all lanes take part in the shuffles)
#pragma unroll
    for (int step = kWave / 2; step > 0; step >>= 1) {
      const int mid = lo + step;
      const int c = __shfl(cul, min(mid, p.ns), kWave);
      if (mid < p.ns && c <= t) lo = mid;
    }
    tb = __shfl(cul, lo, kWave);
    te = __shfl(cul, lo + 1, kWave);
    start = __shfl(spl, lo, kWave);
    if (tok_ok && t >= tb && t < te) b = lo;
  } else {
    const bool lds_cu = p.ns <= kLdsSeqs;
    if (lds_cu) {
      for (int i = tid; i <= p.ns; i += kThreads) s_cu[i] = p.cu_seqlens[i];
      __syncthreads();
    }
    if (tok_ok) {
      b = lds_cu ? find_seq([&](int i) { return s_cu[i]; }, p.ns, t)
                 : find_seq([&](int i) { return p.cu_seqlens[i]; }, p.ns, t);
      if (b >= 0) {
        tb = lds_cu ? s_cu[b] : p.cu_seqlens[b];
        te = lds_cu ? s_cu[b + 1] : p.cu_seqlens[b + 1];
        start = p.start_pos[b];
      }
    }
  }
  const int64_t j = start + (t - tb);
  const bool is_long = b >= 0 && te - tb >= kLong;

  // Slots: every token's for the mapping, and those of the short sequences.
  const bool scatter = b >= 0 && !is_long;
  const uint64_t smask = __builtin_amdgcn_ballot_w64(scatter);
  const bool slots = p.slot_out && g == 0 && wave == 0;
  int64_t slot = -1;
  if (slots || smask != 0) {
    if (b >= 0 && j >= 0 && !(pv.ring > 0 && j < start + (te - tb) - (int64_t)pv.ring * pg)) {
      const int64_t page = page_of(pv, b, j >> pv.pg_shift);
      if (page >= 0) slot = page * pg + (j & (pg - 1));
    }
    if (slots && tok_ok) p.slot_out[t] = slot;
  }

  const int64_t sslot = scatter ? slot : -1;
  if constexpr (kTile8) {
    if (smask == 0) return;
    if (wave < 2) {
      const int64_t s = __shfl(sslot, tid >> 4, kWave);
      if (s >= 0)
        stg128(pv.k_pool + k_offset(pv, s >> pv.pg_shift, hkv, g, (int)(s & (pg - 1)), (tid & 15) * 8), ek);
      return;
    }
    // Eight tokens on 8 aligned slots in a row: one 16-byte V store a dim. (A
    // chunk or a few tokens a sequence at aligned positions; without it 2048
    // aligned tokens among 256 single ones took 17.8 us instead of 10.6, and
    // 256 x 8 aligned tokens 15.3 instead of 7.7.)
    const int d = tid - kHeadDim;
    const int64_t s0 = lane64(sslot, 0);
    const uint64_t in_row = __builtin_amdgcn_ballot_w64(lane < 8 && sslot == s0 + lane);
    if (in_row == 0xFFu && s0 >= 0 && (s0 & 7) == 0) {
      u32x4 w;
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = ev[2 * i] | ((uint32_t)ev[2 * i + 1] << 16);
      stg128(pv.v_pool + v_offset(pv, s0 >> pv.pg_shift, hkv, g, (int)(s0 & (pg - 1)), d), w);
      return;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t s = lane64(sslot, i);
      if (s >= 0) pv.v_pool[v_offset(pv, s >> pv.pg_shift, hkv, g, (int)(s & (pg - 1)), d)] = ev[i];
    }
    return;
  }

  // Short sequences of a larger tile: K rows as sixteen 16-byte pieces, V
  // element by element, all loads ahead of the stores.
  if (smask != 0) {
    u32x4 ks[kSK];
    uint16_t vs[kSV];
    const int ktok = tid >> 4, vtok = wave >> 1;  // of piece 0; a later one's is 16 (K) or 2 (V) tokens on
    const uint16_t *krow = p.k_new + ((int64_t)t0 * hkv + g) * kHeadDim + (tid & 15) * 8;
    const uint16_t *vrow = p.v_new + ((int64_t)t0 * hkv + g) * kHeadDim + (tid & (kHeadDim - 1));
    const int64_t row = (int64_t)hkv * kHeadDim;
#pragma unroll
    for (int i = 0; i < kSK; ++i)
      if ((smask >> (ktok + 16 * i)) & 1u) ks[i] = ldg128(krow + (ktok + 16 * i) * row);
#pragma unroll
    for (int i = 0; i < kSV; ++i)
      if ((smask >> (vtok + 2 * i)) & 1u) vs[i] = vrow[(vtok + 2 * i) * row];
#pragma unroll
    for (int i = 0; i < kSK; ++i) {
      const int64_t s = __shfl(sslot, ktok + 16 * i, kWave);
      if (s >= 0) stg128(pv.k_pool + k_offset(pv, s >> pv.pg_shift, hkv, g, (int)(s & (pg - 1)), (tid & 15) * 8), ks[i]);
    }
#pragma unroll
    for (int i = 0; i < kSV; ++i) {
      const int64_t s = __shfl(sslot, vtok + 2 * i, kWave);
      if (s >= 0)
        pv.v_pool[v_offset(pv, s >> pv.pg_shift, hkv, g, (int)(s & (pg - 1)), tid & (kHeadDim - 1))] = vs[i];
    }
  }

  // Long sequences: the runs that start in this tile (a sequence's first token,
  // or a position that is a multiple of kRun).
  const bool two = pv.pg_shift == 4;
  uint64_t runs = __builtin_amdgcn_ballot_w64(is_long && (t == tb || (j & (kRun - 1)) == 0));
  while (runs != 0) {
    const int l = __builtin_ctzll(runs);
    runs &= runs - 1;
    const int rb = __builtin_amdgcn_readlane(b, l);
    const int rte = __builtin_amdgcn_readlane(te, l);
    const int64_t rj = lane64(j, l);
    const int64_t base = rj & ~(int64_t)(kRun - 1);
    const int first = (int)(rj - base);              // key of token t0 + l in the run
    const int nkeys = min(kRun, first + min(rte, p.total_tokens) - (t0 + l));  // key of the first token past the new ones
    // the ring keeps the latest R*PG positions; positions before 0 do not exist
    int64_t keep_lo = 0;
    if (pv.ring > 0) keep_lo = max(keep_lo, rj + (rte - (t0 + l)) - (int64_t)pv.ring * pg);
    const int klo = (int)min((int64_t)kRun, max((int64_t)first, keep_lo - base));
    if (klo >= nkeys) continue;  // nothing of the run is kept
    const int tk0 = t0 + l - first;  // token of key 0 (read from key klo on only)

    // loads: K pieces in pool order (16 keys x 64 bytes a load), V pieces of
    // keys 8 kg + 4 i + m, dims 32 wave + 8 c .. +7 (kg = lane % 4,
    // c = lane / 4 % 4, m = lane / 16; a wave holds 32 dims of all keys)
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const int r = lane & 15, m = lane >> 4, kg = lane & 3, vc = (lane >> 2) & 3;
    u32x4 kv[2], vv[2];
    int kk[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      kk[i] = 8 * (r >> 2) + 4 * i + (r & 3);
      kv[i] = vv[i] = zero;
      if (kk[i] >= klo && kk[i] < nkeys)
        kv[i] = ldg128(p.k_new + ((int64_t)(tk0 + kk[i]) * hkv + g) * kHeadDim + 32 * wave + 8 * m);
      const int vk = 8 * kg + 4 * i + m;
      if (vk >= klo && vk < nkeys)
        vv[i] = ldg128(p.v_new + ((int64_t)(tk0 + vk) * hkv + g) * kHeadDim + 32 * wave + 8 * vc);
    }
    // a run lies on one page (PG >= 32) or on two (PG = 16); both pools put a
    // block (and a 16-key page-head) at the same element offset
    const int lp = (int)(base >> pv.pg_shift);
    const int page0 = base >= 0 ? uniform_page(pv, rb, lp) : -1;
    const int page1 = two && base >= 0 && nkeys > 16 ? uniform_page(pv, rb, lp + 1) : page0;
    const int64_t boff = (int64_t)((int)base & (pg - 1)) << kHeadDimShift;  // the run's block in its page
    const int64_t off0 = ((((int64_t)page0 * hkv + g) << pv.pg_shift) << kHeadDimShift) + (two ? 0 : boff);
    const int64_t off1 = two ? (((int64_t)page1 * hkv + g) << pv.pg_shift) << kHeadDimShift : off0;
    const bool ok0 = page0 >= 0, ok1 = page1 >= 0;
    {
      const bool second = two && r >= 8;
      uint16_t *dst = pv.k_pool + (second ? off1 : off0) + ((((4 * wave + m) << (pv.vb_shift - 1)) + (two ? r & 7 : r)) << 3);
#pragma unroll
      for (int i = 0; i < 2; ++i)  // halves: 16 16-byte pieces x B / 2 rows apart
        if (kk[i] >= klo && kk[i] < nkeys && (second ? ok1 : ok0)) stg128(dst + ((i << 6) << pv.vb_shift), kv[i]);
    }
    // lane m holds dims 2 m, 2 m + 1 of keys 8 kg .. +7 after the transposes
    uint32_t w[8];
    transpose4(vv[0], w);
    transpose4(vv[1], w + 4);
    u32x4 lo, hi;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      lo[q] = __builtin_amdgcn_perm(w[2 * q + 1], w[2 * q], 0x05040100u);
      hi[q] = __builtin_amdgcn_perm(w[2 * q + 1], w[2 * q], 0x07060302u);
    }
    const bool second = two && kg >= 2;
    if (second ? ok1 : ok0) {
      const uint32_t bits = key_range_bits(8 * kg, klo, nkeys - 1);
      uint16_t *dst = pv.v_pool + (second ? off1 : off0) + ((32 * wave + 8 * vc + 2 * m) << pv.vb_shift) +
                      8 * (two ? kg & 1 : kg);
      uint16_t *dst1 = dst + (1 << pv.vb_shift);  // the next dim
      if (bits == 0xFFu) {
        stg128(dst, lo);
        stg128(dst1, hi);
      } else if (bits != 0u) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if ((bits >> e) & 1u) {
            dst[e] = (uint16_t)(lo[e >> 1] >> (16 * (e & 1)));
            dst1[e] = (uint16_t)(hi[e >> 1] >> (16 * (e & 1)));
          }
        }
      }
    }
  }
}

}  // namespace

hipError_t launch_kv_append(const AppendParams &p, hipStream_t stream) {
  if (p.total_tokens <= 0) return hipSuccess;
  const int tile = append_tile(p.ctx_lens != nullptr, p.ns, p.total_tokens, p.hkv);
  const dim3 grid((unsigned)append_groups(tile, p.total_tokens, p.hkv));
  const auto kernel = tile == 8 ? kv_append_kernel<8> : tile == 16 ? kv_append_kernel<16> : kv_append_kernel<32>;
  return launch_kernel(kernel, grid, dim3(kThreads), stream, p);
}

}  // namespace hswa
