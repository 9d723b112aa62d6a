// Windowed (SWA) chunked prefill: the query at position p attends keys
// p - W + 1 .. p only ("Compute Analysis": an SWA layer's attention covers a
// local window, so its prefill cost is linear in the chunk and the layer is
// bound by moving q, o and the chunk's K/V, not by the matrix cores).
//
// The FULL-layer kernel (prefill.hip) is built for long key ranges: 256 query
// rows per workgroup, four 32 KiB tile buffers, one workgroup per CU. For a
// window of a few hundred keys most of its work is prologue and masked pairs.
// This kernel instead gives each workgroup 128 query rows (4 waves x 32 rows,
// a row = a (position, query head) pair of one KV head's GQA group), streams
// the workgroup's key range W + 128 / G - 1 through two 32-key chunk buffers
// (32 KiB) with the global loads one chunk ahead, and lets each wave skip the
// chunks that lie wholly outside the windows of its own rows.
//
// A wave's chunk is a serial chain (LDS reads, QK^T, softmax, PV, a barrier), so
// the kernel is bound by how many waves share a SIMD: three (168 VGPRs, three
// workgroups a CU) against two with four buffers, two register stages and the V
// operands read ahead: 3 ragged chunks of 300-1200 tokens, W = 512, PG 16,
// 32 / 8 heads 49.2 -> 41.4 us (0.52 PFLOP/s); 4 x 2000, 64 / 8 heads, W = 512
// 216 -> 186, W = 256 138 -> 117.
//
// Per 32-key chunk and wave (bf16 MFMA, fp32 accumulate):
//   S^T[key][row] = K[key][:] . Q[row][:]     (Q held in registers)
//   online softmax per row (exp2, scale * log2 e folded in, running maximum in
//   exp2 units, raised lazily as in the FULL kernel)
//   O^T[d][row]  += V^T[d][key] . P^T[key][row]
// LDS holds each chunk in MFMA operand order (K: 8 blocks of 1 KiB, block
// (ab, t) for lane r + 16 q = dims 32 t + 8 q .. +7 of chunk key
// 8 (r >> 2) + 4 ab + (r & 3), the pool's own K block layout; V^T: block dt for
// lane r + 16 q = keys 8 q .. +7 of dim 16 dt + r), so every operand read is
// one conflict-free ds_read_b128. Keys outside the workgroup's range are
// staged as zeros and every column masks its own window, so stale or NaN cache
// slots never reach an accumulator.
#include <cfloat>

#include "hswa_common.h"
#include "hswa_launch.h"

namespace hswa {
namespace {

constexpr int kWThreads = 256;
constexpr int kWWaves = kWThreads / kWave;  // 4
constexpr int kWRows = kWWaves * 32;         // query rows per workgroup
constexpr int kWChunk = 32;                  // keys per chunk
constexpr int kWBufs = 2;                    // chunk c being read, c + 1 being stored
constexpr int kWKBytes = kWChunk * kHeadDim * 2;  // 8 KiB of K per chunk
constexpr int kWBufBytes = 2 * kWKBytes;          // K, then V^T
constexpr int kWXcds = 8;
constexpr int kWCG = 2;                    // 16-column MFMA groups per wave
constexpr float kWLaneSumLimit = 4096.f;   // lane share of a row sum that raises the maximum

struct WStage {
  u32x4 k[2], v[2];
  uint32_t keep;  // bit i: k[i] holds data (else zeros are stored); bits 8 + 8 i ..: the
                  // elements (keys) of v[i] that hold data; all set inside the range
  bool edge;      // some key of the chunk is out of range (or on an invalid page)
  bool vrow;      // v[] holds key rows (chunk keys), transposed at the store
};

// kPage16: 16-key pages, two of them a chunk; else a chunk lies in one page.
template <bool kPage16>
__global__ __launch_bounds__(kWThreads) __attribute__((amdgpu_waves_per_eu(3))) void prefill_window_kernel(
    PrefillParams p) {
  __shared__ __attribute__((aligned(16))) unsigned char s_lds[kWBufs * kWBufBytes];

  const PoolView &pv = p.pool;
  const int G = p.group;
  const int npos = kWRows / G;  // positions per workgroup

  // Workgroup ids go to the XCDs round-robin; (sequence, KV head) pair
  // x + 8 k runs on XCD x, its position tiles in order, so the workgroups an
  // XCD holds at once are neighbouring tiles of one pair and share their keys
  // in that XCD's L2.
  const int ntq = (p.max_chunk_len + npos - 1) / npos;
  const int npairs = p.ns * p.hkv;
  const int xcd = (int)(blockIdx.x % kWXcds);
  const int local = (int)(blockIdx.x / kWXcds);
  const int k = local / ntq;
  const int tq = local - k * ntq;
  const int pair = xcd + kWXcds * k;
  if (pair >= npairs) return;
  const int b = pair / p.hkv, g = pair - b * p.hkv;

  const int tok0 = p.cu_seqlens[b];
  const int C = min(min(p.cu_seqlens[b + 1], p.total_tokens) - tok0, p.max_chunk_len);
  const int P = p.prefix_lens[b];
  const int q0 = tq * npos;
  if (q0 >= C || P < 0 || tok0 < 0) return;
  const int q1 = min(C, q0 + npos) - 1;
  const int W = pv.window;
  const int pfirst = P + q0, plast = P + q1;
  const int klo = max(0, pfirst - W + 1), khi = plast;

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int r = lane & 15, q = lane >> 4;
  const int hkv = p.hkv, hq = p.hq;
  const int shift = pv.pg_shift, pg = 1 << shift;
  const float c2 = p.scale_log2;

  // Page ids of the workgroup's cached keys: lane i holds the physical page
  // of logical page lp0 + i (-1: not cached, or not a valid page). The chunks
  // cover at most W + npos + 30 <= 670 keys from lp0's first key on: at most
  // 43 pages of 16 keys, so every cached key's page is in this table and the
  // staging never waits on a block-table load.
  const int lp0 = (klo & ~(kWChunk - 1)) >> shift;
  int tab = -1;
  {
    const int lp = lp0 + lane;
    if (P > 0 && lp <= ((min(P, khi + 1) - 1) >> shift)) {
      const int e = pv.ring > 0 ? lp % pv.ring : lp;
      if (e < pv.stride) {
        const int64_t v = pv.table[(int64_t)b * pv.stride + e];
        tab = (v >= 0 && v < pv.num_pages) ? (int)v : -1;
      }
    }
  }

  const int gshift = __builtin_ctz(G);  // groups are powers of two

  // Q^T operands of each of this lane's columns.
  u32x4 qf[kWCG][4];
#pragma unroll
  for (int cg = 0; cg < kWCG; ++cg) {
    const int row = wave * (16 * kWCG) + cg * 16 + r;
    const int po = row / G, head = row - po * G;
    const bool cval = q0 + po <= q1;
    const int64_t tok = tok0 + q0 + (cval ? po : 0);
    const uint16_t *qrow = p.q + (tok * hq + (int64_t)g * G + head) * kHeadDim;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const u32x4 v = ldg128(qrow + 32 * t + 8 * q);
      const u32x4 z = {0u, 0u, 0u, 0u};
      qf[cg][t] = cval ? v : z;
    }
  }
  // This wave's rows: positions po_lo .. po_hi of the tile (none if po_lo is
  // past the last valid one). Its keys are [wklo, wkhi]; a chunk inside
  // [wint_lo, wint_hi] is visible to every one of its columns (no mask).
  const int po_lo = (wave * 16 * kWCG) / G;
  const int po_hi = min((wave * 16 * kWCG + 16 * kWCG - 1) / G, q1 - q0);
  const bool wact = po_lo <= q1 - q0;
  const int wklo = max(klo, P + q0 + po_lo - W + 1);
  const int wkhi = min(khi, P + q0 + po_hi);
  const int wint_lo = max(0, P + q0 + po_hi - W + 1);
  const int wint_hi = P + q0 + po_lo;

  // ---- staging: global -> registers -> LDS ----
  // Thread tid stores K pieces idx = tid and tid + 256 at byte 16 idx of the
  // K block: block (ab, t) = idx >> 6, lane r + 16 qq = idx & 63, i.e. dims
  // 32 t + 8 qq .. +7 of chunk key 8 (r >> 2) + 4 ab + (r & 3). V^T pieces:
  // block dt = idx >> 6 holds for lane r + 16 qq keys 8 qq .. +7 of dim
  // 16 dt + r.
  auto k_key = [](int idx) { return ((idx & 15) >> 2) * 8 + (idx >> 8) * 4 + (idx & 3); };
  auto v_keys = [](int idx) { return ((idx >> 4) & 3) * 8; };
  const u32x4 zero = {0u, 0u, 0u, 0u};
  // physical page of logical page lp (-1: not cached or not valid), from the lane table
  auto page_at = [&](int lp) { return __builtin_amdgcn_readlane(tab, min(lp - lp0, kWave - 1)); };
  // Byte offsets of this thread's piece 0 and the steps to piece 1. A chunk's
  // pieces sit at fixed offsets from a wave-uniform address, so a fetch takes a
  // few vector instructions (forming each piece's address from its key, a page
  // lookup and a 64-bit product each, took 53.9 us for 3 ragged chunks of
  // 300-1200 tokens at W = 512, PG 16, 32 / 8 heads, against 49.1, and 230 for 4 x
  // 2000 at PG 64, 64 / 8 heads, against 214).
  // Pool blocks: the K block in LDS order and the [D][32] V block; with 16-key
  // pages the same pieces of two blocks of 8-row slabs and [D][16].
  const uint32_t v_dim = (uint32_t)((tid >> 6) * 16 + (tid & 15)), vq = (uint32_t)((tid >> 4) & 3);
  const uint32_t pk_off = kPage16 ? (uint32_t)((tid >> 4) * 128 + (tid & 7) * 16) : (uint32_t)tid * 16;
  const uint32_t pv_off = kPage16 ? v_dim * 32 + (vq & 1) * 16 : v_dim * 64 + vq * 16;
  constexpr uint32_t p_step = kPage16 ? 2048 : 4096;
  const bool ksecond = kPage16 && (tid & 8), vsecond = kPage16 && (vq & 2);  // on the chunk's second page
  // Rows of k_new / v_new: K dims 32 t + 8 qq of chunk key k_key, V dims
  // 8 (lane % 16) of chunk key 8 wave + lane / 16; piece 1 four keys on.
  const uint32_t row_bytes = (uint32_t)hkv * (kHeadDim * 2);
  const uint32_t nk_dim = (uint32_t)(((tid >> 6) & 3) * 64 + ((tid >> 4) & 3) * 16), nv_dim = (uint32_t)(lane & 15) * 16;
  const uint32_t nk_off = (uint32_t)k_key(tid) * row_bytes + nk_dim;
  const uint32_t nv_off = (uint32_t)(8 * wave + (lane >> 4)) * row_bytes + nv_dim;
  // The key range is cut at P into cached chunks, aligned to 32 absolute
  // positions (so that 8 consecutive keys of a V^T piece are 16 contiguous
  // bytes of one pool page), and chunks of the new keys, aligned to P. No chunk
  // holds both kinds, and every fetch is the same four 16-byte loads per thread,
  // written straight into the stage registers; pieces or keys outside the
  // range are zeroed only when the stage is stored, so a fetch never waits for
  // its own loads and a store waits only for its own stage.
  const int chi = min(P - 1, khi);  // last cached key (< klo: none)
  const int ncached = klo <= chi ? ((chi - (klo & ~(kWChunk - 1))) >> 5) + 1 : 0;
  const int nbase = max(klo, P) - P;  // first new key's offset from P
  const int nnew = khi >= max(klo, P) ? ((khi - P) >> 5) - (nbase >> 5) + 1 : 0;
  const int nch = ncached + nnew;
  auto chunk_base = [&](int c) {
    return c < ncached ? (klo & ~(kWChunk - 1)) + kWChunk * c : P + kWChunk * ((nbase >> 5) + c - ncached);
  };
  auto fetch = [&](int c, WStage &st) {
    c = min(c, nch - 1);  // past the end: a repeat of the last chunk, never stored
    const int kb = chunk_base(c);
    const bool cached = c < ncached;
    const char *kbase, *vbase;  // wave-uniform, except that a lane picks its page of two
    uint32_t ko[2], vo[2];
    st.keep = 0xFFFF03u;
    st.vrow = !cached;
    if (cached) {
      const int lp = kb >> shift;
      const int pa = page_at(lp), pb = kPage16 ? page_at(lp + 1) : pa;
      auto page_off = [&](int page) {
        const int64_t ph = ((int64_t)max(page, 0) * hkv + g) << (shift + kHeadDimShift + 1);
        return kPage16 ? ph : ph + ((int64_t)((kb & (pg - 1)) >> 5) << (5 + kHeadDimShift + 1));
      };
      const int64_t oa = page_off(pa), ob = page_off(pb);
      kbase = reinterpret_cast<const char *>(pv.k_pool) + (ksecond ? ob : oa);
      vbase = reinterpret_cast<const char *>(pv.v_pool) + (vsecond ? ob : oa);
      ko[0] = pk_off;
      vo[0] = pv_off;
      ko[1] = pk_off + p_step;
      vo[1] = pv_off + p_step;
      st.edge = kb < klo || kb + kWChunk - 1 > chi || pa < 0 || pb < 0;
      if (st.edge) {  // the pieces are all in their pages' bounds: only kept or not
        uint32_t keep = 0u;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int j = kb + k_key(tid + kWThreads * i), j0 = kb + v_keys(tid);
          keep |= (j >= klo && j <= chi && (ksecond ? pb : pa) >= 0 ? 1u : 0u) << i;
          keep |= ((vsecond ? pb : pa) >= 0 ? key_range_bits(j0, klo, chi) : 0u) << (8 + 8 * i);
        }
        st.keep = keep;
      }
    } else {
      const int64_t o = ((int64_t)(tok0 + kb - P) * hkv + g) * (kHeadDim * 2);
      kbase = reinterpret_cast<const char *>(p.k_new) + o;
      vbase = reinterpret_cast<const char *>(p.v_new) + o;
      ko[0] = nk_off;
      vo[0] = nv_off;
      ko[1] = nk_off + 4 * row_bytes;
      vo[1] = nv_off + 4 * row_bytes;
      st.edge = kb < klo || kb + kWChunk - 1 > khi;
      if (st.edge) {
        // keys out of range read the chunk's last one in range (khi >= kb) and
        // are not kept
        uint32_t keep = 0u;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int jk = k_key(tid + kWThreads * i), jv = 8 * wave + 4 * i + (lane >> 4);
          ko[i] = (uint32_t)min(jk, khi - kb) * row_bytes + nk_dim;
          vo[i] = (uint32_t)min(jv, khi - kb) * row_bytes + nv_dim;
          keep |= (kb + jk >= klo && kb + jk <= khi ? 1u : 0u) << i;
          keep |= (kb + jv >= klo && kb + jv <= khi ? 0xFFu : 0u) << (8 + 8 * i);
        }
        st.keep = keep;
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      st.k[i] = ldg128_global(kbase + ko[i]);
      st.v[i] = ldg128_global(vbase + vo[i]);
    }
  };
  auto lds128 = [&](uint32_t off) { return reinterpret_cast<u32x4 *>(s_lds + off); };
  auto buf_off = [&](int buf) { return (uint32_t)__builtin_amdgcn_readfirstlane(buf * kWBufBytes); };
  // V^T bytes of dims 8 (lane % 16) + 2 (lane / 16) and + 1, keys 8 wave .. +7
  const uint32_t st_vrow = kWKBytes + ((((8 * (lane & 15)) >> 4) * 64 + ((8 * (lane & 15) + 2 * (lane >> 4)) & 15) +
                                        16 * wave) * 16) + (lane & 2 ? 16 : 0);
  // 4 x 4 transpose of dwords across the lanes l, l ^ 16, l ^ 32, l ^ 48.
  auto transpose4 = [&](const u32x4 &t, uint32_t (&w)[4]) {
    const auto a = __builtin_amdgcn_permlane32_swap(t[0], t[2], false, false);
    const auto bb = __builtin_amdgcn_permlane32_swap(t[1], t[3], false, false);
    const auto c = __builtin_amdgcn_permlane16_swap((uint32_t)a[0], (uint32_t)bb[0], false, false);
    const auto d = __builtin_amdgcn_permlane16_swap((uint32_t)a[1], (uint32_t)bb[1], false, false);
    w[0] = (uint32_t)c[0];
    w[1] = (uint32_t)c[1];
    w[2] = (uint32_t)d[0];
    w[3] = (uint32_t)d[1];
  };
  auto store = [&](int buf, const WStage &st0) {
    WStage st = st0;
    if (st.edge) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        st.k[i] = (st.keep >> i) & 1u ? st.k[i] : zero;
        st.v[i] = keep_bf16x8(st.v[i], (st.keep >> (8 + 8 * i)) & 0xFFu);
      }
    }
    const uint32_t bo = buf_off(buf);
    *lds128(bo + 16 * tid) = st.k[0];
    *lds128(bo + 16 * (tid + kWThreads)) = st.k[1];
    if (!st.vrow) {
      *lds128(bo + kWKBytes + 16 * tid) = st.v[0];
      *lds128(bo + kWKBytes + 16 * (tid + kWThreads)) = st.v[1];
    } else {
      // lanes l % 16 + 16 m hold keys 8 wave + 4 i + m (piece i) x dims
      // 8 (l % 16) .. +7; after the transposes lane m holds dims 2 m, 2 m + 1
      // of keys 8 wave .. +7, split into one V^T piece per dim
      uint32_t w[8];
      transpose4(st.v[0], *reinterpret_cast<uint32_t(*)[4]>(&w[0]));
      transpose4(st.v[1], *reinterpret_cast<uint32_t(*)[4]>(&w[4]));
      u32x4 lo, hi;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        lo[j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x05040100u);
        hi[j] = __builtin_amdgcn_perm(w[2 * j + 1], w[2 * j], 0x07060302u);
      }
      // Lanes whose block dt is odd store their two dims the other way round:
      // the dims of a store's lanes are 8 apart and would meet two of the sixteen
      // 16-byte bank groups, so they meet four (41.4 -> 39.2 us as above).
      const u32x4 v0 = lane & 2 ? hi : lo, v1 = lane & 2 ? lo : hi;
      *lds128(bo + st_vrow) = v0;
      *lds128(bo + (st_vrow ^ 16)) = v1;
    }
  };

  float m[kWCG], lsum[kWCG];  // m: running maximum in exp2 units
  f32x4 acc[kWCG][8];
#pragma unroll
  for (int cg = 0; cg < kWCG; ++cg) {
    m[cg] = -FLT_MAX;
    lsum[cg] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) acc[cg][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  const uint32_t op_lane = lane * 16;
  // One chunk: QK^T, masks, online softmax, PV. The exponentials are taken
  // against the running maximum as it stands; only if some lane's share of a
  // row sum (8 probabilities) exceeds 2^12 (an infinite one included) is the
  // exact column maximum formed, the maximum raised, the output and row sum
  // rescaled and the exponentials taken again (exact either way: numerator and
  // denominator share the maximum).
  auto chunk = [&](int buf, int kb, int kend) {  // kend: the chunk's last key that holds data
    const uint32_t a = buf_off(buf) + op_lane;
    f32x4 sc[2][kWCG];
#pragma unroll
    for (int ab = 0; ab < 2; ++ab)
#pragma unroll
      for (int cg = 0; cg < kWCG; ++cg) sc[ab][cg] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const u32x4 ka = *lds128(a + 1024 * t);
      const u32x4 kbv = *lds128(a + 4096 + 1024 * t);
#pragma unroll
      for (int cg = 0; cg < kWCG; ++cg) {
        sc[0][cg] = mfma16x16x32(ka, qf[cg][t], sc[0][cg]);
        sc[1][cg] = mfma16x16x32(kbv, qf[cg][t], sc[1][cg]);
      }
    }
    if (!(kb >= wint_lo && kb + kWChunk - 1 <= min(wint_hi, kend))) {
      // this lane's keys are kb + 8 q + e, e = 4 ab + i
      // (the rows' positions are formed here, in the masked chunks only: kept
      // across the loop they would cost registers)
      int row0 = wave * (16 * kWCG) + r;
      asm volatile("" : "+v"(row0));
      const int j0 = kb + 8 * q;
#pragma unroll
      for (int cg = 0; cg < kWCG; ++cg) {
        const int cpos = pfirst + ((row0 + 16 * cg) >> gshift);
        const int lo_e = max(cpos - W + 1 - j0, 0);
        const int hi_e = min(min(cpos, kend) - j0, 7);
        const uint32_t bits = hi_e < lo_e ? 0u : ((2u << hi_e) - 1u) & ~((1u << lo_e) - 1u);
#pragma unroll
        for (int ab = 0; ab < 2; ++ab)
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[ab][cg][i] = (bits >> (4 * ab + i)) & 1u ? sc[ab][cg][i] : -INFINITY;
      }
    }
    u32x4 pf[kWCG];
    float ts[kWCG];
    auto exps = [&]() {
#pragma unroll
      for (int cg = 0; cg < kWCG; ++cg) {
        float pr[8];
#pragma unroll
        for (int ab = 0; ab < 2; ++ab)
#pragma unroll
          for (int i = 0; i < 4; ++i) pr[4 * ab + i] = fast_exp2(fmaf(sc[ab][cg][i], c2, -m[cg]));
        ts[cg] = 0.f;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          pf[cg][jj] = pack_bf16x2(pr[2 * jj], pr[2 * jj + 1]);
          ts[cg] = dot2_bf16_ones(pf[cg][jj], ts[cg]);
        }
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    exps();
    bool raise = false;
#pragma unroll
    for (int cg = 0; cg < kWCG; ++cg) raise = raise || !(ts[cg] <= kWLaneSumLimit);
    if (__builtin_amdgcn_ballot_w64(raise) != 0) {
#pragma unroll
      for (int cg = 0; cg < kWCG; ++cg) {
        const float a8[8] = {sc[0][cg][0], sc[0][cg][1], sc[0][cg][2], sc[0][cg][3],
                             sc[1][cg][0], sc[1][cg][1], sc[1][cg][2], sc[1][cg][3]};
        const float cmax = max_xor32(max_xor16(max8(a8))) * c2;
        const bool up = cmax > m[cg];
        const float alpha = up ? fast_exp2(m[cg] - cmax) : 1.f;
        m[cg] = up ? cmax : m[cg];
        lsum[cg] *= alpha;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) acc[cg][dt] *= alpha;
      }
      exps();
    }
#pragma unroll
    for (int cg = 0; cg < kWCG; ++cg) lsum[cg] += ts[cg];
    // V^T operands in two batches of four (fewer registers live at once)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 vf[4];
#pragma unroll
      for (int d4 = 0; d4 < 4; ++d4) vf[d4] = *lds128(a + kWKBytes + 1024 * (4 * h + d4));
#pragma unroll
      for (int d4 = 0; d4 < 4; ++d4)
#pragma unroll
        for (int cg = 0; cg < kWCG; ++cg) acc[cg][4 * h + d4] = mfma16x16x32(vf[d4], pf[cg], acc[cg][4 * h + d4]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // ---- chunk loop: chunk c is computed from buffer c % 2 while chunk c + 1,
  // loaded a step ahead, is stored into the other one (chunk c - 1's, whose
  // reads the barrier that opens the step ended) and chunk c + 2's loads go out.
  WStage st;
  {
    WStage s0;  // both in flight (the accumulators are not live yet)
    fetch(0, s0);
    fetch(1, st);
    store(0, s0);
  }
  for (int c = 0; c < nch; ++c) {
    const int kb = chunk_base(c);
    __syncthreads();
    if (wact && kb + kWChunk - 1 >= wklo && kb <= wkhi) chunk(c % kWBufs, kb, c < ncached ? chi : khi);
    if (c + 1 < nch) store((c + 1) % kWBufs, st);
    fetch(c + 2, st);
  }

  // ---- normalise and write ----
#pragma unroll
  for (int cg = 0; cg < kWCG; ++cg) {
    const float l = sum_xor32(sum_xor16(lsum[cg]));
    const float inv = 1.f / l;
    const int row = wave * (16 * kWCG) + cg * 16 + r;
    const int po = row / G, head = row - po * G;
    const bool cval = q0 + po <= q1;
    uint16_t *orow = p.out + ((int64_t)(tok0 + q0 + (cval ? po : 0)) * hq + (int64_t)g * G + head) * kHeadDim;
    u32x2 w[8];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      w[dt][0] = pack_bf16x2(acc[cg][dt][0] * inv, acc[cg][dt][1] * inv);
      w[dt][1] = pack_bf16x2(acc[cg][dt][2] * inv, acc[cg][dt][3] * inv);
    }
    store_out_row(orow, w, q, cval);
  }
}

}  // namespace

hipError_t launch_prefill_window(const PrefillParams &p, hipStream_t stream) {
  if (p.ns <= 0 || p.max_chunk_len <= 0 || p.total_tokens <= 0) return hipSuccess;
  const int npos = kWRows / p.group;
  const int64_t ntq = (p.max_chunk_len + npos - 1) / npos;
  const int64_t pairs_per_xcd = ((int64_t)p.ns * p.hkv + kWXcds - 1) / kWXcds;
  const int64_t grid = pairs_per_xcd * ntq * kWXcds;
  return launch_kernel(p.pool.pg_shift == 4 ? prefill_window_kernel<true> : prefill_window_kernel<false>,
                       dim3((unsigned)grid), dim3(kWThreads), stream, p);
}

}  // namespace hswa
