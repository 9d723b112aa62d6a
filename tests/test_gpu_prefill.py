"""GPU parity of hswa_prefill against the fp64 oracle: chunks over cached
prefixes of many lengths (aligned and not), FULL and SWA windows from 1 to
beyond the context, GQA groups 1 to 64, page sizes 16 and 64, several
sequences of mixed lengths in one call."""

import numpy as np
import pytest
import torch

import synth
from oracle import attention as OA
from paper_2607_13095_amd import hswa
from paper_2607_13095_amd.kvcache import LayerKV, pages_for
from tests.hswa_testlib import (SeqHistory, append_history, assert_close, i32, make_layer, to_dev, to_f64)

pytestmark = pytest.mark.gpu


def run_prefill(kind, window, pg, hq, hkv, prefixes, chunks, seed, fill=float("nan"), perm_seed=None,
                max_chunk=None, scale=None):
    ns = len(prefixes)
    final = [p + c for p, c in zip(prefixes, chunks)]
    shape = hswa.Shape(hq, hkv, 128, pg, scale=scale)
    layer, kv = make_layer(kind, window, shape, final, perm_seed or seed, fill=fill)
    hist = SeqHistory(final, hkv, 128, *seed)
    append_history(layer, shape, kv, hist, [0] * ns, prefixes)
    T = sum(chunks)
    qbits = synth.normal_bf16((T, hq, 128), *seed, synth.TAG_Q)
    kn = np.concatenate([hist.k[b][p:p + c] for b, (p, c) in enumerate(zip(prefixes, chunks))])
    vn = np.concatenate([hist.v[b][p:p + c] for b, (p, c) in enumerate(zip(prefixes, chunks))])
    out = torch.full((T, hq, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    hswa.prefill(layer, shape, kv.cache, to_dev(qbits), to_dev(kn), to_dev(vn), i32(synth.cu_seqlens(chunks)),
                 i32(prefixes), max_chunk or max(chunks), out)
    torch.cuda.synchronize()
    gpu = to_f64(out)
    qf = OA.bf16_bits_to_f64(qbits)
    w = window if kind == "swa" else None
    refs, off = [], 0
    for b, (p, c) in enumerate(zip(prefixes, chunks)):
        refs.append(OA.prefill(qf[off:off + c], OA.bf16_bits_to_f64(hist.k[b]), OA.bf16_bits_to_f64(hist.v[b]), p, w,
                               shape.scale))
        off += c
    return gpu, np.concatenate(refs), (layer, shape, kv, hist, kn, vn)


PREFIXES = [0, 1, 127, 128, 200, 64, 0]
CHUNKS = [1, 15, 16, 17, 300, 129, 256]


@pytest.mark.parametrize("pg", [16, 64])
@pytest.mark.parametrize("kind,window", [("full", 0), ("swa", 1), ("swa", 4), ("swa", 128), ("swa", 129),
                                         ("swa", 100000)])
def test_prefill_mixed_batch(gpu_lib, pg, kind, window):
    print(f"[prefill] pg={pg} kind={kind} W={window}", flush=True)
    gpu, ref, _ = run_prefill(kind, window, pg, 64, 8, PREFIXES, CHUNKS, (300, pg, window))
    assert_close(gpu, ref, f"prefill {kind} W={window} PG={pg}")


@pytest.mark.parametrize("hq,hkv", [(8, 8), (8, 1), (16, 1), (64, 1), (32, 4)])
def test_prefill_groups(gpu_lib, hq, hkv):
    print(f"[prefill-groups] hq={hq} hkv={hkv}", flush=True)
    for kind, window in (("full", 0), ("swa", 128)):
        gpu, ref, _ = run_prefill(kind, window, 16, hq, hkv, [0, 300], [200, 77], (301, hq, hkv))
        assert_close(gpu, ref, f"prefill groups {kind} hq={hq} hkv={hkv}")


@pytest.mark.parametrize("hq,hkv", [(32, 32), (64, 16)])
def test_prefill_many_kv_heads(gpu_lib, hq, hkv):
    """More KV heads than the configs' 8: chunk rows of Hkv * 256 bytes, read by
    the full-chunk-tile buffer loads at per-lane row offsets, and page-heads of
    Hkv * PG * 256 bytes for the interior tiles (PG 64); FULL, and SWA with a
    window that takes the FULL kernel's masked path."""
    print(f"[prefill-many-kv] hq={hq} hkv={hkv}", flush=True)
    for kind, window in (("full", 0), ("swa", 1000)):
        gpu, ref, _ = run_prefill(kind, window, 64, hq, hkv, [0, 130, 1100], [300, 200, 129], (308, hq, hkv))
        assert_close(gpu, ref, f"prefill many KV heads {kind} hq={hq} hkv={hkv}")


def test_prefill_long_chunk_over_prefix(gpu_lib):
    """A 2048-token chunk over a 1000-token prefix, FULL and SWA (wraps the ring)."""
    for kind, window in (("full", 0), ("swa", 128)):
        gpu, ref, _ = run_prefill(kind, window, 64, 64, 8, [1000, 3], [2048, 700], (302,))
        assert_close(gpu, ref, f"long chunk {kind}")


def test_prefill_empty_chunks(gpu_lib):
    """Sequences with an empty chunk in the batch are skipped; max_chunk_len 0 is a no-op."""
    gpu, ref, _ = run_prefill("full", 0, 16, 8, 1, [5, 0, 40], [3, 0, 20], (303,))
    assert_close(gpu, ref, "empty chunk in batch")


@pytest.mark.parametrize("scale", [1.0, 4.0])
def test_prefill_large_scale(gpu_lib, scale):
    """Scales above ln 2 (scale * log2 e > 1, e.g. queries that arrive
    pre-scaled): the running maximum starts finite in exp2 units, so a column
    whose first tile is wholly masked (SWA rows whose window starts past the
    workgroup's first tile) gets no NaN. The 512-token SWA prefill (8 / 1 heads,
    PG 16) and a chunk over a cached prefix at 64 / 8 heads, PG 64."""
    print(f"[prefill-scale] scale={scale}", flush=True)
    gpu, ref, _ = run_prefill("swa", 128, 16, 8, 1, [0], [512], (304, 1), scale=scale)
    assert_close(gpu, ref, f"swa prefill 512, scale {scale}")
    for kind, window in (("swa", 128), ("full", 0)):
        gpu, ref, _ = run_prefill(kind, window, 64, 64, 8, [1000, 3], [2048, 700], (304, 2), scale=scale)
        assert_close(gpu, ref, f"{kind} prefill over a prefix, scale {scale}")


@pytest.mark.parametrize("hq,hkv,window", [(64, 8, 129), (64, 8, 130), (128, 8, 145), (128, 8, 146),
                                           (32, 8, 512), (32, 8, 513), (64, 8, 33)])
def test_prefill_window_kernel_boundaries(gpu_lib, hq, hkv, window):
    """SWA prefill takes one of three kernels: with a GQA group G >= 8 and
    W + 256 / G - 1 <= 160 the persistent one over runs of tiles, otherwise up
    to W = 512 the per-tile windowed one, and beyond that the FULL-style one.
    Each side of both limits, over prefixes that put window starts before,
    across and after the prefix / chunk boundary (PG 16 and 64), against the
    oracle."""
    print(f"[prefill-boundaries] hq={hq} hkv={hkv} W={window}", flush=True)
    for pg in (16, 64):
        gpu, ref, _ = run_prefill("swa", window, pg, hq, hkv, [0, 37, 300, 1000], [700, 333, 64, 900],
                                  (305, hq, window, pg))
        assert_close(gpu, ref, f"prefill W={window} hq={hq} hkv={hkv} PG={pg}")


# Tiles of cached keys over every page class: prefixes around tile, page and
# block-table-window edges (64 table entries: 1024 keys of 16-key pages, 2048 of
# 32-key ones), a window past the windowed kernels' range with a ring and with
# released pages: (page size, window, prefix, chunk)
CACHED_TILE_CASES = [
    (16, 0, 1, 70), (16, 0, 15, 3), (16, 0, 63, 130), (16, 0, 64, 64), (16, 0, 65, 1), (16, 0, 1023, 20),
    (16, 0, 1040, 90), (16, 0, 2113, 33), (32, 0, 31, 65), (32, 0, 33, 64), (32, 0, 2047, 40), (32, 0, 4200, 17),
    (64, 0, 63, 129), (64, 0, 4097, 30), (128, 0, 130, 100), (256, 0, 300, 64), (16, 600, 1700, 100),
    (32, 700, 2500, 80), (64, 513, 1111, 200), (128, 1000, 1500, 65),
]


@pytest.mark.parametrize("pg,window,prefix,chunk", CACHED_TILE_CASES)
def test_prefill_cached_tiles(gpu_lib, pg, window, prefix, chunk):
    print(f"[prefill-tiles] PG={pg} W={window} P={prefix} C={chunk}", flush=True)
    hq, hkv, d = 8, 2, 128
    shape = hswa.Shape(hq, hkv, d, pg)
    lens = [prefix, max(0, prefix - 17)]
    final = [p + chunk for p in lens]
    kind = "swa" if window else "full"
    layer, kv = make_layer(kind, window, shape, final, (203, pg, prefix))  # NaN in every unused slot
    hist = SeqHistory(final, hkv, d, 203, pg, prefix)
    append_history(layer, shape, kv, hist, [0, 0], lens)
    qb = synth.normal_bf16((2 * chunk, hq, d), 203, pg, prefix, synth.TAG_Q)
    kn = np.concatenate([hist.k[b][p:] for b, p in enumerate(lens)])
    vn = np.concatenate([hist.v[b][p:] for b, p in enumerate(lens)])
    out = torch.full((2 * chunk, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    hswa.prefill(layer, shape, kv.cache, to_dev(qb), to_dev(kn), to_dev(vn), i32([0, chunk, 2 * chunk]), i32(lens),
                 chunk, out)
    torch.cuda.synchronize()
    gpu, qf = to_f64(out), OA.bf16_bits_to_f64(qb)
    for b, p in enumerate(lens):
        ref = OA.prefill(qf[b * chunk:(b + 1) * chunk], OA.bf16_bits_to_f64(hist.k[b]),
                         OA.bf16_bits_to_f64(hist.v[b]), p, window or None)
        assert_close(gpu[b * chunk:(b + 1) * chunk], ref, f"PG {pg} W {window} P {p}")


@pytest.mark.parametrize("pg", [16, 32, 64])
def test_prefill_invalid_page_reads_as_zero(gpu_lib, pg):
    """A cached page whose table entry is invalid counts as zero keys and values."""
    print(f"[prefill-invalid] PG={pg}", flush=True)
    hq, hkv, d, prefix, chunk = 8, 2, 128, 200, 40
    shape = hswa.Shape(hq, hkv, d, pg)
    layer, kv = make_layer("full", 0, shape, [prefix + chunk], (204, pg))
    hist = SeqHistory([prefix + chunk], hkv, d, 204, pg)
    append_history(layer, shape, kv, hist, [0], [prefix])
    qb = synth.normal_bf16((chunk, hq, d), 204, pg, synth.TAG_Q)
    kf, vf = OA.bf16_bits_to_f64(hist.k[0]), OA.bf16_bits_to_f64(hist.v[0])
    for entry, bad in ((1, -1), (192 // pg, kv.num_pages)):  # a whole tile's page, and the last (partial) tile's
        saved = int(kv.block_table[0, entry])
        kv.block_table[0, entry] = bad
        k, v = kf.copy(), vf.copy()
        k[entry * pg:min(prefix, (entry + 1) * pg)] = 0
        v[entry * pg:min(prefix, (entry + 1) * pg)] = 0
        out = torch.full((chunk, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        hswa.prefill(layer, shape, kv.cache, to_dev(qb), to_dev(hist.k[0][prefix:]), to_dev(hist.v[0][prefix:]),
                     i32([0, chunk]), i32([prefix]), chunk, out)
        torch.cuda.synchronize()
        kv.block_table[0, entry] = saved
        assert_close(to_f64(out), OA.prefill(OA.bf16_bits_to_f64(qb), k, v, prefix, None), f"PG {pg} entry {entry}")


@pytest.mark.parametrize("pg,hq,hkv,prefixes,chunks", [
    (64, 16, 2, [5000], [33]),                        # one tile row, cut into many pieces
    (16, 8, 1, [3001, 0, 700], [70, 1, 129]),         # pieces inside the cached and the new keys
    (32, 8, 4, [1100, 0, 64, 2047], [90, 0, 300, 5]),  # an empty chunk; 128 positions a tile
    (128, 64, 1, [1024], [9]),                        # four positions a tile, no key past the first page run
    (64, 32, 8, [0], [1500]),                         # no cached key: causal tiles of unequal length
])
def test_prefill_split(gpu_lib, pg, hq, hkv, prefixes, chunks):
    """Calls cut into spans of key tiles, against the oracle and the unsplit call
    (both round the same fp32 sums, taken in another order, to bf16)."""
    print(f"[prefill-split] pg={pg} {hq}/{hkv} {prefixes} {chunks}", flush=True)
    gpu, ref, (layer, shape, kv, hist, kn, vn) = run_prefill("full", 0, pg, hq, hkv, prefixes, chunks,
                                                             (205, pg, hq, hkv))
    ns, t, mc = len(chunks), sum(chunks), max(chunks)
    lib, sh, ca = hswa.load(), shape.c(), kv.cache.c()
    need = lib.hswa_prefill_workspace_bytes(layer.c(), sh, ca, ns, t, mc)
    assert need > 0
    assert_close(gpu, ref, f"split prefill {prefixes} {chunks}")
    q = to_dev(synth.normal_bf16((t, hq, 128), 205, pg, hq, hkv, synth.TAG_Q))
    k, v, cu, pre = to_dev(kn), to_dev(vn), i32(synth.cu_seqlens(chunks)), i32(prefixes)
    out = torch.full((t, hq, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    ptr = [x.data_ptr() for x in (q, k, v, cu, pre)]
    stream = torch.cuda.current_stream().cuda_stream
    assert lib.hswa_prefill(layer.c(), sh, ca, *ptr, ns, t, mc, out.data_ptr(), stream) == 0
    torch.cuda.synchronize()
    assert_close(gpu, to_f64(out), f"split against unsplit {prefixes} {chunks}")
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    assert lib.hswa_prefill_ws(layer.c(), sh, ca, *ptr, ns, t, mc, ws.data_ptr(), 256, out.data_ptr(), stream) == -3


@pytest.mark.parametrize("prefix,chunk", [(130, 70), (0, 40), (1500, 40)])
def test_prefill_split_table_larger_than_context(gpu_lib, prefix, chunk):
    """Scratch is taken by what the block table can hold; contexts far shorter
    than that run as whole tiles (the first two) or in short spans."""
    print(f"[prefill-split] table for 9000, {chunk} over {prefix}", flush=True)
    shape = hswa.Shape(32, 4, 128, 64)
    layer, kv = make_layer("full", 0, shape, [9000], (206, prefix))
    hist = SeqHistory([prefix + chunk], 4, 128, 206, prefix)
    append_history(layer, shape, kv, hist, [0], [prefix])
    assert hswa.load().hswa_prefill_workspace_bytes(layer.c(), shape.c(), kv.cache.c(), 1, chunk, chunk) > 0
    qb = synth.normal_bf16((chunk, 32, 128), 206, prefix, synth.TAG_Q)
    out = torch.full((chunk, 32, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    hswa.prefill(layer, shape, kv.cache, to_dev(qb), to_dev(hist.k[0][prefix:]), to_dev(hist.v[0][prefix:]),
                 i32([0, chunk]), i32([prefix]), chunk, out)
    torch.cuda.synchronize()
    ref = OA.prefill(OA.bf16_bits_to_f64(qb), OA.bf16_bits_to_f64(hist.k[0]), OA.bf16_bits_to_f64(hist.v[0]), prefix,
                     None)
    assert_close(to_f64(out), ref, f"{chunk} over {prefix}")


def _split_and_unsplit(hq, hkv, pg, prefixes, chunks, width):
    """hswa_prefill_ws (through the binding) and hswa_prefill on a block table of
    `width` positions a sequence, with random pools."""
    shape, layer = hswa.Shape(hq, hkv, 128, pg), hswa.Layer.full()
    final = [a + b for a, b in zip(prefixes, chunks)]
    kv = LayerKV(layer, shape, final, perm=np.random.default_rng(3).permutation(pages_for(layer, pg, final)), fill=0.0,
                 stride=max(width // pg, max(-(-n // pg) for n in final)))
    g = torch.Generator(device="cuda").manual_seed(9)
    for pool in (kv.k_pool, kv.v_pool):
        pool.normal_(generator=g)
    t, ns = sum(chunks), len(chunks)
    q, k, v = (torch.randn((t, h, 128), generator=g, device="cuda").to(torch.bfloat16) for h in (hq, hkv, hkv))
    cu, pre, mc = i32(synth.cu_seqlens(chunks)), i32(prefixes), max(chunks)
    args = (layer.c(), shape.c(), kv.cache.c())
    assert hswa.load().hswa_prefill_workspace_bytes(*args, ns, t, mc) > 0
    cut, unsplit = (torch.full((t, hq, 128), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    hswa.prefill(layer, shape, kv.cache, q, k, v, cu, pre, mc, cut)
    assert hswa.load().hswa_prefill(*args, q.data_ptr(), k.data_ptr(), v.data_ptr(), cu.data_ptr(), pre.data_ptr(), ns,
                                    t, mc, unsplit.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return cut, unsplit


@pytest.mark.parametrize("hq,hkv,pg,prefixes,chunks,cuts", [
    (64, 8, 64, [0], [300], False),
    (64, 8, 64, [0], [1500], False),                       # more tiles than workgroups of the cut
    (64, 8, 64, [1000] * 8, [64] * 8, False),
    (64, 8, 16, [0] * 4, [600, 1, 0, 577], False),         # an empty sequence, part tiles
    (24, 12, 32, [50] * 3, [300, 30, 600], False),         # heads that do not divide over the XCDs
    (8, 1, 64, [0] * 70, [20] * 70, False),                # more sequences than lanes
    (64, 8, 64, [64], [700], False),
    (64, 8, 64, [4000], [600], True),
    (16, 16, 64, [0], [1000], True),                       # few tiles, whatever the prefix
    (48, 3, 64, [0, 300], [900, 2000], True),
    (8, 1, 64, [0] * 69 + [6000], [20] * 70, True),        # one long context among many short ones
    (32, 8, 16, [463, 750, 695, 2957], [446, 1471, 731, 615], True),
])
def test_prefill_cut_by_lengths(gpu_lib, hq, hkv, pg, prefixes, chunks, cuts):
    """Whether a call is cut into spans follows from its lengths, not from the
    width of its block table: one that does not gain works as the unsplit call,
    bit for bit (no sum is taken in another order), one that gains is cut."""
    print(f"[prefill-cut] {hq}/{hkv} PG={pg} {prefixes[-1]} {chunks[:4]} ns={len(chunks)}", flush=True)
    for width in (32768, 131072):
        cut, unsplit = _split_and_unsplit(hq, hkv, pg, prefixes, chunks, width)
        assert not torch.isnan(unsplit).any()
        assert torch.equal(cut, unsplit) != cuts, f"table of {width}"
        assert_close(to_f64(cut), to_f64(unsplit), f"table of {width}")


def test_prefill_max_context_takes_no_scratch(gpu_lib, monkeypatch):
    """A call that cannot gain within max_context asks for no scratch; the bound
    changes no value, also where it is too small."""
    shape, layer = hswa.Shape(64, 8, 128, 64), hswa.Layer.full()
    kv = LayerKV(layer, shape, [5000], fill=0.0, stride=2048)
    kv.k_pool.normal_(), kv.v_pool.normal_()
    taken = []
    scratch = hswa._prefill_scratch
    monkeypatch.setattr(hswa, "_prefill_scratch", lambda n, s: taken.append(n) or scratch(n, s))
    for prefix, chunk, bounds in ((0, 1500, {None: 1, 1500: 0, 2048 * 64: 1, 10**12: 1}), (4000, 100, {None: 1, 4100: 1, 1: 0})):
        q, k, v = (torch.randn((chunk, h, 128), device="cuda").to(torch.bfloat16) for h in (64, 8, 8))
        outs = []
        for bound, calls in bounds.items():
            out = torch.full((chunk, 64, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
            taken.clear()
            hswa.prefill(layer, shape, kv.cache, q, k, v, i32([0, chunk]), i32([prefix]), chunk, out, max_context=bound)
            assert len(taken) == calls, (prefix, bound)
            outs.append(to_f64(out))
        for o in outs[1:]:
            assert_close(o, outs[0], f"{chunk} over {prefix}")


@pytest.mark.parametrize("pg", [16, 32, 64, 256])
@pytest.mark.parametrize("prefix", [480, 509])
def test_prefill_window_pages(gpu_lib, pg, prefix):
    """The windowed kernel over every kind of page, with an invalid ring entry
    inside the window (a zero key and value) and NaN in unused slots."""
    print(f"[prefill-window] PG={pg} P={prefix}", flush=True)
    hq, hkv, d, window, chunk = 16, 2, 128, 200, 75
    shape = hswa.Shape(hq, hkv, d, pg)
    layer, kv = make_layer("swa", window, shape, [prefix + chunk], (207, pg))
    hist = SeqHistory([prefix + chunk], hkv, d, 207, pg)
    append_history(layer, shape, kv, hist, [0], [prefix])
    qb = synth.normal_bf16((chunk, hq, d), 207, pg, synth.TAG_Q)
    kf, vf = OA.bf16_bits_to_f64(hist.k[0]), OA.bf16_bits_to_f64(hist.v[0])
    for bad in (None, 400 // pg):
        if bad is not None:
            kv.block_table[0, bad % hswa.ring_pages(window, pg)] = -1
            kf[bad * pg:min(prefix, (bad + 1) * pg)] = 0
            vf[bad * pg:min(prefix, (bad + 1) * pg)] = 0
        out = torch.full((chunk, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        hswa.prefill(layer, shape, kv.cache, to_dev(qb), to_dev(hist.k[0][prefix:]), to_dev(hist.v[0][prefix:]),
                     i32([0, chunk]), i32([prefix]), chunk, out)
        torch.cuda.synchronize()
        assert_close(to_f64(out), OA.prefill(OA.bf16_bits_to_f64(qb), kf, vf, prefix, window), f"PG {pg} bad {bad}")


def _swa_prefill_us(prefix):
    """us per SWA prefill of 4 x 16 tokens (64 / 8 heads, W = 128), from replays of a graph."""
    shape, layer = hswa.Shape(64, 8, 128, 64), hswa.Layer.swa(128)
    kv = LayerKV(layer, shape, [prefix + 16] * 4, fill=0.0)
    q = torch.randn((64, 64, 128), device="cuda").to(torch.bfloat16)
    k = torch.randn((64, 8, 128), device="cuda").to(torch.bfloat16)
    cu, pre, out = i32(range(0, 65, 16)), i32([prefix] * 4), torch.empty_like(q)
    call = lambda: hswa.prefill(layer, shape, kv.cache, q, k, k, cu, pre, 16, out)  # noqa: E731
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(20):
            call()
    times = []
    for _ in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        graph.replay()
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 50)
    return min(times)


def test_prefill_short_range_loads_its_own_chunks(gpu_lib):
    """A short chunk over no prefix does not pay for the chunks of a whole window
    (7.5 us; 8.9 with every chunk of the ring loaded. Over a full window 11.8)."""
    short, full = _swa_prefill_us(0), _swa_prefill_us(2000)
    print(f"[prefill-short] no prefix {short:.2f} us, over 2000 {full:.2f} us", flush=True)
    assert short < 0.72 * full
