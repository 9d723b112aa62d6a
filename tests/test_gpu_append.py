"""GPU parity of hswa_kv_append: slot mapping and pool bytes are bit-exact
against the layout oracle, including ring-wrap eviction for SWA layers."""

import numpy as np
import pytest
import torch

import synth
from oracle import layout as OL
from paper_2607_13095_amd import hswa
from tests.hswa_testlib import append_history, make_layer, SeqHistory, to_bits

pytestmark = pytest.mark.gpu

NAN_BITS = None


def _check_pools(kv, exp_k, exp_v):
    got_k, got_v = to_bits(kv.k_pool), to_bits(kv.v_pool)
    assert np.array_equal(got_k, exp_k)
    assert np.array_equal(got_v, exp_v)


# (kind, window, page size, Hkv, list of append calls: per call, per seq: (start, end))
CASES = [
    ("full", 0, 16, 1, [[(0, 37), (0, 16), (0, 1)]]),
    ("full", 0, 64, 8, [[(0, 130), (0, 64)], [(130, 131), (64, 200)]]),
    ("swa", 4, 16, 2, [[(0, 9), (0, 40)], [(9, 10), (40, 41)], [(10, 50), (41, 42)]]),
    ("swa", 128, 16, 1, [[(0, 512)]]),
    ("swa", 128, 64, 8, [[(0, 300), (0, 129), (0, 5)], [(300, 301), (129, 130), (5, 6)], [(301, 700), (130, 140), (6, 7)]]),
    ("swa", 1, 16, 1, [[(0, 33)], [(33, 34)]]),
    ("swa", 129, 64, 8, [[(0, 1000)], [(1000, 1008)], [(1008, 1017)]]),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_append_bit_exact(gpu_lib, case):
    kind, window, pg, hkv, calls = CASES[case]
    print(f"[append] case={case} kind={kind} W={window} PG={pg} Hkv={hkv}", flush=True)
    shape = hswa.Shape(hkv * 2, hkv, 128, pg)
    ns = len(calls[0])
    final = [max(c[b][1] for c in calls) for b in range(ns)]
    layer, kv = make_layer(kind, window, shape, final, (100, case))
    hist = SeqHistory(final, hkv, 128, 100, case)
    exp_k, exp_v = to_bits(kv.k_pool), to_bits(kv.v_pool)
    okind = OL.SWA if kind == "swa" else OL.FULL
    for call in calls:
        starts = [s for s, _ in call]
        ends = [e for _, e in call]
        slots = append_history(layer, shape, kv, hist, starts, ends)
        exp_slots = OL.slot_mapping(okind, window or None, pg, kv.table_host, starts,
                                    [e - s for s, e in call])
        assert np.array_equal(slots, exp_slots), "slot mapping differs from the oracle"
        kn = np.concatenate([hist.k[b][s:e] for b, (s, e) in enumerate(call)])
        vn = np.concatenate([hist.v[b][s:e] for b, (s, e) in enumerate(call)])
        exp_k, exp_v = OL.apply_append(exp_k, exp_v, exp_slots, kn, vn)
        torch.cuda.synchronize()
        _check_pools(kv, exp_k, exp_v)
    # the oracle's view of which ring slot holds which position agrees as well
    if kind == "swa":
        r = OL.ring_pages(window, pg)
        for b in range(ns):
            for (entry, off), pos in OL.ring_positions(window, pg, final[b]).items():
                page = kv.table_host[b][entry]
                assert np.array_equal(OL.k_rows(to_bits(kv.k_pool), page, off), hist.k[b][pos])
        assert r == hswa.ring_pages(window, pg)


def test_append_empty_and_noop(gpu_lib):
    shape = hswa.Shape(8, 1, 128, 16)
    layer, kv = make_layer("full", 0, shape, [16], (101,))
    before = to_bits(kv.k_pool)
    empty = torch.empty((0, 1, 128), dtype=torch.bfloat16, device="cuda")
    hswa.kv_append(layer, shape, kv.cache, empty, empty, torch.tensor([0, 0], dtype=torch.int32, device="cuda"),
                   torch.tensor([0], dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    assert np.array_equal(before, to_bits(kv.k_pool))


# Runs of 32 positions, their edges, and sequences on both sides of the lengths
# that are scattered token by token: (kind, window, page size, Hkv, [(start, count)] per sequence)
RUN_CASES = [
    # all counts around 8 and 32 from every alignment of a 16-byte piece
    ("full", 0, 16, 2, [(3 * i, c) for i, c in enumerate([7, 8, 9, 31, 32, 33, 63, 64, 65, 97, 1, 200])]),
    ("full", 0, 32, 1, [(5 + 7 * i, c) for i, c in enumerate([33, 32, 31, 64, 96, 100, 1, 2, 300])]),
    ("full", 0, 128, 3, [(8 * i, c) for i, c in enumerate([40, 8, 9, 500, 129])]),
    # long chunks next to single decode tokens in one call (a mixed step)
    ("full", 0, 64, 2, [(100, 1000)] + [(17 * i, 1) for i in range(40)] + [(31, 333)]),
    # short appends only: the 8-token tiles, with sequences of up to 31 tokens
    ("full", 0, 64, 4, [(11 * i, 1 + i % 31) for i in range(50)]),
    # rings: the call evicts its own first tokens, or keeps them all
    ("swa", 128, 16, 1, [(0, 700), (37, 150), (5, 9), (500, 161)]),
    ("swa", 33, 32, 2, [(0, 95), (1, 96), (2, 97), (3, 1), (64, 64)]),
    # more sequences than the LDS copy of cu_seqlens holds
    ("full", 0, 16, 1, [(i % 16, 1 + (i % 500 == 0) * 40) for i in range(4100)]),
    # 8-token tiles of eight tokens on aligned slots, next to tiles whose batch
    # offset, position or page breaks the row, and a last tile that is not full
    ("full", 0, 16, 2, [(8, 8), (16, 16), (0, 1), (24, 7), (4, 8), (0, 8), (120, 24), (0, 5)]),
    ("full", 0, 64, 1, [(64, 256)] + [(31 * i, 1) for i in range(300)]),
    ("swa", 20, 16, 1, [(0, 120), (40, 8), (48, 88)]),
    # many short sequences in a tile: runs of eight and more tokens, single ones between
    ("full", 0, 64, 2, [(8 * i, 8) for i in range(20)] + [(0, 600)] + [(5 * i, 1 + i % 9) for i in range(12)]),
    ("full", 0, 16, 1, [(3 * i, 17 + i % 3) for i in range(40)]),
]


@pytest.mark.parametrize("case", range(len(RUN_CASES)))
@pytest.mark.parametrize("heads", [0, 8])
def test_append_runs_bit_exact(gpu_lib, heads, case):
    """With the case's own head count, and with 8 (few heads take 8-token tiles)."""
    kind, window, pg, hkv, seqs = RUN_CASES[case]
    hkv = heads or hkv
    print(f"[append-runs] case={case} kind={kind} W={window} PG={pg} Hkv={hkv} ns={len(seqs)}", flush=True)
    shape = hswa.Shape(hkv, hkv, 128, pg)
    starts = [s for s, _ in seqs]
    final = [s + c for s, c in seqs]
    layer, kv = make_layer(kind, window, shape, final, (101, case))
    hist = SeqHistory(final, hkv, 128, 101, case)
    exp_k, exp_v = to_bits(kv.k_pool), to_bits(kv.v_pool)
    slots = append_history(layer, shape, kv, hist, starts, final)
    exp_slots = OL.slot_mapping(OL.SWA if kind == "swa" else OL.FULL, window or None, pg, kv.table_host, starts,
                                [c for _, c in seqs])
    assert np.array_equal(slots, exp_slots), "slot mapping differs from the oracle"
    kn = np.concatenate([hist.k[b][s:s + c] for b, (s, c) in enumerate(seqs)])
    vn = np.concatenate([hist.v[b][s:s + c] for b, (s, c) in enumerate(seqs)])
    exp_k, exp_v = OL.apply_append(exp_k, exp_v, exp_slots, kn, vn)
    torch.cuda.synchronize()
    _check_pools(kv, exp_k, exp_v)


def _append_us(starts, count):
    """us per append of `count` tokens to each sequence (8 heads, PG 64)."""
    shape = hswa.Shape(8, 8, 128, 64)
    layer, kv = make_layer("full", 0, shape, [s + count for s in starts], (102,))
    n = len(starts) * count
    k = torch.randn((n, 8, 128), device="cuda").to(torch.bfloat16)
    cu = torch.arange(0, n + 1, count, dtype=torch.int32, device="cuda")
    pos = torch.tensor(starts, dtype=torch.int32, device="cuda")
    times = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        hswa.kv_append(layer, shape, kv.cache, k, k, cu, pos)
        a.record()
        for _ in range(20):
            hswa.kv_append(layer, shape, kv.cache, k, k, cu, pos)
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 50)
    return min(times)


def test_append_aligned_tokens_take_wide_stores(gpu_lib):
    """Eight tokens on aligned slots are one 16-byte V store a dim, not eight
    2-byte ones: 1000 x 8 tokens take about half the time of the same tokens
    three positions on (25 against 46 us)."""
    aligned, shifted = _append_us([8 * (i % 64) for i in range(1000)], 8), _append_us([8 * (i % 64) + 3 for i in range(1000)], 8)
    print(f"[append-wide] aligned {aligned:.1f} us, shifted {shifted:.1f} us", flush=True)
    assert aligned < 0.75 * shifted
