"""The host plan that splits the keys of query tiles over workgroups: every key of every tile is
given to exactly one workgroup, within the plan's capacities (pure host code: no GPU needed)."""
import ctypes

import numpy as np
import pytest

KEY_TILE, ROWS, MAX_PARTS, MAX_PIECES, MAX_TILES, MAX_ENTRIES, XCD_ENTRIES = 64, 256, 32, 512, 256, 256, 64


class Item(ctypes.Structure):
    _fields_ = [(f, ctypes.c_int32) for f in ("xcd", "slot", "pair", "tile", "chunk", "chunks", "piece")]


@pytest.fixture(scope="module")
def plan(built_lib):
    lib = ctypes.CDLL(built_lib)
    items, merged = (Item * 20000)(), (Item * 512)()

    def call(lens, hkv, group, cus):
        arr = np.ascontiguousarray(lens, dtype=np.int32)
        n_merged = ctypes.c_int32()
        n = lib.ls_internal_split_prefill(len(arr), hkv, group, arr.ctypes.data_as(ctypes.c_void_p), cus, items,
                                          len(items), merged, len(merged), ctypes.byref(n_merged))
        assert n >= 0
        return list(items[:n]), list(merged[:n_merged.value])
    return call


def _check(lens, hkv, group, items, merged):
    qtok = ROWS // group
    n, c = np.array(lens).T
    want = {(s * hkv + g, t) for s in range(len(n)) for g in range(hkv) for t in range(-(-int(n[s]) // qtok))}
    parts = {}
    slots = {}
    for it in items:
        parts.setdefault((it.pair, it.tile), []).append((it.chunk, it.chunks, it.piece))
        slots.setdefault(it.xcd, []).append(it.slot)
    assert set(parts) == want
    assert all(sorted(v) == list(range(len(v))) for v in slots.values()) and all(0 <= x < 8 for x in slots)
    bases = {}
    for (pair, tile), got in parts.items():
        chunks = got[0][1]
        assert [k for k, _, _ in sorted(got)] == list(range(chunks)) and all(m == chunks for _, m, _ in got)
        if chunks > 1:
            assert chunks <= MAX_PARTS
            base = {p - k for k, _, p in got}
            assert len(base) == 1
            bases[(pair, tile)] = (base.pop(), chunks)
            # the kernel's bounds of part k: they join up over the tile's key tiles
            s = pair // hkv
            last = min((tile + 1) * qtok, int(n[s])) - 1
            tiles = -(-(int(c[s]) + last + 1) // KEY_TILE)
            bounds = [tiles * k // chunks for k in range(chunks + 1)]
            assert bounds[0] == 0 and bounds[-1] == tiles and bounds == sorted(bounds)
    pieces = [b + k for b, chunks in bases.values() for k in range(chunks)]
    assert len(set(pieces)) == len(pieces) <= MAX_PIECES and (not pieces or (min(pieces) == 0 and max(pieces) < MAX_PIECES))
    assert {(m.pair, m.tile): (m.piece, m.chunks) for m in merged} == bases and len(merged) == len(bases) <= MAX_TILES
    # runs of one entry: the same pair and part, tiles counting down
    for x in slots:
        own = sorted((it for it in items if it.xcd == x), key=lambda it: it.slot)
        runs = 1 + sum((a.pair, a.chunk, a.chunks, a.tile) != (b.pair, b.chunk, b.chunks, b.tile + 1)
                       for a, b in zip(own, own[1:]))
        assert runs <= XCD_ENTRIES


@pytest.mark.parametrize("cus", [256, 24, 200, 8])
@pytest.mark.parametrize("hkv", [1, 2, 4, 8])
def test_every_key_of_every_tile_once(plan, hkv, cus):
    rng = np.random.default_rng(hkv * 1000 + cus)
    split = 0
    for rep in range(150):
        S = int(np.exp(rng.uniform(0, np.log(256 // hkv + 0.5))))
        hi_n, hi_c = int(np.exp(rng.uniform(0, np.log(2048)))), int(np.exp(rng.uniform(0, np.log(32768))))
        lens = np.stack([rng.integers(0 if rep % 3 else 1, hi_n + 1, S), rng.integers(0, hi_c + 1, S)], 1)
        if rep % 10 == 0:
            lens[0, 1] = 262144 - lens[0, 0]
        group = int(rng.choice([1, 2, 4, 8]))
        items, merged = plan(lens, hkv, group, cus)
        if items:
            split += 1
            _check(lens, hkv, group, items, merged)
        else:
            assert not merged
    assert split > 10 or cus == 8


# One turn; a remainder of a second wave; a long turn beside few and beside so many short ones that
# its parts are more entries than the plan holds; the longest context; a batch of as many pairs as the
# plan holds, and of more; six waves of tiles; short contexts; no new tokens.
@pytest.mark.parametrize("lens,hkv,group,cus,split", [
    ([(301, 9043)], 4, 8, 256, True), ([(560, 6300), (560, 6100), (560, 6049), (560, 5500)], 4, 8, 256, True),
    ([(8, 30000)] + [(8, 100)] * 2, 8, 8, 256, True), ([(8, 30000)] + [(8, 100)] * 31, 8, 8, 256, False),
    ([(2048, 260000)], 1, 1, 256, True), ([(8, 9000)] * 64, 4, 8, 256, False), ([(8, 9000)] * 65, 4, 8, 256, False),
    ([(2048, 4000)] * 24, 4, 8, 256, False), ([(100, 100)] * 4, 4, 8, 256, False), ([(0, 5000)] * 4, 4, 8, 256, False)])
def test_chosen_batches(plan, lens, hkv, group, cus, split):
    items, merged = plan(lens, hkv, group, cus)
    assert bool(items) == split == bool(merged)
    if items:
        _check(lens, hkv, group, items, merged)
