"""The plans of key tiles in pieces and of key loops in parts (host arithmetic): every part of every tile and workgroup once, those with
sums next to one another where the slots say, all within the bounds of kernel arguments and slots; and the host time that a plan may take."""
import random
import time

import pytest

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W

HEADS = [(4, 2), (28, 4), (32, 8), (40, 8), (6, 3), (8, 1), (16, 16), (64, 1)]


def packings():
    rng = random.Random(5)
    fixed = [([1024], [8], [256] * 8), ([60, 60], [26, 26], [85] * 52), ([8192], [16], W.ragged_lengths(5100, 16, 64, 256)), ([1400, 1089], [4, 2], [20, 5, 0, 33, 1, 70]),
             ([28] * 27, [19] * 27, [41] * 27 * 19), ([58] * 27, [17] * 27, [14] * 27 * 17), ([23] * 24, [21] * 24, [7] * 24 * 21), ([100], [0], []), ([0], [1], [1500])]
    for p in fixed:
        yield from ((*p, *h) for h in HEADS)
    for _ in range(300):
        n = rng.choice((1, 1, 2, 3, 8, 30))
        prompt, resp = int(2 ** rng.uniform(0, 13)), int(2 ** rng.uniform(0, 10))
        Gs = [rng.randint(0, 24) for _ in range(n)]
        yield [rng.randint(prompt // 3, prompt) + 1 for _ in range(n)], Gs, [rng.randint(0, resp) for _ in range(sum(Gs))], *rng.choice(HEADS)


def groups(pl, Gs, rl):
    at = 0
    for p, G in zip(pl, Gs):
        yield p, rl[at:at + G]
        at += G


@pytest.mark.parametrize("flags", [0, B.SP_FLAG_RESPONSE_ROWS])
def test_every_key_tile_is_walked_once(flags):
    planned = 0
    for pl, Gs, rl, hq, hkv in packings():
        words, sums, _, n_slots = B.sp_attn_pieces(pl, Gs, rl, hq, hkv, flags)
        if not words:
            assert not sums and n_slots == 0
            continue
        planned += 1
        tokens, at = [], 0                                   # a tile's first packed token, and its keys
        for p, r in groups(pl, Gs, rl):
            total = p + sum(r)
            tokens += [(at + s, min(128, total - s)) for s in range(0, total, 128)]
            at += total
        assert len(words) <= 768 and n_slots * hkv <= 384 and n_slots * hkv * 131072 <= B.sums_bytes(at, len(pl), hq, hkv, B.SP_BF16)
        parts = {}
        for w in words:
            parts.setdefault(w & 0xffff, []).append((w >> 16 & 0xff, w >> 24))
        assert sorted(parts) == list(range(len(tokens)))
        assert all(p == [(i, len(p)) for i in range(len(p))] for p in parts.values())
        slot = 0
        for a, tok in zip(sums[::2], sums[1::2]):
            first, n, keys = a & 0xffff, a >> 16 & 0xff, (a >> 24) + 1
            tile = words[first] & 0xffff
            assert first == slot and n > 1 and [w & 0xffff for w in words[first:first + n]] == [tile] * n and tokens[tile] == (tok, keys)
            slot += n
        assert slot == n_slots > 0 and all(w >> 24 == 1 for w in words[slot:])
    assert planned > 40


@pytest.mark.parametrize("flags", [0, B.SP_FLAG_RESPONSE_ROWS])
def test_every_key_loop_is_walked_once(flags):
    planned, whole = 0, []
    for pl, Gs, rl, hq, hkv in packings():
        words, sums, first_slot, n_slots = B.sp_attn_pieces(pl, Gs, rl, hq, hkv, flags, of_rows=True)
        if not words:
            assert not sums and n_slots == 0
            continue
        planned += 1
        rep, want, bases, at = hq // hkv, set(), [], 0
        for p, r in groups(pl, Gs, rl):
            total = p + sum(r)
            n = -(-total // 128)
            for ti in range(n):                              # row tiles from the group's end, four waves of 32 rows over `rep` heads each
                base = (n - 1 - ti) * 128
                for hr in range(rep):
                    i = rep - 1 - hr
                    t0, t1 = base + 32 * (4 * i // rep), min(base + 32 * ((4 * i + 3) // rep) + 32, total)
                    if t0 < total and not (flags and t1 <= p):
                        want.add((len(bases), hr))
                bases.append(at + base)
            at += total
        assert len(words) <= 768 and len(sums) // 3 <= 240 and n_slots * hkv * 67584 <= B.sums_bytes(at, len(pl), hq, hkv, B.SP_BF16)
        parts = {}
        for w in words:
            parts.setdefault((w & 1023, w >> 10 & 63), []).append((w >> 16 & 0xff, w >> 24))
        assert set(parts) == want
        assert all(p == [(i, len(p)) for i in range(len(p))] for p in parts.values())
        slot = 0
        for a, tok, i in zip(sums[::3], sums[1::3], sums[2::3]):
            first, n = a & 0xffff, a >> 16
            w = words[first_slot + first]
            assert first == slot and n > 1 and [x & 0xffff for x in words[first_slot + first:first_slot + first + n]] == [w & 0xffff] * n
            assert bases[w & 1023] == tok and rep - 1 - (w >> 10 & 63) == i
            slot += n
        assert slot == n_slots > 0 and all(w >> 24 == 1 for w in words[:first_slot] + words[first_slot + slot:])
        whole.append(first_slot)
    assert planned > 10 and (not flags or 64 in whole)       # (8192 + 16 answers, 40 / 8 heads: a full round stays whole, the last one is cut)


def test_a_plan_does_not_take_longer_for_more_q_heads_per_kv_head():
    def us(hq):
        best = 1.0
        for _ in range(15):
            t = time.perf_counter()
            B.sp_attn_pieces([40], [130], [600] * 130, hq, 1)
            best = min(best, time.perf_counter() - t)
        return best
    assert us(128) < 3 * us(8)                               # played in single steps, nine times


def test_arguments_are_checked():
    for bad in (([-1], [1], [5], 8, 8), ([5], [1], [5], 8, 3), ([5], [1], [5], 8, 8, 4)):
        with pytest.raises(B.SpAttnError):
            B.sp_attn_pieces(*bad)
