"""Lane-level CPU model of the LPT loops of the partition kernels for up to 64
bins, as they are now: narrow keys relative to the least load, rebased at
every batch; up to kLptStepBins bins item by item (kLptSteps a turn, the
lanes past the items raising nothing); above, rounds of equal weights and
prefix rounds from kLptRoundMin and kLptPrefixMin items, raised keys merged
where they are in order and sorted (32 lanes up to 32 bins) where not, the
items loaded anew after each round.  Every choice has to be sequential LPT's,
and every key has to fit 32 bits below the padding.  The constants are read
from the source."""
import os
import re

import numpy as np
import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2207_04350_amd", "csrc", "cg_device.h")
PAD = 0xFFFFFFFF


def _const(name):
    with open(SRC) as f:
        return int(re.search(r"constexpr int %s = (\d+);" % name, f.read()).group(1))


STEP_BINS, STEPS = _const("kLptStepBins"), _const("kLptSteps")
ROUND_MIN, PREFIX_MIN = _const("kLptRoundMin"), _const("kLptPrefixMin")


def _lpt(ws, P):
    load, out = [0] * P, []
    for w in ws:
        b = min(range(P), key=lambda b: (load[b], b))
        out.append(b)
        load[b] += w
    return out, load


def _bits(P):
    kb = 0
    while (1 << kb) < P:
        kb += 1
    return kb


def _network(x, lanes):
    """The bitonic sort of the first `lanes` of 64 lanes."""
    x = list(x)
    k = 2
    while k <= lanes:
        j = k // 2
        while j > 0:
            p = [x[l ^ j] for l in range(64)]
            x = [min(x[l], p[l]) if ((l & j) == 0) == ((l & k) == 0) else max(x[l], p[l])
                 for l in range(64)]
            j //= 2
        k *= 2
    return x


def _merge(x, c):
    """Two sorted runs, lanes 0..c-1 and c..63: the first turned round, then
    the last six stages of the bitonic sort."""
    x = [x[c - 1 - l] if l < c else x[l] for l in range(64)]
    for j in (32, 16, 8, 4, 2, 1):
        p = [x[l ^ j] for l in range(64)]
        x = [min(x[l], p[l]) if (l & j) == 0 else max(x[l], p[l]) for l in range(64)]
    return x


class _Loop:
    def __init__(self, ws, P):
        self.ws, self.P, self.kb = ws, P, _bits(P)
        self.mask = (1 << self.kb) - 1
        self.key = [l if l < P else PAD for l in range(64)]
        self.base_load, self.out, self.seen = 0, [None] * len(ws), set()

    def rebase(self):
        sub = self.key[0] & ~self.mask
        self.key = [k - sub if l < self.P else k for l, k in enumerate(self.key)]
        self.base_load += sub

    def raised(self, key, w):
        k = key + (w << self.kb)
        assert k < PAD, "a raised key reaches the padding"
        return k

    def step(self, at, w):
        k0 = self.key[0]
        nk = self.raised(k0, w) if w else k0
        nxt = self.key[1:] + [PAD]
        self.key = [min(nxt[l], max(nk, self.key[l])) for l in range(64)]
        if at is not None:
            self.out[at] = k0 & self.mask

    def few(self):
        for base in range(0, len(self.ws), 64):
            self.rebase()
            cnt = min(64, len(self.ws) - base)
            for t0 in range(0, cnt, STEPS):
                for t in range(t0, t0 + STEPS):
                    assert t < 64
                    self.step(base + t if t < cnt else None, self.ws[base + t] if t < cnt else 0)
        return self

    def rounds(self):
        ws, P, base, T = self.ws, self.P, 0, len(self.ws)
        while base < T:
            self.rebase()
            cnt, t = min(64, T - base), 0
            while t < cnt:
                w = ws[base + t]
                nk = self.raised(self.key[0], w)
                m = sum(k < nk for k in self.key)
                run = 1
                while t + run < cnt and ws[base + t + run] == w:
                    run += 1
                c, cp, r = min(run, m), 0, None
                if m >= PREFIX_MIN and c < m:
                    r = [self.raised(self.key[l], ws[base + t + l]) if l < cnt - t and l < P else PAD
                         for l in range(64)]
                    low = PAD
                    while cp < min(cnt - t, P) and self.key[cp] < low:
                        low = min(low, r[cp])
                        cp += 1
                if cp >= PREFIX_MIN:
                    for l in range(cp):
                        self.out[base + t + l] = self.key[l] & self.mask
                    down = any(r[l - 1] > r[l] for l in range(1, cp))
                    x = [r[l] if l < cp else self.key[l] for l in range(64)]
                    self.key = (_network(x, 32 if P <= 32 else 64)) if down else _merge(x, cp)
                    self.seen.add("sorted" if down else "merged")
                    t += cp
                    if base + cnt < T:
                        cnt = t
                elif c >= ROUND_MIN:
                    for l in range(c):
                        self.out[base + t + l] = self.key[l] & self.mask
                    self.key = _merge([self.raised(k, w) if l < c else k
                                       for l, k in enumerate(self.key)], c)
                    self.seen.add("equal")
                    t += c
                    if base + cnt < T:
                        cnt = t
                else:
                    self.seen.add("step")
                    self.step(base + t, w)
                    t += 1
                assert self.key == sorted(self.key)
            base += cnt
        return self

    def loads(self):
        out = [0] * self.P
        for k in self.key[:self.P]:
            out[k & self.mask] = (k + self.base_load) >> self.kb
        return out


def _weights(kind, n, rng):
    w = {"few values": lambda: rng.integers(1, 6, n),
         "many values": lambda: rng.integers(1, 2000, n),
         "powers": lambda: 2 ** rng.integers(0, 14, n),
         "heavy": lambda: np.concatenate([[300_000, 40_000][:min(n, 2)],
                                          rng.integers(1, 900, max(n - 2, 0))]),
         "equal": lambda: np.full(n, 7)}[kind]()
    return sorted((int(x) for x in w), reverse=True)


KINDS = ["few values", "many values", "powers", "heavy", "equal"]


@pytest.mark.parametrize("kind", KINDS)
def test_few_bins_item_by_item(kind):
    rng = np.random.default_rng(11)
    for P in (1, 2, 3, 5, 8, 15, 16):
        assert P <= STEP_BINS and 64 % STEPS == 0
        for n in (0, 1, STEPS - 1, STEPS, STEPS + 1, 63, 64, 65, 130, 300):
            ws = _weights(kind, n, rng)
            got = _Loop(ws, P).few()
            assert (got.out, got.loads()) == _lpt(ws, P), (P, n)


def test_rounds():
    rng = np.random.default_rng(12)
    seen = set()
    for kind in KINDS:
        for P in (17, 31, 32, 33, 63, 64):
            for n in (1, 5, 64, 65, 200, 700):
                ws = _weights(kind, n, rng)
                got = _Loop(ws, P).rounds()
                assert (got.out, got.loads()) == _lpt(ws, P), (kind, P, n)
                seen |= got.seen
    assert seen == {"step", "equal", "sorted", "merged"}
