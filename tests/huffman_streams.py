"""Streams of the Huffman stage made by hand, and which of its two forms the decoder gives a pass of a stream: a slice
of the payload in LDS, or a ring of words per thread."""
from __future__ import annotations

import os
import re

import numpy as np

CHUNK = 256
SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_11400_amd", "csrc", "fh_huffman.hip")


def decoder_shapes():
    """{threads: words of the payload slice in LDS} of the decoder's two workgroups, the narrow one first, and the chunks
    per compute unit up to which a call with exact counts is given the narrow one."""
    with open(SOURCE) as f:
        text = f.read()
    one = lambda pattern: [int(v) for v in re.search(pattern, text).groups()]
    (narrow,), (wide,), (words,) = (one(rf"constexpr int {name} = (\d+);") for name in ("kDecodeThreadsSmall", "kDecodeThreads", "kSmallWords"))
    a, b = one(r"kAll = THREADS >= 768 \? (\d+) \* (\d+) : THREADS \* kSmallWords")
    return {narrow: narrow * words, wide: a * b}, words * narrow // 64


def offsets_of(stream, n):
    chunks = -(-n // CHUNK)
    return stream[256: 256 + 4 * (chunks + 1)].view(np.uint32).astype(np.int64)


def passes(offsets, first, stop, threads, stage):
    """[(chunks, staged)] of the passes in which a workgroup takes the chunks first .. stop of a valid stream."""
    out = []
    while first < stop:
        want = min(stop - first, threads)
        fitting = int(np.searchsorted(offsets[first + 1: first + want + 1], offsets[first] + stage, side="right"))
        staged = fitting > 0 and 4 * fitting >= 3 * min(want, 768)
        out.append((fitting if staged else want, staged))
        first += out[-1][0]
    return out


def canonical_stream(data, lengths):
    """The stream of `data` under a canonical code of the given lengths (256 of them, Kraft's sum at most 1)."""
    lengths = np.asarray(lengths, dtype=np.int64)
    assert sum(2.0 ** -l for l in lengths if l) <= 1.0
    code, codes, last = 0, np.zeros(256, np.int64), 0
    for s in sorted((s for s in range(256) if lengths[s]), key=lambda s: (lengths[s], s)):
        code <<= int(lengths[s]) - last
        last = int(lengths[s])
        codes[s] = code
        code += 1
    n = data.size
    l, c = lengths[data], codes[data]
    assert (l > 0).all()
    chunk = np.arange(n) // CHUNK
    bits_of = np.bincount(chunk, weights=l).astype(np.int64)
    offsets = np.concatenate([[0], np.cumsum((bits_of + 31) // 32)])
    before = np.cumsum(l) - l
    at = 32 * offsets[chunk] + before - (before[::CHUNK])[chunk]
    bits = np.zeros(32 * int(offsets[-1]), np.uint8)
    for k in range(int(l.max())):
        m = l > k
        bits[at[m] + k] = (c[m] >> (l[m] - 1 - k)) & 1
    payload = np.packbits(bits).view(">u4").astype("<u4")
    return np.concatenate([lengths.astype(np.uint8), offsets.astype(np.uint32).view(np.uint8), payload.view(np.uint8)])


def long_codes(rng, n, noise):
    """(data, stream): a code with lengths 1 .. 15 once each and 24 for the other 241 values, data that draws from the short
    ones, and from the 241 in the chunks first .. stop of `noise`: 192 words each, the most a chunk can have."""
    lengths = np.concatenate([np.arange(1, 16), np.full(241, 24)])
    data = np.minimum(rng.geometric(0.5, n) - 1, 14)
    for first, stop in noise:
        part = data[first * CHUNK: stop * CHUNK]
        part[:] = rng.integers(15, 256, part.size)
    data = data.astype(np.uint8)
    return data, canonical_stream(data, lengths)
