"""The select that holds a row in registers (rows of up to 32768 scores, or up
to 131072 bf16 / 65536 fp32 ones when a launch has at most 256 rows), at the
sizes where it can go wrong: row lengths around one and all vectors per thread
and around what it takes at all, rows that start off a 16-byte boundary, m
close to the row length, thresholds on either side of zero, more equal scores
than its lists hold, samples that mislead it, infinities and NaNs.  Expected
sets come from a sort by order-preserving integer keys (NaNs by sign, as the
selects rank them), ties to the lower position."""
import zlib

import numpy as np
import pytest
import torch

import paper_2607_24593_amd as pv
from gpu_util import dev, host, say
from workload.gen import encode_bf16

pytestmark = pytest.mark.gpu


def _keys(rows):
    u = rows.view(np.uint32).astype(np.int64)
    mag = u & 0x7FFFFFFF
    return np.where(u >> 31, -mag, mag)  # -0 and +0 alike


def _check(rows, n0, step, m, bf16, ld_pad=0, off=0, label=""):
    """rows [R, n] float32; laid out with row stride n + ld_pad, `off` elements into a buffer."""
    R, n = rows.shape
    if bf16:
        bits = encode_bf16(rows)
        nan = np.isnan(rows)
        bits[nan] = (rows.view(np.uint32)[nan] >> 16).astype(np.uint16)
        rows = (bits.astype(np.uint32) << 16).view(np.float32)
    ld = n + ld_pad
    buf = np.zeros(off + R * ld, dtype=np.uint16 if bf16 else np.float32)
    buf[off:].reshape(R, ld)[:, :n] = bits if bf16 else rows
    t = dev(buf)[off:].view(R, ld)
    say("resident", label, R, n, n0, step, m, bf16, ld_pad, off)
    got = host(pv.pivot_topk_rows_bf16(t, n0, step, m) if bf16 else pv.pivot_topk_rows(t, n0, step, m))
    key = _keys(rows)
    for r in range(R) if n <= 200000 else (0, 1, 128, R - 1):
        k = n0 + r * step
        order = np.lexsort((np.arange(k), -key[r, :k]))[:m]
        exp = np.sort(np.concatenate([order, np.full(m - len(order), -1)]))
        assert np.array_equal(np.sort(got[r]), exp), (label, r, k)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n,m,R", [
    (9, 8, 2), (17, 3, 2), (2049, 2048, 3), (4096, 4095, 2), (4097, 4096, 2), (6001, 4096, 3), (7000, 4608, 2),
    (8191, 2048, 2), (8193, 2048, 2), (32767, 300, 2), (32769, 2049, 2), (65535, 4096, 2), (65536, 2048, 2),
    (65537, 2048, 2), (131071, 4608, 2), (131072, 2048, 2), (131073, 2048, 2),
    (2048, 2047, 260), (4101, 2048, 260), (8192, 4096, 260), (16384, 2048, 260), (16385, 4608, 260),
    (20011, 2048, 260), (32768, 4096, 260), (32769, 4096, 260),
    (8192, 4096, 2), (16384, 4096, 2), (16385, 4608, 2), (32768, 4096, 2), (65536, 4096, 256),  # edges of few rows
])
def test_lengths(n, m, R, bf16):
    rng = np.random.default_rng(n + m)
    _check(rng.standard_normal((R, n)).astype(np.float32), n, 0, m, bf16, label="lengths")


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("pad,off", [(1, 0), (3, 1), (0, 2), (5, 7)])
def test_rows_off_a_boundary(pad, off, bf16):
    rng = np.random.default_rng(pad * 8 + off)
    _check(rng.standard_normal((9, 5002)).astype(np.float32), 4994, 1, 1000, bf16, pad, off, "few")
    _check(rng.standard_normal((300, 9003)).astype(np.float32), 8703, 1, 2000, bf16, pad, off, "many")


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("R", [4, 270])
@pytest.mark.parametrize("kind", ["negative", "around_zero", "ties", "two_values", "constant", "tails", "sample_high",
                                  "sample_low", "inf", "nan", "lowest"])
def test_values(kind, R, bf16):
    rng = np.random.default_rng(zlib.crc32(kind.encode()))
    n, m = 24000, 4096
    x = rng.standard_normal((R, n)).astype(np.float32)
    if kind == "negative":
        x -= 20
    elif kind == "around_zero":  # the m-th key lies among the smallest magnitudes of both signs
        x -= np.quantile(x, 1 - m / n)
        x[:, ::7] *= 1e-30
    elif kind == "ties":
        x = np.round(x * 2) / 2
    elif kind == "two_values":
        x = rng.choice([-0.0, 0.0], size=(R, n)).astype(np.float32)
        x[:, 100:1100] = 1.0
    elif kind == "constant":
        x[:] = -3.5
    elif kind == "tails":
        x = np.sign(x) * np.exp(4 * np.abs(x))
    elif kind == "sample_high":  # the blocks that are sampled hold most of the high scores
        x[:, : 4096] += 6
    elif kind == "sample_low":
        x[:, -9000:] += 6
    elif kind == "inf":
        x[:, ::5] = np.inf
        x[:, 1::5] = -np.inf
    elif kind == "nan":
        x[:, 3::11] = np.nan
        x[:, 5::1001] = -np.nan
    elif kind == "lowest":  # masked scores: fewer than m above the type's lowest
        x[:, 3000:] = np.finfo(np.float32).min
    _check(x.astype(np.float32), n, 0, m, bf16, label=kind)


def test_one_sequence_past_the_limit():
    """Rows that grow past 32768 scores in one launch: both parts of it."""
    rng = np.random.default_rng(8)
    _check(rng.standard_normal((560, 33100)).astype(np.float32), 31600, 2, 2048, True, label="growing")
    _check(rng.standard_normal((560, 33100)).astype(np.float32), 31600, 2, 2048, False, label="growing")


@pytest.mark.parametrize("n,m", [(250001, 4096), (300000, 4500), (524288, 2048)])
def test_long_rows_take_a_larger_sample(n, m):
    """bf16 rows past those, streamed: lengths at which 4096 samples are too few."""
    rng = np.random.default_rng(n)
    x = rng.standard_normal((3, n)).astype(np.float32)
    _check(np.tile(x, (87, 1)), n - 260, 1, m, True, (-n) % 8, label="long")
