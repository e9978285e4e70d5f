"""GPU quantile estimator (App. G) vs the oracle's chunked estimate.

Each chunk's sort and quantile picks are exact on both sides; the
length-weighted average is a double sum that the oracle takes in chunk order
and the GPU in a tree, so the two may round differently.  Every entry must lie
within one fp32 ulp of the oracle's, plus the bound of the two double
summations (2 * nchunks * 2^-53 * max|x|, relative to the map's scale), which
matters only for entries near 0; the GPU map must be strictly increasing."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev, host, needs_gpu, say
from paper_2110_02861_amd import bq, workloads

pytestmark = [pytest.mark.gpu, needs_gpu]


def _inputs():
    rng = workloads.host_rng(0, "c2", 20, 0)
    return {
        "one": np.array([0.75], np.float32),
        "short": rng.standard_normal(100).astype(np.float32),
        "one_chunk": rng.standard_normal(4096).astype(np.float32),
        "chunk_plus_one": rng.standard_normal(4097).astype(np.float32),
        "ragged": workloads.student_t_host(3 * 4096 + 123, seed=3),
        "abs_t": np.abs(workloads.student_t_host(200_000, seed=4)),
        "ties": np.round(rng.standard_normal(50_000) * 3).astype(np.float32),
        "zeros": np.zeros(9000, np.float32),
        "constant": np.full(10_000, 3.0, np.float32),
        "negative": -np.abs(rng.standard_normal(30_000)).astype(np.float32) - 1.0,
        "wide_range": (np.sign(rng.standard_normal(40_000)) *
                       10.0 ** rng.uniform(-30, 30, 40_000)).astype(np.float32),
        "group_edge": rng.standard_normal(64 * 4096 + 1).astype(np.float32),
        "normal_1m": rng.standard_normal(1 << 20).astype(np.float32),
    }


def _nchunks(n, chunk=4096):
    return (n + chunk - 1) // chunk


def _map_scale(x, chunk=4096):
    """max |q_i| of Eq. 5 over the chunk-averaged quantiles (double), the
    divisor that normalizes the map."""
    S = np.zeros(257)
    for c0 in range(0, x.size, chunk):
        s = np.sort(x[c0:c0 + chunk].astype(np.float64))
        S += s.size * s[np.arange(257) * s.size // 257]
    Q = S / x.size
    return float(np.max(np.abs((Q[:-1] + Q[1:]) / 2)))


def _check_map(got, ref, x):
    assert np.all(np.diff(got) > 0)
    xmax = float(np.max(np.abs(x)))
    if xmax == 0.0:
        np.testing.assert_array_equal(got.view(np.uint32), ref.view(np.uint32))
        return
    tol = np.spacing(np.abs(ref)).astype(np.float64) + \
        2.0 * _nchunks(x.size) * 2.0 ** -53 * xmax / _map_scale(x)
    err = np.abs(got.astype(np.float64) - ref.astype(np.float64))
    assert np.all(err <= tol), (np.argmax(err / tol), float(np.max(err / tol)))


@pytest.mark.parametrize("name", list(_inputs()))
def test_estimate_matches_oracle(name):
    x = _inputs()[name]
    say(f"quantile estimate {name} n={x.size}")
    q = bq.bq_estimate_quantile_codebook(dev(x))
    torch.cuda.synchronize()
    _check_map(host(q), oracle.chunked_quantile_codebook(x), x)


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_estimate_of_a_view_4_byte_aligned(offset):
    """x = full[offset:] is only 4-byte aligned: full chunks take the scalar
    loads, with the same result."""
    full = workloads.student_t_host(3 * 4096 + 77, seed=6)
    x = full[offset:]
    say(f"quantile estimate of a view at offset {offset}")
    full_d = dev(full)
    q = bq.bq_estimate_quantile_codebook(full_d[offset:])
    torch.cuda.synchronize()
    _check_map(host(q), oracle.chunked_quantile_codebook(x), x)


def _bucket_inputs():
    """Values whose distribution decides how a chunk's ranks are found: buckets
    of one value in thousands (accepted), of 33 to 128 different values (sorted by
    a wave), many of these or larger ones (the chunk is sorted), of 9 to 32 values,
    a value that is a large part of the chunk (set aside), one sign, both zeros,
    the ends of the range; short chunks."""
    rng = workloads.host_rng(0, "c2", 21, 0)
    n = 3 * 4096 + 1001
    normal = rng.standard_normal(n).astype(np.float32)
    mostly_zero = normal.copy()
    mostly_zero[rng.random(n) < 0.7] = 0.0
    signed_zero = mostly_zero.copy()
    signed_zero[::3] *= np.float32(-1.0)
    cluster = np.float32(1.0) + np.float32(1e-4) * normal
    spread = cluster.copy()
    spread[:: 500] = np.float32(1e-6)
    clump = np.where(rng.random(n) < 0.01, rng.integers(1 << 23, 1 << 30, n),
                     (0x3f800000 + rng.integers(0, 24, n))).astype(np.uint32).view(np.float32)
    outliers = normal.copy()
    outliers[::1021] = np.float32(-3.4028235e38)
    scales = normal * (np.float32(1e-6) ** (np.arange(n) % 4)).astype(np.float32)
    columns = normal * (np.float32(1e-6) ** (np.arange(n) // 4 % 4)).astype(np.float32)
    def one_bucket(k):
        # one value a bucket, but for k different ones around a rank that is asked for;
        # in a chunk each of positive and of negative values
        bits = 0x3f800000 + 2028 * np.arange(4096)
        rank = 100 * 4096 // 257
        bits[rank - k // 2:rank - k // 2 + k] = \
            0x3f800000 + 2028 * rank // 1024 * 1024 + 1023 // k * np.arange(k)
        x = bits.astype(np.uint32).view(np.float32)
        return np.concatenate([rng.permutation(x), -rng.permutation(x)])
    def clusters(each, step, steps):
        # of `each` values, 2^c and up to `steps` steps of 2^(c - step) more
        c = np.arange(4096) // each - 4096 // each // 2
        part = rng.integers(0, steps, 4096)
        return rng.permutation(2.0 ** c * (1 + part * 2.0 ** -step)).astype(np.float32)
    return {
        "often_inside": np.where(rng.random(n) < 0.4, np.float32(-0.5), normal),
        "often_lowest": np.maximum(normal, np.float32(-0.1)),
        "often_largest": np.minimum(normal, np.float32(-0.1)),
        "often_and_three": np.where(np.arange(4096) % 1365 == 7, normal[:4096], np.float32(0.3)),
        "often_and_crowds": np.where(rng.random(n) < 0.4, np.float32(0.3), np.tanh(3 * normal)),
        "often_and_runs": np.where(rng.random(n) < 0.4, 0.0, 1 / (1 + np.exp(-3 * normal))),
        "often_minus_zero": np.where(rng.random(n) < 0.5, np.float32(-0.0), np.abs(normal)),
        "often_in_short": np.where(rng.random(1500) < 0.5, np.float32(2.0), normal[:1500]),
        "often_in_ordered": np.sort(np.maximum(normal, 0)),
        "some_runs": 1 / (1 + np.exp(-3 * normal)),
        "many_runs": clusters(40, 20, 80),
        "long_runs": clusters(400, 22, 800),
        "round_long_runs": clusters(400, 15, 40),
        "runs_both_signs": rng.permutation(np.concatenate([clusters(170, 20, 80),
                                                           -clusters(170, 20, 80)])),
        "outliers": outliers,
        "in_order": np.sort(normal),
        "in_order_down": np.sort(normal)[::-1].copy(),
        "scales_in_turn": scales,
        "scales_in_turn_by_4": columns,
        "mostly_zero": mostly_zero,
        "signed_zeros": signed_zero,
        "all_minus_zero": np.full(n, -0.0, np.float32),
        "one_zero": np.where(np.arange(n) % 4096 == 777, np.float32(0.0), normal),
        "one_minus_zero": np.where(np.arange(n) % 4096 == 3000, np.float32(-0.0), np.abs(normal)),
        "zero_among_tiny": np.where(np.arange(n) % 64 == 9, np.float32(0.0), 1e-38 * normal),
        "narrow": cluster,
        "narrow_negative": -cluster,
        "narrow_and_tiny": spread,
        "bf16_grid": (normal.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32),
        "clump": clump,
        "squares": normal * normal,
        "subnormal": (rng.integers(0, 5000, n).astype(np.uint32)).view(np.float32),
        "whole_range": np.concatenate([[np.float32(3.4028235e38), np.float32(-3.4028235e38)],
                                       normal, 1e-30 * normal]).astype(np.float32),
        "two_values": np.where(rng.random(n) < 0.5, 0.25, -3.0).astype(np.float32),
        **{f"one_bucket_of_{k}": one_bucket(k) for k in (2, 8, 9, 16, 17, 32, 33)},
        "4095": normal[:4095],
        "3073": normal[:3073],
        "2048": normal[:2048],
        "1025": normal[:1025],
        "1024": normal[:1024],
        "1023": normal[:1023],
        "257": normal[:257],
        "2": normal[:2],
    }


def _chunk_map(x, chunk=4096):
    """The map from exactly sorted chunks, averaged in double in the library's
    order: chunks within groups of 64, then the groups."""
    nch = _nchunks(x.size)
    groups = []
    for g in range(0, nch, 64):
        s = np.zeros(257)
        for c in range(g, min(nch, g + 64)):
            v = np.sort(x[c * chunk:(c + 1) * chunk])
            s = s + float(v.size) * v[np.arange(257) * v.size // 257].astype(np.float64)
        groups.append(s)
    Q = np.zeros(257)
    for s in groups:
        Q = Q + s
    Q = Q / x.size
    q = (Q[:-1] + Q[1:]) * 0.5
    top = np.max(np.abs(q))
    m = (q / top if top > 0 else q).astype(np.float32)
    for i in range(1, 256):
        if not m[i] > m[i - 1]:
            m[i] = np.nextafter(m[i - 1], np.float32(np.inf))
    return m


@pytest.mark.parametrize("name", list(_bucket_inputs()))
def test_rank_selection_for_any_distribution(name):
    """Every rank is exact, so the map equals that of sorted chunks bit for bit
    (the same sums in the same order)."""
    x = np.asarray(_bucket_inputs()[name], np.float32)
    say(f"quantile ranks {name} n={x.size}")
    q = bq.bq_estimate_quantile_codebook(dev(x))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(host(q), _chunk_map(x))


def test_estimate_feeds_the_quantizer():
    """The estimated map is a valid map for the block-wise kernels."""
    x = workloads.student_t_host(1 << 18, seed=5)
    x_d = dev(x)
    say("quantile estimate -> quantize")
    q_d = bq.bq_estimate_quantile_codebook(x_d)
    codes, absmax = bq.bq_quantize_blockwise(q_d, x_d, 2048)
    torch.cuda.synchronize()
    q = host(q_d)
    assert np.all(np.diff(q) > 0)
    c_ref, a_ref = oracle.quantize_blockwise(q, x, 2048)
    np.testing.assert_array_equal(host(codes), c_ref)
    np.testing.assert_array_equal(host(absmax), a_ref)


def _timed_inputs(n):
    """n values on the GPU by what is unlike normal values about their chunks,
    and n normal values."""
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    normal = torch.randn(n, device="cuda", generator=g)
    u = torch.rand(n, device="cuda", generator=g)
    return {
        "17 to 32 values in a rank's bucket": u,
        "an outlier in every chunk": torch.where(
            torch.arange(n, device="cuda") % 4096 == 5, 1e38, normal),
        "in order": normal.sort().values,
        "33 to 128 different values in some buckets": torch.sigmoid(3 * normal),
        "ties: one value": torch.full((n,), 0.1, device="cuda"),
        "ties: 99 % zeros": torch.where(u < 0.99, 0.0, normal),
        "ties: ReLU": normal.relu(),
    }, normal


def _estimate_us(x, rounds=9, calls=10):
    ws = torch.empty(bq.lib().bq_quantile_workspace_bytes(x.numel()) // 8, dtype=torch.float64,
                     device="cuda")
    out = torch.empty(256, device="cuda")
    us = []
    for _ in range(rounds):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(calls):
            bq.bq_estimate_quantile_codebook(x, out, ws)
        b.record()
        b.synchronize()
        us.append(a.elapsed_time(b) * 1e3 / calls)
    return sorted(us)[rounds // 2]


@pytest.mark.parametrize("n,most", [(300_007, 1.45), (1 << 24, 1.65)])
def test_estimate_time_hardly_depends_on_the_values(n, most):
    """None of these distributions may cost more than a full sort of every chunk
    would: 16 us of 300,007 values and 64 of 2^24, 1.2 and 1.7 times what normal
    values take (the inputs: 1.1 and up to 1.45 times; `most` leaves room for the
    clock).  Where the map is full of ties, one thread moves them apart for 20 us
    more."""
    inputs, normal = _timed_inputs(n)
    base = _estimate_us(normal)
    slow = {}
    for name, x in inputs.items():
        say(f"time of the quantile estimate: {name}")
        t = _estimate_us(x)
        limit = most * base + (22.0 if "ties" in name else 0.0)
        say(f"{t:.1f} us, normal values {base:.1f}, limit {limit:.1f}")
        if t > limit:
            slow[name] = (t, limit)
    assert not slow, slow
