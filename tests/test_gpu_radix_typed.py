"""GPU parity of the signed and floating-point radix sorts (int32, float32,
float16 keys; ascending and descending), through the C ABI.

A stable sort has one correct output, so keys (as bit patterns) and the
permutation must equal the oracle's exactly -- including the IEEE 754
totalOrder placement of -0/+0, infinities, subnormals and NaNs of both signs
and several payloads.
"""
import numpy as np
import pytest

import oracle
from gpu_util import announce, assert_equal_first_diff, to_dev, to_host
from paper_2505_15112_amd import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 5, 255, 8191, 8192, 8193, 65_539, (1 << 20) + 17]


@pytest.fixture(scope="module")
def ops():
    from paper_2505_15112_amd import ops
    return ops


def _i32_sets(n, seed):
    rng = np.random.default_rng(seed)
    yield "uniform", rng.integers(-2**31, 2**31, n, dtype=np.int64).astype(np.int32)
    yield "ties", rng.integers(-3, 4, n).astype(np.int32)
    k = rng.integers(-2**31, 2**31, n, dtype=np.int64).astype(np.int32)
    k[::3] = -2**31
    k[1::5] = 2**31 - 1
    yield "extremes", k


SPECIAL_F32 = np.array([0x00000000, 0x80000000, 0x7F800000, 0xFF800000, 0x7FC00000, 0xFFC00000,
                        0x7F800001, 0xFF800001, 0x7FFFFFFF, 0xFFFFFFFF, 0x00000001, 0x80000001,
                        0x3F800000, 0xBF800000], np.uint32)
SPECIAL_F16 = np.array([0x0000, 0x8000, 0x7C00, 0xFC00, 0x7E00, 0xFE00, 0x7C01, 0xFC01, 0x7FFF,
                        0xFFFF, 0x0001, 0x8001, 0x3C00, 0xBC00], np.uint16)


def _float_sets(n, seed, dt):
    rng = np.random.default_rng(seed)
    bt, special = (np.uint32, SPECIAL_F32) if dt is np.float32 else (np.uint16, SPECIAL_F16)
    v = (rng.standard_normal(n) * 100).astype(dt)
    yield "normal", v
    t = v.copy()
    t[::2] = np.round(t[::2] / 50) * 50  # many ties, both zeros
    t[::7] = -t[::7] * 0
    yield "ties_zeros", t
    b = v.view(bt).copy()
    b[::3] = special[rng.integers(0, special.size, b[::3].size)]
    yield "specials", b.view(dt)
    if dt is np.float32:
        yield "bits", rng.integers(0, 2**32, n, dtype=np.uint64).astype(np.uint32).view(dt)
    else:
        yield "bits", rng.integers(0, 2**16, n).astype(np.uint16).view(dt)


def _check(ops, fn, ofn, keys, desc, with_perm, what, bt):
    import torch
    kd = torch.from_numpy(keys.copy()).cuda()
    ko, po = fn(kd, descending=desc, with_perm=with_perm)
    rk, rp = ofn(keys, descending=desc)
    assert_equal_first_diff(to_host(ko).view(bt), rk.view(bt), what + " keys")
    if with_perm:
        assert_equal_first_diff(to_host(po), rp, what + " perm")


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("desc", [False, True])
def test_sort_i32(ops, n, desc):
    for name, k in _i32_sets(n, n):
        announce("sort i32", n, desc, name)
        _check(ops, ops.radix_sort_i32, oracle.sort_i32, k, desc, True,
               f"i32 n={n} desc={desc} {name}", np.int32)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("desc", [False, True])
def test_sort_f32(ops, n, desc):
    for name, k in _float_sets(n, n + 1, np.float32):
        announce("sort f32", n, desc, name)
        _check(ops, ops.radix_sort_f32, oracle.sort_f32, k, desc, True,
               f"f32 n={n} desc={desc} {name}", np.uint32)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("desc", [False, True])
def test_sort_f16(ops, n, desc):
    for name, k in _float_sets(n, n + 2, np.float16):
        announce("sort f16", n, desc, name)
        _check(ops, ops.radix_sort_f16, oracle.sort_f16, k, desc, True,
               f"f16 n={n} desc={desc} {name}", np.uint16)


def test_keys_only_and_misaligned(ops):
    """No permutation, and key arrays one element off 16-byte alignment."""
    import torch
    announce("typed sorts keys only / misaligned")
    n = 3 * 8192 + 5
    k = np.random.default_rng(3).standard_normal(n + 1).astype(np.float32)
    kd = torch.from_numpy(k).cuda()[1:]
    ko, po = ops.radix_sort_f32(kd, descending=True, with_perm=False)
    assert po is None
    rk, _ = oracle.sort_f32(k[1:], descending=True)
    assert_equal_first_diff(to_host(ko).view(np.uint32), rk.view(np.uint32), "f32 keys only")
    h = W.scan_f16(n + 1, seed=4)
    hd = torch.from_numpy(h).cuda()[1:]
    ko, po = ops.radix_sort_f16(hd)
    rk, rp = oracle.sort_f16(h[1:])
    assert_equal_first_diff(to_host(ko).view(np.uint16), rk.view(np.uint16), "f16 misaligned")
    assert_equal_first_diff(to_host(po), rp, "f16 misaligned perm")


def test_sort_f32_desc_n2_24(ops):
    """The top-p sampler's sort: descending float32 probabilities at 2^24."""
    import torch
    announce("sort f32 desc n=2^24")
    n = 1 << 24
    probs = W.topp_probs(128, n // 128, seed=0).reshape(-1)
    rng = np.random.default_rng(5)
    probs = probs[rng.permutation(n)]  # unsorted
    ko, po = ops.radix_sort_f32(torch.from_numpy(probs).cuda(), descending=True)
    rk, rp = oracle.sort_f32(probs, descending=True)
    assert_equal_first_diff(to_host(po), rp, "f32 desc 2^24 perm")
    assert_equal_first_diff(to_host(ko).view(np.uint32), rk.view(np.uint32), "f32 desc 2^24 keys")


@pytest.mark.parametrize("n", [1, 2, 63, 255, 511, 512, 513, 2047, 2048, 2049, 4096, 4097, 8191,
                               8192, 8193, 16_383, 16_384, 16_385])
@pytest.mark.parametrize("desc", [False, True])
def test_one_workgroup_rows(ops, n, desc):
    """Rows of up to 16384 keys are sorted by one workgroup each: every size it
    comes in, and one more than the largest.  The places past a row's end hold the largest
    code, so many keys share it here (the largest integer ascending, the least
    descending, NaNs of both signs): ties with the padding keep index order."""
    import torch
    announce("one-workgroup rows", n, desc)
    rng = np.random.default_rng(n)
    edge = np.int32(-2**31) if desc else np.int32(2**31 - 1)
    k = np.where(rng.random(n) < 0.4, edge, rng.integers(-5, 5, n)).astype(np.int32)
    ko, po = ops.radix_sort_i32(to_dev(k), descending=desc)
    order = np.argsort(-k.astype(np.int64) if desc else k, kind="stable")
    assert_equal_first_diff(to_host(po), order.astype(np.int32), f"i32 perm {n}")
    assert_equal_first_diff(to_host(ko), k[order], f"i32 keys {n}")
    only, none = ops.radix_sort_i32(to_dev(k), descending=desc, with_perm=False)
    assert none is None
    assert_equal_first_diff(to_host(only), k[order], f"i32 keys only {n}")
    u = np.where(rng.random(n) < 0.5, 0xFFFFFFFF, rng.integers(0, 2**32, n)).astype(np.uint32)
    ko, po = ops.radix_sort_u32(to_dev(u.view(np.int32)))
    order = np.argsort(u, kind="stable")
    assert_equal_first_diff(to_host(po), order.astype(np.int32), f"u32 perm {n}")
    # rows of floats with NaNs, and half keys
    f = rng.integers(-3, 4, (3, n)).astype(np.float32)
    f[rng.random((3, n)) < 0.2] = np.nan
    f[rng.random((3, n)) < 0.2] = -np.float32(np.nan)
    ko, po = ops.radix_sort_rows_f32(to_dev(f), descending=desc)
    rk, rp = oracle.sort_rows_f32(f, descending=desc)
    assert_equal_first_diff(to_host(po), rp, f"row perm {n}")
    assert_equal_first_diff(to_host(ko).view(np.uint32), rk.view(np.uint32), f"row keys {n}")
    h = f[0].astype(np.float16)
    ko, po = ops.radix_sort_f16(to_dev(h), descending=desc)
    b = h.view(np.uint16).astype(np.int64)
    code = np.where(b >= 0x8000, 0xFFFF - b, b + 0x8000)
    order = np.argsort(-code if desc else code, kind="stable")
    assert_equal_first_diff(to_host(po), order.astype(np.int32), f"f16 perm {n}")
    assert torch.equal(ko.cpu().view(torch.int16), torch.from_numpy(h[order]).view(torch.int16))


@pytest.mark.parametrize("n", [16_385, 18_432, 65_537, 3 << 19, (3 << 19) + 1, (1 << 22) - 1,
                               1 << 22])
@pytest.mark.parametrize("least", [False, True])
def test_tile_choice(ops, n, least):
    """Sorts of more than 16384 keys take tiles of 2048, 4096 or 8192 keys by
    their size, and 8192 whatever the size in a workspace that has no room for
    the longer count table: both sides of each line, on one workspace."""
    import torch
    from paper_2505_15112_amd import _lib
    announce("tile choice", n, least)
    rng = np.random.default_rng(n)
    want = _lib.workspace_bytes(_lib.OP_RADIX_SORT, n, bits=8)
    if least:  # tiles of 8192 keys: 256 counts each, and the scan of that table
        entries = 256 * -(-n // 8192)
        want = (_lib.workspace_bytes(_lib.OP_SCAN, entries) + 15) // 16 * 16 + 4 * entries
    ws = torch.zeros((want + 7) // 8 * 8, dtype=torch.uint8, device="cuda")[:want]
    k = rng.integers(-2**31, 2**31, n, dtype=np.int64).astype(np.int32)
    ko, po = ops.radix_sort_i32(to_dev(k), ws=ws)
    order = np.argsort(k, kind="stable")
    assert_equal_first_diff(to_host(po), order.astype(np.int32), f"i32 perm {n}")
    assert_equal_first_diff(to_host(ko), k[order], f"i32 keys {n}")
    only, _ = ops.radix_sort_i32(to_dev(k), descending=True, with_perm=False, ws=ws)
    assert_equal_first_diff(to_host(only), k[order][::-1], f"i32 keys only {n}")
    h = rng.integers(-9, 10, n).astype(np.float16)  # many ties
    ko, po = ops.radix_sort_f16(to_dev(h), descending=True, ws=ws)
    b = h.view(np.uint16).astype(np.int64)
    order = np.argsort(-np.where(b >= 0x8000, 0xFFFF - b, b + 0x8000), kind="stable")
    assert_equal_first_diff(to_host(po), order.astype(np.int32), f"f16 perm {n}")
    assert torch.equal(ko.cpu().view(torch.int16), torch.from_numpy(h[order]).view(torch.int16))
    # rows that share the total, their ends inside a tile
    rows = 3 if n > 65_537 else 1
    f = rng.integers(-9, 10, (rows, n // rows)).astype(np.float32)
    ko, po = ops.radix_sort_rows_f32(to_dev(f), descending=True)
    rk, rp = oracle.sort_rows_f32(f, descending=True)
    assert_equal_first_diff(to_host(po), rp, f"row perm {n}")
    assert_equal_first_diff(to_host(ko).view(np.uint32), rk.view(np.uint32), f"row keys {n}")
