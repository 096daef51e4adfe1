"""GPU parity of the batched row sort, weighted sampling and the top-p sampler
on unsorted rows (through the C ABI), against the oracle.

Row sort: keys bit-exact and in-row indices exact (a stable sort is unique),
special values included.  Samplers: the draw is the oracle's, or lies in the
rounding band around the threshold (the GPU sums in fp32, the oracle in
fp64); rows whose sums are exact in fp32 must match exactly; and, with the
draws theta on a fine grid, the draws reproduce the weights' distribution.
"""
import numpy as np
import pytest

import oracle
from gpu_util import (announce, assert_equal_first_diff, draw_accept, draw_tol, to_dev, to_host,
                      topp_accept)
from paper_2505_15112_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ops():
    from paper_2505_15112_amd import ops
    return ops


# (3, 200_003): more than 16 tiles per row, so the count table's row scan takes
# the multi-tile (look-back) schedule; (1, 2^20): the 1-D table scan.
SORT_SHAPES = [(1, 1), (3, 5), (1000, 100), (4, 8192), (3, 8193), (7, 10_001),
               (2, 3 * 8192 + 5), (16, 131_072), (3, 200_003), (1, 1 << 20)]


def _row_keys(rows, length, seed):
    k = W.values_f32(rows * length, seed=seed).reshape(rows, length)
    rng = np.random.default_rng(seed)
    specials = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 1.0, -1.0], np.float32)
    pick = rng.random((rows, length)) < 0.05
    k[pick] = specials[rng.integers(0, specials.size, int(pick.sum()))]
    neg_nan = rng.random((rows, length)) < 0.01
    k[neg_nan] = -np.float32(np.nan)
    return k


@pytest.mark.parametrize("shape", SORT_SHAPES, ids=lambda s: f"{s[0]}x{s[1]}")
@pytest.mark.parametrize("desc", [False, True])
def test_sort_rows_f32(ops, shape, desc):
    rows, length = shape
    announce("sort rows f32", shape, desc)
    k = _row_keys(rows, length, seed=rows + length)
    ko, po = ops.radix_sort_rows_f32(to_dev(k), descending=desc)
    rk, rp = oracle.sort_rows_f32(k, descending=desc)
    assert_equal_first_diff(to_host(ko).view(np.uint32), rk.view(np.uint32), f"keys {shape}")
    assert_equal_first_diff(to_host(po), rp, f"idx {shape}")


def test_sort_rows_keys_only_and_misaligned(ops):
    import torch
    announce("sort rows keys-only / misaligned")
    k = _row_keys(5, 9000, seed=3)
    ko, po = ops.radix_sort_rows_f32(to_dev(k), descending=True, with_perm=False)
    assert po is None
    assert_equal_first_diff(to_host(ko).view(np.uint32),
                            oracle.sort_rows_f32(k, True)[0].view(np.uint32), "keys only")
    flat = to_dev(_row_keys(1, 4 * 8200 + 1, seed=4).reshape(-1))
    view = flat[1:].reshape(4, 8200)  # 4-byte aligned, not 16-byte aligned
    assert view.data_ptr() % 16 != 0
    ko, po = ops.radix_sort_rows_f32(view)
    host = to_host(view)
    rk, rp = oracle.sort_rows_f32(host)
    assert_equal_first_diff(to_host(ko).view(np.uint32), rk.view(np.uint32), "misaligned keys")
    assert_equal_first_diff(to_host(po), rp, "misaligned idx")
    assert ops.radix_sort_rows_f32(torch.empty((0, 5), dtype=torch.float32,
                                               device="cuda"))[0].numel() == 0


# ---------------------------------------------------------------- weighted sampling

def _check_weighted(g, w, theta, what):
    csum, _ = oracle.scan_rows_f32(w)
    ref = oracle.weighted_sample_f32(w, theta)
    bad = []
    for r in range(w.shape[0]):
        if g[r] == ref[r]:
            continue
        total = float(csum[r, -1])
        u = float(theta[r]) * total
        if not draw_accept(int(g[r]), csum[r], u, draw_tol(float(theta[r]), total),
                           w.shape[1] - 1):
            bad.append(r)
    assert not bad, f"{what}: rows {bad[:5]} gpu {g[bad[:5]]} oracle {ref[bad[:5]]}"
    return ref


@pytest.mark.parametrize("length", [1, 3, 64, 4096, 4097, 10_003, 16_384, 16_385, 65_536, 65_537,
                                    131_072, (1 << 20) + 3, 1 << 22, (1 << 22) + 1])
def test_weighted_sample(ops, length):
    """Rows of 4097 to 2^22 take the two-kernel path (4096-element tiles up to
    16384, 8192 above), longer ones the single kernel with per-row arrival."""
    rows = 24 if length < (1 << 20) else 3
    announce("weighted sample", rows, length)
    w = W.sample_weights(rows, length, seed=length)
    theta = W.sample_theta(rows, seed=length)
    g = to_host(ops.weighted_sample_f32(to_dev(w), to_dev(theta)))
    _check_weighted(g, w, theta, f"weighted len={length}")


@pytest.mark.parametrize("length", [5, 4097, 131_072, (1 << 20) + 7])
def test_weighted_sample_exact(ops, length):
    """Integer weights 0..3 and theta in quarters: every fp32 sum and product
    is exact, so the draw must be the oracle's and never a zero weight."""
    rows = 16
    announce("weighted exact", length)
    rng = np.random.default_rng(length)
    w = rng.integers(0, 4, (rows, length)).astype(np.float32)
    w[:, 0] = 1.0
    theta = (rng.integers(0, 4, rows) / 4.0).astype(np.float32)
    g = to_host(ops.weighted_sample_f32(to_dev(w), to_dev(theta)))
    assert_equal_first_diff(g, oracle.weighted_sample_f32(w, theta), f"weighted exact {length}")
    assert all(w[r, g[r]] > 0 for r in range(rows))


def test_weighted_sample_distribution(ops):
    """One weight row repeated with theta on the grid (j + 1/2) / R: token i is
    drawn for a share w_i / W of the grid (inverse transform), so its count is
    R * w_i / W to within one grid step on each side."""
    announce("weighted distribution")
    R, length = 8192, 1000
    w1 = W.sample_weights(1, length, seed=99)
    w = np.repeat(w1, R, axis=0)
    theta = ((np.arange(R) + 0.5) / R).astype(np.float32)
    g = to_host(ops.weighted_sample_f32(to_dev(w), to_dev(theta)))
    counts = np.bincount(g, minlength=length)
    expect = R * w1[0].astype(np.float64) / w1[0].astype(np.float64).sum()
    assert np.all(np.abs(counts - expect) <= 2.0), np.max(np.abs(counts - expect))
    assert counts[w1[0] == 0].sum() == 0


def test_weighted_sample_edges(ops):
    import torch
    announce("weighted edges")
    e = ops.weighted_sample_f32(torch.empty((3, 0), dtype=torch.float32, device="cuda"),
                                to_dev(np.zeros(3, np.float32)))
    assert to_host(e).tolist() == [-1] * 3
    # theta = 0 draws the first non-zero weight; a single non-zero weight is always drawn
    w = np.zeros((4, 70_000), np.float32)
    w[0, 5] = 2.0
    w[1, 69_999] = 1.0
    w[2, 33_333] = 0.5
    w[3, :] = 1.0
    for th in (0.0, 0.5, 0.999):
        theta = np.full(4, th, np.float32)
        g = to_host(ops.weighted_sample_f32(to_dev(w), to_dev(theta)))
        assert g[:3].tolist() == [5, 69_999, 33_333], (th, g)
        assert g[3] == int(np.float64(np.float32(th)) * 70_000), (th, g)


# ---------------------------------------------------------------- top-p sampler

def _check_topp_sample(tok, cut, probs, theta, p, what):
    rows, length = probs.shape
    rt, rc = oracle.topp_sample_f32(probs, theta, p)
    sk, sp = oracle.sort_rows_f32(probs, descending=True)
    bad = []
    for r in range(rows):
        if tok[r] == rt[r] and cut[r] == rc[r]:
            continue
        csum = np.cumsum(sk[r].astype(np.float64))
        k = int(cut[r])
        if not topp_accept(k, int(rc[r]), csum, p):
            bad.append((r, "cutoff"))
            continue
        inv = np.empty(length, np.int64)
        inv[sp[r]] = np.arange(length)
        j = int(inv[tok[r]]) if 0 <= tok[r] < length else -1
        ck = float(csum[k])
        u = float(theta[r]) * ck
        if not draw_accept(j, csum, u, draw_tol(float(theta[r]), ck), k):
            bad.append((r, "token"))
    assert not bad, f"{what}: {bad[:5]} gpu {tok[:5]}/{cut[:5]} oracle {rt[:5]}/{rc[:5]}"
    return rt, rc


@pytest.mark.parametrize("length", [1, 3, 100, 4096, 4097, 10_003, 65_536, 65_537, 131_072,
                                    200_003, 1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("p", [0.0, 0.5, 0.9, 0.99, 1.5])
def test_topp_sample(ops, length, p):
    """Rows of 4097 to 2^20 draw on the early-exit kernels (the cutoff and the
    draw past the head quarter when p is large), others on the single kernel."""
    rows = 8
    announce("topp sample", rows, length, p)
    probs = W.sample_probs(rows, length, seed=length)
    theta = W.sample_theta(rows, seed=length + 1)
    tok, cut = ops.topp_sample_f32(to_dev(probs), to_dev(theta), p, with_cutoff=True)
    _check_topp_sample(to_host(tok), to_host(cut), probs, theta, p, f"topp sample {length} {p}")


@pytest.mark.parametrize("length", [7, 8192, 70_001, 131_072])
def test_topp_sample_exact(ops, length):
    """Probabilities that are multiples of 2^-24 below 16 * 2^-24, p a dyadic,
    theta in eighths: every fp32 sum and product is exact, ties are many
    (stable order decides), and the GPU must give the oracle's tokens."""
    rows = 16
    announce("topp sample exact", length)
    rng = np.random.default_rng(length)
    probs = (rng.integers(0, 16, (rows, length)) * 2.0**-24).astype(np.float32)
    theta = (rng.integers(0, 8, rows) / 8.0).astype(np.float32)
    total = probs.astype(np.float64).sum(axis=1)
    for frac in (0.25, 0.5, 0.875):
        p = float(np.float32(np.ldexp(np.round(np.ldexp(total.min() * frac, 24)), -24)))
        tok, cut = ops.topp_sample_f32(to_dev(probs), to_dev(theta), p, with_cutoff=True)
        rt, rc = oracle.topp_sample_f32(probs, theta, p)
        assert_equal_first_diff(to_host(cut), rc, f"exact cutoff {length} {frac}")
        assert_equal_first_diff(to_host(tok), rt, f"exact token {length} {frac}")


def test_topp_sample_distribution(ops):
    """One row repeated with theta on a grid: kept token i (in the sorted
    prefix 0..k) is drawn for a share S_i / C_k of the grid; tokens outside
    the nucleus are never drawn."""
    announce("topp distribution")
    R, length, p = 8192, 2000, 0.8
    row = W.sample_probs(1, length, seed=123)
    probs = np.repeat(row, R, axis=0)
    theta = ((np.arange(R) + 0.5) / R).astype(np.float32)
    tok, cut = ops.topp_sample_f32(to_dev(probs), to_dev(theta), p, with_cutoff=True)
    tok, cut = to_host(tok), to_host(cut)
    k = int(oracle.topp_sample_f32(row, theta[:1], p)[1][0])
    assert np.all(cut == cut[0]) and topp_accept(int(cut[0]), k,
                                                 np.cumsum(np.sort(row[0])[::-1]
                                                           .astype(np.float64)), p)
    sk, sp = oracle.sort_rows_f32(row, descending=True)
    kept = sp[0, :int(cut[0]) + 1]
    counts = np.bincount(tok, minlength=length)
    assert counts[np.setdiff1d(np.arange(length), kept)].sum() == 0
    pk = sk[0, :int(cut[0]) + 1].astype(np.float64)
    expect = R * pk / pk.sum()
    assert np.all(np.abs(counts[kept] - expect) <= 2.0), np.max(np.abs(counts[kept] - expect))


def test_topp_sample_edges(ops):
    import torch
    announce("topp sample edges")
    tok, cut = ops.topp_sample_f32(torch.empty((2, 0), dtype=torch.float32, device="cuda"),
                                   to_dev(np.zeros(2, np.float32)), 0.9, with_cutoff=True)
    assert to_host(tok).tolist() == [-1, -1] and to_host(cut).tolist() == [-1, -1]
    # p <= 0 keeps only the most probable token; a one-hot row always gives its token
    probs = W.sample_probs(4, 50_000, seed=8)
    probs[3] = 0.0
    probs[3, 12_345] = 1.0
    theta = np.array([0.0, 0.3, 0.99, 0.7], np.float32)
    tok = to_host(ops.topp_sample_f32(to_dev(probs), to_dev(theta), 0.0))
    assert tok[:3].tolist() == np.argmax(probs[:3], axis=1).tolist()
    assert tok[3] == 12_345


@pytest.mark.parametrize("seed", [0, 1])
def test_topp_sample_config_128x131072(ops, seed):
    announce("topp sample config", seed)
    probs = W.sample_probs(128, 131_072, seed=seed)
    theta = W.sample_theta(128, seed=seed)
    tok, cut = ops.topp_sample_f32(to_dev(probs), to_dev(theta), 0.9, with_cutoff=True)
    _check_topp_sample(to_host(tok), to_host(cut), probs, theta, 0.9, f"config seed={seed}")


def test_weighted_sample_config_128x131072(ops):
    announce("weighted config")
    w = W.sample_probs(128, 131_072, seed=5)
    theta = W.sample_theta(128, seed=5)
    g = to_host(ops.weighted_sample_f32(to_dev(w), to_dev(theta)))
    _check_weighted(g, w, theta, "weighted config")


# ---------------------------------------------------------------- the sampler's partial sort

PARTIAL_LENGTHS = [4097, 12_288, 12_289, 32_768, 40_961, 100_003, 131_072, 262_145, 1 << 20]


def _partial_rows(kind, rows, length, rng):
    """Small integers (every running sum exact in fp32 up to 2^21) whose order
    and density try the bins and groups of the partial sort."""
    if kind == "ties":  # a few values, many times each: bins larger than LDS
        x = rng.integers(0, 4, (rows, length))
    elif kind == "equal":
        x = np.ones((rows, length), np.int64)
    elif kind == "top":  # one element holds most of the mass, in no sample
        x = rng.integers(0, 2, (rows, length))
        x[np.arange(rows), rng.integers(0, length, rows)] = 1 << 20
    elif kind == "signed":
        x = rng.integers(-3, 4, (rows, length))
    else:  # special
        x = rng.integers(0, 4, (rows, length)).astype(np.float32)
        for r, v in enumerate([np.inf, np.nan, -np.inf, -np.nan, -0.0]):
            x[r % rows, rng.integers(0, length)] = v
    return np.ascontiguousarray(x, dtype=np.float32)


@pytest.mark.parametrize("length", PARTIAL_LENGTHS)
@pytest.mark.parametrize("kind", ["ties", "equal", "top", "signed", "special"])
def test_topp_sample_partial_sort_exact(ops, length, kind):
    """Rows of 4097 to 2^20 are sorted as far as the draw reads them; with
    exact sums cutoff and token must be the oracle's: p met early, late, at the
    last element and never."""
    rows = 6 if length < (1 << 18) else 2
    announce("topp partial sort", length, kind)
    rng = np.random.default_rng(length)
    x = _partial_rows(kind, rows, length, rng)
    theta = (rng.integers(0, 8, rows) / 8.0).astype(np.float32)
    total = float(np.nanmin(np.where(np.isfinite(x), x, 0).astype(np.float64).sum(axis=1)))
    for p in (1.0, np.floor(abs(total) / 2), abs(total), 2.0**22):
        rt, rc = oracle.topp_sample_f32(x, theta, p)
        tok, cut = ops.topp_sample_f32(to_dev(x), to_dev(theta), p, with_cutoff=True)
        assert_equal_first_diff(to_host(cut), rc, f"cutoff {length} {kind} {p}")
        assert_equal_first_diff(to_host(tok), rt, f"token {length} {kind} {p}")


@pytest.mark.parametrize("length", PARTIAL_LENGTHS)
@pytest.mark.parametrize("rows", [1, 9, 300])
def test_topp_sample_cutoff_as_sorted_rows(ops, length, rows):
    """On any data the cutoff is the one that the same additions find on the
    whole sorted rows (row sort, then the top-p cutoff), and the token the draw's
    there within rounding: flat, peaked, bf16 and
    masked probabilities, small and large batches (both tile and group sizes)."""
    if rows * length > 1 << 24:
        pytest.skip("the largest batches add nothing")
    import torch
    announce("topp cutoff as on sorted rows", rows, length)
    g = torch.Generator(device="cuda")
    g.manual_seed(length + rows)
    z = torch.randn((rows, length), device="cuda", generator=g)
    theta = torch.rand(rows, device="cuda", generator=g)
    for x in (torch.softmax(2 * z, 1), torch.softmax(1e-4 * z, 1), torch.softmax(8 * z, 1),
              torch.softmax((2 * z).bfloat16().float(), 1), torch.softmax(z, 1) * (z > 1.5)):
        for p in (0.1, 0.9, 0.999, 1.0):
            _check_as_sorted(ops, x.contiguous(), theta, p, f"{rows} x {length}")


def _check_as_sorted(ops, x, theta, p, what):
    """Cutoff and token of the sampler against the rows sorted whole: the same
    cutoff as the top-p cutoff finds there, and a token whose place in the sorted
    row is the draw's, or in the rounding band around its threshold."""
    import torch
    srt, perm = ops.radix_sort_rows_f32(x, descending=True)
    tok, cut = ops.topp_sample_f32(x, theta, p, with_cutoff=True)
    want = ops.topp_cutoff_f32(srt, p)
    assert torch.equal(cut, want), (what, p, cut[:4], want[:4])
    pos = to_host((perm == tok[:, None]).int().argmax(dim=1))
    assert torch.equal(perm.gather(1, to_dev(pos).long()[:, None]).squeeze(1), tok), (what, p)
    csum = to_host(torch.cumsum(srt.double(), dim=1))
    th = to_host(theta).astype(np.float64)
    for r, k in enumerate(to_host(cut)):
        total = float(csum[r, k])
        assert draw_accept(int(pos[r]), csum[r], th[r] * total, draw_tol(th[r], total), int(k)), \
            (what, p, r, int(pos[r]), int(k))


def _crowded_rows(kind, rows, length, seed):
    """Probabilities far from evenly spread over their range: flat rows (keys a
    few hundred or thousand apart) with one large element or a share of zeros,
    rows mostly zero, rows of one value, few values, values at three scales, and
    rows whose values the sampler's sample misses (4 elements in each of 512
    places, zeros here), a fifth of them equal."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    z = torch.randn((rows, length), device="cuda", generator=g)
    u = torch.rand((rows, length), device="cuda", generator=g)
    if kind.startswith("spike"):
        x = torch.softmax(float(kind[5:]) * z, 1) * 0.95
        return x.scatter_(1, torch.randint(0, length, (rows, 1), device="cuda", generator=g), 0.05)
    if kind.startswith("mask"):
        return torch.softmax((float(kind[4:]) * z).masked_fill(u < 0.1, float("-inf")), 1)
    if kind == "rare":
        return torch.softmax((2 * z).masked_fill(u < 0.99, float("-inf")), 1)
    if kind == "equal":
        return torch.full_like(z, 1.0 / length)
    if kind == "flat":
        return torch.softmax(1e-3 * z, 1)
    if kind == "soft":
        return torch.softmax(2 * z, 1)
    if kind == "bf16":
        return torch.softmax(2 * z, 1).bfloat16().float()
    if kind == "hidden":
        x = torch.softmax(2 * z, 1).masked_fill(u < 0.2, 1.0 / length)
        at = torch.arange(512, device="cuda") * (length - 4) // 511
        x[:, (at[:, None] + torch.arange(4, device="cuda")).flatten()] = 0.0
        return x
    x = torch.softmax(1e-6 * z, 1) * 0.5  # scales
    x = torch.where(u < 0.3, x * 1e-20, x)
    return torch.where(u > 0.9, torch.softmax(z, 1), x).contiguous()


@pytest.mark.parametrize("length", [4097, 8192, 12_288, 12_289, 131_072])
@pytest.mark.parametrize("kind", ["spike.1", "spike.001", "spike.000001", "mask.1", "mask.001",
                                  "mask.00001", "mask.000001", "rare", "equal", "scales",
                                  "hidden"])
def test_topp_sample_crowded(ops, length, kind):
    """Rows whose keys crowd in a small part of their range, on both sides of the
    row length up to which one workgroup sorts a row whole."""
    import torch
    announce("topp crowded", length, kind)
    rows = 9
    x = _crowded_rows(kind, rows, length, seed=length)
    theta = torch.rand(rows, device="cuda", generator=torch.Generator("cuda").manual_seed(length))
    for p in (0.3, 0.9, 1.0, 2.0):
        _check_as_sorted(ops, x, theta, p, f"{kind} {length}")


@pytest.mark.parametrize("length", [4097, 12_288])
def test_topp_sample_crowded_exact(ops, length):
    """Sixteen values 2^-10 apart and zeros, every sum exact: cutoff and token are
    the oracle's.  The values share two slots of the sort in LDS with thousands
    of keys each, so the row goes by digit passes."""
    announce("topp crowded exact", length)
    rows = 6
    rng = np.random.default_rng(length)
    x = (1.0 + rng.integers(0, 16, (rows, length)) * 2.0**-10).astype(np.float32)
    x[rng.random((rows, length)) < 0.1] = 0.0
    theta = (rng.integers(0, 8, rows) / 8.0).astype(np.float32)
    for p in (1.0, np.floor(0.5 * length), 0.8 * length, 2.0**22):
        p = float(np.float32(p))
        rt, rc = oracle.topp_sample_f32(x, theta, p)
        tok, cut = ops.topp_sample_f32(to_dev(x), to_dev(theta), p, with_cutoff=True)
        assert_equal_first_diff(to_host(cut), rc, f"cutoff {length} {p}")
        # theta in eighths of a sum with up to 14 + 10 bits: the product is rounded
        same = to_host(tok) == rt
        csum = np.cumsum(-np.sort(-x.astype(np.float64), axis=1), axis=1)
        for r in np.flatnonzero(~same):
            order = np.argsort(-x[r].astype(np.float64), kind="stable")
            total = csum[r, rc[r]]
            pos = int(np.flatnonzero(order == to_host(tok)[r])[0])
            assert draw_accept(pos, csum[r], theta[r] * total, 2.0**-23 * theta[r] * total,
                               int(rc[r])), (length, p, r)


def _best_us(f, batches=8, calls=3):
    import torch
    for _ in range(4):
        f()
    best = float("inf")
    for _ in range(batches):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        torch.cuda.synchronize()
        a.record()
        for _ in range(calls):
            f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1000 / calls)
    return best


@pytest.mark.parametrize("rows,length", [(3, 40_000), (3, 262_145), (3, 1 << 20), (70, 262_145)])
@pytest.mark.parametrize("kind", ["soft", "flat", "bf16", "scales", "hidden", "mask.00001"])
def test_topp_sample_many_groups(ops, rows, length, kind):
    """Long rows sorted to their end: many groups a row (of 4096 elements, and from
    2^23 elements on of 11264), each with its own part of the row's list, and the
    token looked up in the draw's group; groups too large for LDS, of few values
    and of many."""
    import torch
    announce("topp many groups", length, kind, rows)
    x = _crowded_rows(kind, rows, length, seed=length)
    theta = torch.tensor([0.0, 0.5, 0.999], device="cuda").repeat(rows)[:rows].contiguous()
    for p in (0.5, 0.99, 2.0):
        _check_as_sorted(ops, x, theta, p, f"{kind} {length}")


@pytest.mark.parametrize("length", [4097, 12_289, 131_072, 1 << 20])
def test_topp_sample_scratch_contents(ops, length):
    """What the scratch holds before the call (the sorted row is written as far as
    the crossing only) changes nothing: infinities, NaN, large values of both signs."""
    import torch
    from paper_2505_15112_amd import _lib
    announce("topp scratch contents", length)
    rows = 3
    x = torch.cat([_crowded_rows(k, 1, length, seed=3) for k in ("soft", "rare", "flat")])
    theta = torch.tensor([0.999, 0.5, 0.999], device="cuda")
    scr = ops.scratch(_lib.OP_TOPP_SAMPLE, x.device, rows, length)
    for p in (0.05, 0.9):
        got = []
        for bits in (0, 0x7F800000, 0x7FC00000, 0x7F7FFFFF, 0x7F7FFFFF - 2**31, -1):
            scr.view(torch.int32).fill_(bits)
            got.append(ops.topp_sample_f32(x, theta, p, with_cutoff=True, scratch_buf=scr))
        for tok, cut in got[1:]:
            assert torch.equal(tok, got[0][0]) and torch.equal(cut, got[0][1]), (length, p)
        _check_as_sorted(ops, x, theta, p, f"scratch {length}")


TIMED = [((1, 1 << 20), k) for k in ("soft", "flat", "equal", "mask.00001", "mask.000001")] + \
        [((4, 200_003), k) for k in ("soft", "flat", "bf16", "rare", "scales", "mask.00001")] + \
        [((128, 131_072), k) for k in ("flat", "rare", "equal", "scales", "mask.000001")] + \
        [((128, 8192), k) for k in ("spike.001", "mask.1", "mask.001", "mask.000001")] + \
        [((64, 12_288), k) for k in ("spike.001", "mask.1", "mask.001", "mask.000001", "equal")]


@pytest.mark.parametrize("shape,kind", TIMED, ids=lambda v: v if isinstance(v, str)
                         else f"{v[0]}x{v[1]}")
def test_topp_sample_time_bounded(ops, shape, kind):
    """The partial sort never costs much more than the sort of whole rows that
    it stands in for, whatever the values: the sampler takes at most twice (rows of
    2^20, whose crowds one workgroup counts: 3 times) the row sort and two
    cutoffs on its result (its own cutoff and the draw), or 3 times its own time
    on softmax rows of the same shape if that is longer
    (unbounded group sorts took 10 to 50 times as long)."""
    import torch
    from paper_2505_15112_amd import _lib
    rows, length = shape
    announce("topp time", shape, kind)
    x = _crowded_rows(kind, rows, length, seed=5)
    z = torch.softmax(2 * torch.randn(x.shape, device="cuda"), 1)
    theta = torch.rand(rows, device="cuda")
    ws = ops.workspace(_lib.OP_TOPP_SAMPLE, x.device, rows=rows, length=length)
    scr = ops.scratch(_lib.OP_TOPP_SAMPLE, x.device, rows, length)
    wss = ops.workspace(_lib.OP_SORT_ROWS, x.device, rows=rows, length=length)
    wsc = ops.workspace(_lib.OP_SCAN_ROWS, x.device, rows=rows, length=length)
    for p in (0.9, 1.0):
        def sample(v):
            return ops.topp_sample_f32(v, theta, p, with_cutoff=True, ws=ws, scratch_buf=scr)
        srt = ops.radix_sort_rows_f32(x, descending=True)[0]
        whole = _best_us(lambda: ops.radix_sort_rows_f32(x, descending=True, ws=wss)) + \
            2 * _best_us(lambda: ops.topp_cutoff_f32(srt, p, ws=wsc))
        t, usual = _best_us(lambda: sample(x)), _best_us(lambda: sample(z))
        print(f"[time] {shape} {kind} p={p}: {t:.1f} us, row sort and cutoffs {whole:.1f}, "
              f"softmax rows {usual:.1f}", flush=True)
        assert t <= max((3 if length == 1 << 20 else 2) * whole, 3 * usual), (shape, kind, p, t, whole, usual)
