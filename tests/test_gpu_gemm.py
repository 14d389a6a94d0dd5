"""Prefill GEMM (bf16 MFMA, fp32 accumulation) on the GPU against the fp64 oracle."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2607_14618_amd as pq
from synth import make_layer, random_quant_linear, MIX_PREFILL_4
from gpu_util import dev, np_, packed_linear, oracle_ref, assert_parity

pytestmark = pytest.mark.gpu

SHAPES = [
    (64, [(2, 128)]),
    (1, [(3, 32)]),
    (100, [(2, 160), (3, 96), (4, 128), (8, 96), (16, 32)]),
    (130, [(2, 992), (3, 704), (4, 256), (8, 64), (16, 32)]),
    (37, [(2, 32), (3, 32), (4, 32), (8, 32), (16, 32)]),
    (257, [(4, 480), (16, 96)]),
    (64, [(16, 256)]),
]


def _xb(m, k, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((m, k), generator=g)
    idx = torch.randperm(k, generator=g)[: max(1, k // 100)]
    x[:, idx] *= 50
    return x.bfloat16()


@pytest.mark.parametrize("n,blocks", SHAPES)
@pytest.mark.parametrize("m", [1, 7, 128, 300])
def test_gemm_parity_small(n, blocks, m):
    k = sum(l for _, l in blocks)
    lin = random_quant_linear(n, k, blocks, seed=2000 + n + k + m, mode="codes")
    pl = packed_linear(lin)
    x = _xb(m, k, seed=n + m)
    y = pl.prefill(x.to(dev()))
    torch.cuda.synchronize()
    y_ref, bound = oracle_ref(lin, x)
    assert_parity(y, y_ref, bound, f"gemm n={n} blocks={blocks} m={m}")
    xp = pl.permute(x.to(dev()))
    y2 = pl.prefill(xp, pre_permuted=True)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)


def test_gemm_one_hot_rows_are_exact():
    """(q - z) is exact in bf16, s is applied once in fp32, 16-bit weights enter as
    hi + lo: a one-hot activation row selects one dequantized weight exactly."""
    import oracle
    blocks = [(2, 160), (3, 96), (4, 128), (8, 96), (16, 32)]
    lin = random_quant_linear(100, 512, blocks, seed=9, mode="codes")
    pl = packed_linear(lin)
    cols = [0, 3, 200, 511]
    x = torch.zeros((len(cols), 512), dtype=torch.bfloat16)
    for i, j in enumerate(cols):
        x[i, j] = 1.0
    y = pl.prefill(x.to(dev()))
    torch.cuda.synchronize()
    w_hat = oracle.dequantize(lin.blocks, np_(lin.codes).view(np.uint16), np_(lin.scales),
                              np_(lin.zeros))
    inv = np.argsort(lin.perm)
    for i, j in enumerate(cols):
        assert np.array_equal(np_(y)[i].astype(np.float64), w_hat[:, inv[j]]), j


def test_gemm_rows_match_gemv():
    """Each GEMM row equals the GEMV of that token within the tolerance (the
    activations are bf16 values, exactly representable in fp16 here)."""
    blocks = [(2, 992), (3, 704), (4, 256), (8, 64), (16, 32)]
    lin = random_quant_linear(200, 2048, blocks, seed=4, mode="gauss")
    pl = packed_linear(lin)
    x = (torch.randn((5, 2048), generator=torch.Generator().manual_seed(3)) * 4).bfloat16()
    assert torch.equal(x.half().bfloat16(), x)
    yg = pl.prefill(x.to(dev()))
    yv = pl.decode(x.half().to(dev()))
    torch.cuda.synchronize()
    y_ref, bound = oracle_ref(lin, x)
    assert_parity(yg, y_ref, bound, "gemm")
    assert_parity(yv, y_ref, bound, "gemv")
    assert np.all(np.abs(np_(yg) - np_(yv)) <= 2e-3 * bound)


def test_gemm_config3_llama2_13b_prefill():
    """Llama2-13B layer at M=512, 4.0-bit mix: 512 seeded rows of each linear."""
    lins, groups = make_layer(3, m=512, x_dtype=torch.bfloat16, device=dev())
    rng = np.random.default_rng(3)
    for lin in lins:
        x = groups[lin.group].x
        pl = packed_linear(lin)
        assert pl.layout.code_bits == 4 * lin.n * lin.k
        y = pl.prefill(x.to(dev()))
        torch.cuda.synchronize()
        rows = np.sort(rng.choice(lin.n, 512, replace=False))
        y_ref, bound = oracle_ref(lin, x, rows=rows)
        assert_parity(np_(y)[:, rows], y_ref, bound, f"config 3 {lin.name}")


def test_gemm_batch_matches_single_calls():
    """q/k/v-like batch (shared x and permutation) and the single-linear calls
    (which may split K and add the splits in order) both meet the oracle bound."""
    blocks = [(2, 992), (3, 704), (4, 256), (8, 64), (16, 32)]
    lins = [random_quant_linear(n, 2048, blocks, seed=70 + i, mode="gauss") for i, n in enumerate((320, 192, 64))]
    perm = lins[0].perm
    for lin in lins[1:]:
        lin.perm = perm  # one input group: same channel permutation
    pls = [packed_linear(lin) for lin in lins]
    x = _xb(300, 2048, seed=5)
    xd = x.to(dev())
    ys = pq.prefill_batch(pls, [xd] * 3)
    singles = [pl.prefill(xd) for pl in pls]
    torch.cuda.synchronize()
    for lin, y, y1 in zip(lins, ys, singles):
        y_ref, bound = oracle_ref(lin, x)
        assert_parity(y, y_ref, bound, f"gemm batch n={lin.n}")
        assert_parity(y1, y_ref, bound, f"gemm single n={lin.n}")


@pytest.mark.parametrize("m", [1, 77, 513])
def test_gemm_batch_mixed_items(m):
    """Items of different shapes and bit mixes, with and without a permutation."""
    specs = [(100, [(2, 160), (3, 96), (4, 128), (8, 96), (16, 32)]), (257, [(4, 480), (16, 96)]),
             (64, [(3, 32)]), (130, [(2, 992), (3, 704), (4, 256), (8, 64), (16, 32)])]
    lins, xs = [], []
    for i, (n, blocks) in enumerate(specs):
        k = sum(l for _, l in blocks)
        lin = random_quant_linear(n, k, blocks, seed=300 + i, mode="codes")
        lins.append(lin)
        xs.append(_xb(m, k, seed=40 + i))
    pls = [packed_linear(lin) for lin in lins]
    xd = [x.to(dev()) for x in xs]
    items = []
    for i, (pl, x) in enumerate(zip(pls, xd)):
        if i % 2:
            items.append((pl.layout, pl.packed, None, pl.permute(x), None))
        else:
            items.append((pl.layout, pl.packed, pl.perm, x, None))
    ys = pq.gemm_batch(items)
    torch.cuda.synchronize()
    for lin, x, y in zip(lins, xs, ys):
        y_ref, bound = oracle_ref(lin, x)
        assert_parity(y, y_ref, bound, f"gemm batch mixed n={lin.n} m={m}")


def test_gemm_batch_rejects_bad_requests():
    lin = random_quant_linear(64, 128, [(4, 128)], seed=1, mode="codes")
    pl = packed_linear(lin)
    x = _xb(4, 128, seed=1).to(dev())
    with pytest.raises(ValueError):
        pq.gemm_batch([])
    with pytest.raises(ValueError):
        pq.gemm_batch([(pl.layout, pl.packed, pl.perm, x, None)] * (pq._lib.MAX_BATCH + 1))
    with pytest.raises(ValueError):
        pq.gemm_batch([(pl.layout, pl.packed, pl.perm, x, None), (pl.layout, pl.packed, pl.perm, x[:3], None)])


def test_gemm_wide_path_rescale():
    """A launch of more than one round of work-groups: mixed blocks, a 16-bit
    block, rows whose scale is zero, a non-integer zero point, ragged M."""
    blocks = [(2, 160), (3, 96), (4, 128), (8, 96), (16, 32)]
    lins = []
    for i in range(2):
        lin = random_quant_linear(25600, 512, blocks, seed=900 + i, mode="codes")
        sc = lin.scales.clone()
        sc[7, :] = 0           # row 7: every group scale zero
        sc[4097, 1] = 0        # one group of one row
        lin.scales = sc
        if i == 1:
            zz = lin.zeros.clone()
            zz[100, 0] = 3.5   # a non-integer zero point (its group's second pass)
            lin.zeros = zz
        lins.append(lin)
    pls = [packed_linear(lin) for lin in lins]
    x = _xb(200, 512, seed=17)
    ys = pq.prefill_batch(pls, [x.to(dev())] * 2)
    torch.cuda.synchronize()
    for lin, y in zip(lins, ys):
        y_ref, bound = oracle_ref(lin, x)
        assert_parity(y, y_ref, bound, f"gemm wide n={lin.n}")


def test_gemm_and_gemv_beyond_the_lds_row_gather():
    """K = 40960 > 32768: the prefill row gather takes its global-memory form; the
    decode GEMV plans many splits of one tile."""
    blocks = [(2, 20480), (3, 12288), (4, 6144), (8, 1024), (16, 1024)]
    k = sum(l for _, l in blocks)
    lin = random_quant_linear(96, k, blocks, seed=77, mode="codes")
    pl = packed_linear(lin)
    xb = _xb(5, k, seed=3)
    y = pl.prefill(xb.to(dev()))
    xh = (torch.randn((3, k), generator=torch.Generator().manual_seed(4))).half()
    yv = pl.decode(xh.to(dev()))
    torch.cuda.synchronize()
    y_ref, bound = oracle_ref(lin, xb)
    assert_parity(y, y_ref, bound, "gemm k=40960")
    yv_ref, bv = oracle_ref(lin, xh)
    assert_parity(yv, yv_ref, bv, "gemv k=40960")


SMALL_Z = [0.001, 0.03, -0.001, 2.0 ** -24, 0.0999]


def _small_z_linear(n, k, blocks, seed):
    """Codes-mode layer where rows 0..9 have all low-bit codes 0 and every zero
    point of rows 0..19 is a small non-integer (fp16 of SMALL_Z, cycled): with
    q = 0 the product is s * (0 - z) * x, so any rounding of z shows in full."""
    lin = random_quant_linear(n, k, blocks, seed=seed, mode="codes")
    codes = lin.codes.clone()
    zeros = lin.zeros.clone()
    k0 = 0
    for b, ln in blocks:
        if b != 16:
            codes[:10, k0:k0 + ln] = 0
        k0 += ln
    for r in range(min(20, n)):
        for g in range(zeros.shape[1]):
            zeros[r, g] = SMALL_Z[(r + g) % len(SMALL_Z)]
    lin.codes, lin.zeros = codes, zeros
    return lin


@pytest.mark.parametrize("case", ["split_k", "one_tile", "eight_wave", "wide"])
def test_gemm_small_non_integer_zero_points(case):
    """Zero points below 2^-3 that are not integers meet the bound on rows whose
    codes are all 0 (their sums are of the second pass alone) and on random-code
    rows: one linear with K split, and batches of one row block per linear, of
    half a round of work-groups (64 row blocks each) and of nearly one (100 each).
    Seven tokens: one token tile (others: test_gemm_every_form)."""
    mixed = [(2, 992), (3, 704), (4, 256), (8, 64), (16, 32)]
    small = [(2, 160), (3, 96), (4, 128), (8, 96), (16, 32)]
    if case == "split_k":
        specs = [(100, mixed)]            # one linear, 2 tiles, 18 groups: K split
    elif case == "one_tile":
        specs = [(100, small), (70, small)]
    elif case == "eight_wave":
        specs = [(16384, small), (16384, small)]
    else:
        specs = [(25600, small), (25600, small)]
    lins = [_small_z_linear(n, sum(l for _, l in bl), bl, seed=4100 + i) for i, (n, bl) in enumerate(specs)]
    k = lins[0].k
    for lin in lins[1:]:
        lin.perm = lins[0].perm
    pls = [packed_linear(lin) for lin in lins]
    x = _xb(7, k, seed=41)
    xd = x.to(dev())
    ys = [pls[0].prefill(xd)] if len(pls) == 1 else pq.prefill_batch(pls, [xd] * len(pls))
    torch.cuda.synchronize()
    for lin, y in zip(lins, ys):
        y_ref, bound = oracle_ref(lin, x)
        assert_parity(y, y_ref, bound, f"gemm small z {case} n={lin.n}")
        # the all-zero-code rows alone (their products are -s z x only)
        assert_parity(np_(y)[:, :10], y_ref[:, :10], bound[:, :10], f"gemm small z rows {case}")


def _fractional(lin, seed):
    """Every zero point off the integers in [0, 255]: fractions, negatives, and a
    few past 255."""
    g = torch.Generator().manual_seed(seed)
    z = torch.rand(lin.zeros.shape, generator=g) * 20 - 4
    z[:, ::3] = torch.rand(z[:, ::3].shape, generator=g) * 0.5 - 0.25
    z[::7, 1] = 300.5
    lin.zeros = z.half()
    return lin


@pytest.mark.parametrize("m", [9, 33, 130])
def test_gemm_fractional_zero_points_every_group(m):
    """All groups of all bit-widths with zero points that are not integers in
    [0, 255]: the group's two parts, (q - zi) and (zi - z), have together at most
    three times the weight of q - z, so three times the rounding of any summation
    order bounds the error."""
    k = sum(ln for _, ln in STEADY)
    lin = _fractional(random_quant_linear(130, k, STEADY, seed=5300 + m, mode="codes"), 5301)
    x = _xb(m, k, seed=53)
    y = packed_linear(lin).prefill(x.to(dev()))
    torch.cuda.synchronize()
    y_ref, bound = oracle_ref(lin, x)
    err = np.abs(np_(y).astype(np.float64) - y_ref)
    assert np.all(err <= 3 * (k + 2 * 20 + 32) * 2.0 ** -24 * bound)


def test_gemm_fractional_zero_points_take_at_most_twice_as_long():
    """A zero point that is not an integer costs a second pass over its group's
    products, not a second unpacking: less than twice the time (of graph replays,
    so that the host's share does not count)."""
    n, k, m = 5120, 5120, 512
    blocks = [(2, 1024), (3, 1536), (4, 1760), (8, 736), (16, 64)]
    x = _xb(m, k, seed=54).to(dev())
    times = []
    for fractional in (False, True):
        lin = random_quant_linear(n, k, blocks, seed=54, mode="codes")
        pl = packed_linear(_fractional(lin, 54) if fractional else lin)
        batch = pq.PreparedBatch("gemm", [(pl.layout, pl.packed, pl.perm, x, None)])
        batch.run()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                batch.run()
        runs = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b))
        times.append(sorted(runs)[4])
    assert times[1] < 2 * times[0], times


# Blocks of 13-16 chunks, four groups each (the weights' loads run two groups
# ahead): all but the 8-bit block end in a partial group.
STEADY = [(2, 416), (3, 448), (4, 480), (8, 512), (16, 416)]


@pytest.mark.parametrize("launch", ["split_k", "batch"])
@pytest.mark.parametrize("zp", ["integer", "small_non_integer"])
def test_gemm_steady_groups_every_bit_width(launch, zp):
    """Long blocks of every bit-width: a single linear and a two-linear batch,
    whose K splits start inside blocks; integer zero points, and rows with small
    non-integer ones in every group.  300 tokens: the last token tile is ragged;
    130 rows: the row block has a tile past the end."""
    k = sum(ln for _, ln in STEADY)
    make = _small_z_linear if zp == "small_non_integer" else (
        lambda n, k_, bl, seed: random_quant_linear(n, k_, bl, seed=seed, mode="codes"))
    lins = [make(130, k, STEADY, 5100), make(64, k, STEADY, 5101)]
    lins[1].perm = lins[0].perm
    pls = [packed_linear(lin) for lin in lins]
    x = _xb(300, k, seed=51)
    xd = x.to(dev())
    if launch == "split_k":
        ys = [pls[0].prefill(xd)]
        lins = lins[:1]
    else:
        ys = pq.prefill_batch(pls, [xd, xd])
    torch.cuda.synchronize()
    for lin, y in zip(lins, ys):
        y_ref, bound = oracle_ref(lin, x)
        assert_parity(y, y_ref, bound, f"gemm steady {launch} {zp} n={lin.n}")


def test_gemm_row_gather_past_the_prefetched_passes():
    """K = 20480: the prefill row gather stages the row in LDS but loads the
    indices of its last passes (past the first 16384 channels) in its loop."""
    blocks = [(2, 8192), (3, 6144), (4, 4096), (8, 1024), (16, 1024)]
    k = sum(ln for _, ln in blocks)
    lin = random_quant_linear(80, k, blocks, seed=61, mode="codes")
    pl = packed_linear(lin)
    xb = _xb(9, k, seed=62)
    y = pl.prefill(xb.to(dev()))
    torch.cuda.synchronize()
    y_ref, bound = oracle_ref(lin, xb)
    assert_parity(y, y_ref, bound, "gemm k=20480")


# Every block-end form (1 .. 4 chunks in the last group), two 16-bit groups, and
# enough groups for K splits that start inside blocks.
EDGE_BLOCKS = [(2, 544), (3, 320), (4, 608), (8, 256), (16, 160)]


@pytest.mark.parametrize("n", [1, 64, 130, 257, 600])
@pytest.mark.parametrize("m", [1, 16, 17, 33, 48, 80, 81, 112, 128, 129, 250])
def test_gemm_token_and_row_tile_edges(n, m):
    """Token counts at the edges of token tiles, and work-groups with 1 .. 4
    packed tiles (and a tile past the end), K split, one or two token tiles per
    work-group: fp32 sums of exact products, so the error stays below the worst case
    of any summation order, (k + groups + splits) roundings of 2^-24 of
    sum |w_hat x|."""
    k = sum(ln for _, ln in EDGE_BLOCKS)
    lin = random_quant_linear(n, k, EDGE_BLOCKS, seed=7000 + n, mode="codes")
    zz = lin.zeros.clone()
    zz[n // 2, 2] = 5.5   # one group of one wave takes the second pass
    lin.zeros = zz
    pl = packed_linear(lin)
    x = _xb(m, k, seed=m)
    y = pl.prefill(x.to(dev()))
    y2 = pl.prefill(x.to(dev()))
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    y_ref, bound = oracle_ref(lin, x)
    err = np.abs(np_(y).astype(np.float64) - y_ref)
    # the non-integer zero point splits its group's products in two parts, |q - zi| +
    # |zi - z| <= 3 |q - z|: at most three times the rounding
    tol = np.full(n, (k + 18 + 32) * 2.0 ** -24)
    tol[n // 2] *= 3
    assert np.all(err <= tol * bound)


@pytest.fixture(scope="module")
def tall():
    """65536 rows: 256 row blocks, so a launch is one round at one work-group per
    row block and the plan takes every token tile of the prompt into it."""
    blocks = [(2, 160), (3, 96), (4, 128), (8, 96), (16, 160)]
    lin = random_quant_linear(65536, 640, blocks, seed=8100, mode="codes")
    zz = lin.zeros.clone()
    zz[33000, 1] = 5.5
    lin.zeros = zz
    return lin, packed_linear(lin)


@pytest.mark.parametrize("m", [16, 17, 33, 64, 65, 96, 97, 128, 129])
def test_gemm_every_token_tile_count(tall, m):
    """One full round of work-groups at 1 .. 8 token tiles each, and two rounds, on
    short blocks (one or two groups) and sampled rows of every wave and the rows
    around a non-integer zero point: the bound of test_gemm_token_and_row_tile_edges."""
    lin, pl = tall
    x = _xb(m, lin.k, seed=m)
    y = pl.prefill(x.to(dev()))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(0, 256, 5), np.arange(32992, 33008), np.arange(65400, 65536, 7)]))
    y_ref, bound = oracle_ref(lin, x, rows=rows)
    err = np.abs(np_(y)[:, rows].astype(np.float64) - y_ref)
    tol = np.full(len(rows), (lin.k + 18 + 32) * 2.0 ** -24)
    tol[rows == 33000] *= 3
    assert np.all(err <= tol * bound)


# Rows and tokens whose plan has the token tiles and splits named: GEMM_FORMS in
# tests/host/plan_check.cpp asserts each.  Every block has three groups or more and
# the last row block is ragged.
LONG = [(2, 1440), (3, 1472), (4, 1504), (8, 1536), (16, 416)]
GEMM_FORMS = {
    "1, split": (LONG, 2051, 11), "1": (STEADY, 40963, 3),
    "2, split": (LONG, 1157, 183), "2": (STEADY, 3205, 577),
    "3, split": (LONG, 1157, 337), "3": (STEADY, 5381, 401),
    "4, split": (LONG, 2051, 374), "4": (STEADY, 5381, 529),
    "5, split": (LONG, 2051, 449), "5": (STEADY, 8195, 449),
    "6, split": (LONG, 3205, 361), "6": (STEADY, 8195, 561),
    "7, split": (LONG, 3205, 321), "7": (STEADY, 12805, 481),
    "8, split": (LONG, 3205, 481), "8": (STEADY, 12805, 561),
}


@pytest.mark.parametrize("form", list(GEMM_FORMS))
def test_gemm_every_form(form):
    """Every kernel instance (1 .. 8 token tiles per work-group) with K whole and
    split inside blocks, a non-integer zero point in a block of each bit-width:
    rows of the first and the ragged last row block, and those around the zero
    points, within the bound of test_gemm_token_and_row_tile_edges."""
    blocks, n, m = GEMM_FORMS[form]
    k = sum(ln for _, ln in blocks)
    lin = random_quant_linear(n, k, blocks, seed=8400 + n, mode="codes")
    fractional, g0 = {}, 0
    for i, (b, ln) in enumerate(blocks[:4]):
        groups = -(-ln // 128)
        for g in (0, groups - 1):     # the block's first and its last (partial) group
            r = (n // 5) * i + 40 * (g > 0) + 7
            lin.zeros[r, g0 + g] = 1.5 + 0.25 * i
            fractional[r] = b
        g0 += groups
    x = _xb(m, k, seed=m)
    y = packed_linear(lin).prefill(x.to(dev()))
    torch.cuda.synchronize()
    near = np.concatenate([np.arange(r - 3, r + 4) for r in fractional])
    rows = np.unique(np.concatenate([np.arange(0, 256, 17), np.arange(n - n % 256 - 20, n, 13), [n - 1], near]))
    y_ref, bound = oracle_ref(lin, x, rows=rows)
    err = np.abs(np_(y)[:, rows].astype(np.float64) - y_ref)
    tol = np.full(len(rows), (k + 52 + 32) * 2.0 ** -24)
    tol[np.isin(rows, list(fractional))] *= 3
    assert np.all(err <= tol * bound)


@pytest.mark.parametrize("clustered", [True, False])
def test_gemm_batch_runs_in_the_room_of_its_copies(clustered):
    """A batch needs only the permuted copies: with less than the query it splits
    K as far as the partial sums fit (not at all without room), with the same
    parity; a single linear keeps its queried size.  18 groups and 33 tokens:
    the full plan splits K nine ways."""
    blocks = [(2, 992), (3, 704), (4, 256), (8, 64), (16, 32)]
    k, m, ns = 2048, 33, (320, 130)
    lins = [random_quant_linear(n, k, blocks, seed=610 + i, mode="gauss") for i, n in enumerate(ns)]
    lins[1].perm = lins[0].perm
    pls = [packed_linear(lin) for lin in lins]
    x = _xb(m, k, seed=61)
    xd = x.to(dev())
    perm = None if clustered else pls[0].perm
    given = pls[0].permute(xd) if clustered else xd
    ys = [torch.empty((m, n), device=dev()) for n in ns]
    arr = (pq._lib.GemvItem * 2)(*[pq._lib.GemvItem(ctypes.pointer(pl.layout), pl.packed.data_ptr(), pq._lib._ptr(perm),
                                                    given.data_ptr(), y.data_ptr(), None) for pl, y in zip(pls, ys)])
    lib, copies = pq.lib(), 0 if clustered else m * k * 2
    full = lib.polyq_gemm_batch_workspace_bytes(arr, 2, m)
    partial = sum(-(-m * n * 4 // 256) * 256 for n in ns)
    assert copies % 256 == 0 and full > copies + 2 * partial
    ws = torch.empty(full, dtype=torch.uint8, device=dev())
    for room, at in [(copies, 0), (copies + 2 * partial, 0), (full - 1, 0), (full, 0)] + [(full - 4, 4)] * clustered:
        for y in ys:
            y.fill_(float("nan"))
        ptr = ws.data_ptr() + at if room else None
        assert lib.polyq_gemm_batch(arr, 2, m, ptr, room, None) == 0, (room, at)
        torch.cuda.synchronize()
        for lin, y in zip(lins, ys):
            y_ref, bound = oracle_ref(lin, x)
            assert_parity(y, y_ref, bound, f"gemm batch in {room} of {full} bytes n={lin.n}")
    if not clustered:
        assert lib.polyq_gemm_batch(arr, 2, m, ws.data_ptr(), copies - 1, None) == 5   # POLYQ_ERR_CAPACITY
        assert lib.polyq_gemm_batch(arr, 2, m, ws.data_ptr() + 4, full - 4, None) == 1  # POLYQ_ERR_ARG
    one = lib.polyq_gemm_batch_workspace_bytes(arr, 1, m)
    assert one > copies and lib.polyq_gemm_batch(arr, 1, m, ws.data_ptr(), one - 1, None) == 5
