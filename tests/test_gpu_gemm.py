"""Parity of the shard-product kernels with the fp64 oracle.
bf16 inputs / fp32 accumulate: |gpu - oracle| <= 1e-2 * (|A| |B|)_ij  (+ half an ulp of a bf16 store);
fp32: <= 1e-5 * (|A| |B|)_ij."""
import itertools

import numpy as np
import pytest
import torch

import paper_1805_04170_amd as tt
from oracle import layers as ly
from synthetic import bf16_bits_to_f64, normal_f32, to_bf16_bits

from gpu_util import DEV, dev_to_np, np_to_dev

pytestmark = pytest.mark.gpu


def check(count, M, N, K, ta, tb, in_dt, out_dt, relu, seed):
    bf = in_dt == "bf16"
    As, Bs, Cs, want, mags = [], [], [], [], []
    for s in range(count):
        a = normal_f32(seed, 2 * s, (M, K), 1.0)
        b = normal_f32(seed, 2 * s + 1, (K, N), 0.05)
        if bf:
            a, b = to_bf16_bits(a), to_bf16_bits(b)
        af = bf16_bits_to_f64(a) if bf else a.astype(np.float64)
        bfl = bf16_bits_to_f64(b) if bf else b.astype(np.float64)
        z = af @ bfl
        want.append(np.maximum(z, 0) if relu else z)
        mags.append(ly.abs_product(af, bfl))
        As.append(np_to_dev(a.T if ta else a, bf))
        Bs.append(np_to_dev(b.T if tb else b, bf))
        Cs.append(torch.full((M, N), float("nan"), dtype=torch.bfloat16 if out_dt == "bf16" else torch.float32, device=DEV))
    tt.tt_shard_gemm(As, Bs, Cs, M, N, K, ta, tb, in_dt, out_dt, tt.TT_ACT_RELU if relu else tt.TT_ACT_NONE)
    torch.cuda.synchronize()
    for s in range(count):
        got = dev_to_np(Cs[s])
        gf = bf16_bits_to_f64(got) if out_dt == "bf16" else got.astype(np.float64)
        tol = (1e-2 if bf else 1e-5) * mags[s]                      # the stated bound, nothing added
        err = np.abs(gf - want[s])
        assert np.all(np.isfinite(gf)), (s, "non-finite output")
        assert np.all(err <= tol + 1e-30), (s, float(err.max()), float((err / (tol + 1e-30)).max()))
        # the bound is loose for fp32 accumulation; also require a tight typical error so a dropped k-tile cannot hide:
        # 1e-4 of the magnitude product, plus the rounding of the stored result where that is bf16 (8 significant bits,
        # round to nearest: at most 2^-8 of the value)
        if bf:
            tight = 1e-4 * mags[s] + (2.0 ** -8 * np.abs(want[s]) if out_dt == "bf16" else 0.0)
            assert np.all(err <= tight + 1e-30), (s, float((err / (tight + 1e-30)).max()))


LAYOUTS = [(0, 0), (0, 1), (1, 0), (1, 1)]


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
def test_bf16_mfma_tiles_and_tails(ta, tb, out_dt):
    # several 128/256 tiles plus ragged tails in M, N and K (all multiples of 8 along contiguous dims)
    check(3, 264, 200, 328, ta, tb, "bf16", out_dt, False, 31)
    check(2, 128, 136, 64, ta, tb, "bf16", out_dt, True, 32)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
def test_bf16_small_and_tall(ta, tb):
    check(8, 32, 512, 1024, ta, tb, "bf16", "f32", False, 33)      # batch-split shard: few rows
    check(1, 520, 72, 40, ta, tb, "bf16", "bf16", False, 34)        # three row tiles, one short K tile


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M", [1, 16, 32, 33, 64, 65])
def test_bf16_few_rows(M, tb):
    # a small batch against wide weights: 32- and 64-row tiles, ragged columns, K with and without a tail, K of one tile
    check(8, M, 1000, 328, 0, tb, "bf16", "bf16", True, 70)
    check(3, M, 264, 64, 0, tb, "bf16", "f32", False, 71)
    check(1, M, 136, 1024, 0, tb, "bf16", "f32", False, 72)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
def test_bf16_unaligned_falls_back(ta, tb):
    check(2, 37, 125, 50, ta, tb, "bf16", "bf16", True, 35)         # 125-wide rows: no 16-byte vectors
    check(2, 33, 10, 17, ta, tb, "bf16", "f32", False, 36)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
def test_fp32(ta, tb):
    check(4, 32, 10, 256, ta, tb, "f32", "f32", False, 37)
    check(2, 70, 130, 65, ta, tb, "f32", "f32", True, 38)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_odd_sized_products(ta, tb, dt):
    # K over one, two, four and eight waves with tails; single results; enough 64 x 64 blocks for those, with one row or
    # column left over (the row pairs of bf16 operands)
    for i, (n, M, N, K) in enumerate([(2, 33, 47, 1051), (1, 1, 1, 1), (3, 40, 31, 263), (1, 5, 67, 131), (4, 577, 449, 515), (8, 257, 450, 97)]):
        check(n, M, N, K, ta, tb, dt, dt if i % 2 else "f32", bool(i & 1), 60 + i)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_short_odd_sized_products(ta, tb, dt):
    # both kernels on either side of the lines: few tiles (K = 16 and 17), a strip, tiles for every CU
    for i, (n, M, N, K) in enumerate([(2, 65, 35, 16), (2, 65, 35, 17), (1, 33, 131, 33), (1, 5, 33001, 15), (64, 65, 67, 9), (64, 65, 67, 97), (5, 511, 513, 31)]):
        check(n, M, N, K, ta, tb, dt, dt if i % 2 else "f32", bool(i & 1), 80 + i)


def test_odd_sized_forward_products_of_many_tiles():
    check(8, 511, 513, 83, 0, 0, "bf16", "bf16", True, 67)         # 64 x 64 tiles, two per CU
    check(1, 2047, 1025, 17, 0, 0, "bf16", "f32", False, 68)


@pytest.mark.parametrize("M,N,K", [(33, 35, 1), (1, 67, 65), (65, 1, 129), (100, 225, 1500), (1023, 961, 63), (32, 100, 257)])
def test_odd_sized_forward_products_add_in_the_order_of_k(M, N, K):
    # bit for bit a chain of fp32 fused multiply-adds (float64 holds every sum of these operands exactly), on either tile
    rng = np.random.default_rng(M + N + K)
    a, b = (to_bf16_bits(rng.uniform(0.25, 2.0, s).astype(np.float32) * rng.choice([-1, 1], s).astype(np.float32)) for s in ((M, K), (K, N)))
    af, bf = bf16_bits_to_f64(a), bf16_bits_to_f64(b)
    want = np.zeros((M, N), np.float32)
    for k in range(K):
        want = (want.astype(np.float64) + af[:, k:k + 1] * bf[k:k + 1]).astype(np.float32)
    c = torch.empty((M, N), dtype=torch.float32, device=DEV)
    up = [torch.from_numpy(x.view(np.int16)).to(DEV).view(torch.bfloat16) for x in (a, b)]
    tt.tt_shard_gemm([up[0]], [up[1]], [c], M, N, K, 0, 0, "bf16", "f32")
    assert np.array_equal(dev_to_np(c), want)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
def test_products_without_terms_are_zero(ta, tb):
    # K = 0: operands of no elements (their addresses are not read), results of zeros
    for M, N, dt, out, count in itertools.product((1, 33), (1, 33), ("bf16", "f32"), ("bf16", "f32"), (1, 3)):
        a = [torch.ones(64, dtype=torch.bfloat16 if dt == "bf16" else torch.float32, device=DEV) for _ in range(count)]
        c = [torch.full((M, N), float("nan"), dtype=torch.bfloat16 if out == "bf16" else torch.float32, device=DEV) for _ in range(count)]
        tt.tt_shard_gemm(a, a, c, M, N, 0, ta, tb, dt, out)
        for x in c:
            assert torch.equal(x.cpu(), torch.zeros((M, N), dtype=x.dtype)), (M, N, dt, out)


def run_error_against_one_chain(ta, tb, M, N, K, dt):
    # fp32 results of odd-sized products that need not keep the order of K are cut into four chains of additions or more.  The error
    # of a chain of n additions grows at least as the square root of n (0.5 of a single chain's for four; 0.6 here, as the first
    # additions of bf16 products are exact), and joining eight chains adds three levels of additions that round by 2.5e-8 of
    # the result each (uniform rounding: 2^-24 / sqrt(3), 0.72 of it on average over the mantissa): 4.3e-8 together.
    rng = np.random.default_rng(K + ta + 2 * tb)
    a, b = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (K, N)))
    if dt == "bf16":
        a, b = (bf16_bits_to_f64(to_bf16_bits(x)).astype(np.float32) for x in (a, b))
    one = np.zeros((M, N), np.float32)
    for k in range(K):      # fused: the product of two fp32 values is exact in float64, and the sum is rounded to fp32 next to correctly
        one = (one.astype(np.float64) + a[:, k:k + 1].astype(np.float64) * b[k:k + 1]).astype(np.float32)
    want = a.astype(np.float64) @ b.astype(np.float64)
    c = torch.empty((M, N), dtype=torch.float32, device=DEV)
    up = [torch.from_numpy(np.ascontiguousarray(x)).to(torch.bfloat16 if dt == "bf16" else torch.float32).to(DEV) for x in (a.T if ta else a, b.T if tb else b)]
    tt.tt_shard_gemm([up[0]], [up[1]], [c], M, N, K, ta, tb, dt, "f32")
    got = np.linalg.norm(dev_to_np(c).astype(np.float64) - want)
    bound = np.hypot(0.6 * np.linalg.norm(one.astype(np.float64) - want), 4.3e-8 * np.linalg.norm(want))
    assert bound < 0.9 * np.linalg.norm(one.astype(np.float64) - want)      # (a single chain would not pass)
    assert got <= bound, (ta, tb, M, N, K, dt)


@pytest.mark.parametrize("ta,tb", [(0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K", [(101, 225, 129), (257, 255, 255), (257, 255, 447), (1023, 961, 159), (1281, 1279, 191)])
def test_odd_sized_products_are_not_one_chain_of_additions(ta, tb, dt, M, N, K):
    run_error_against_one_chain(ta, tb, M, N, K, dt)


def test_fp32_keeps_subnormal_products_and_sums():
    # results below the smallest normal fp32 number (1.2e-38): K = 64 products of 2^-70 x 2^-65
    a = torch.full((40, 64), 2.0 ** -70, dtype=torch.float32, device=DEV)
    b = torch.full((64, 33), 2.0 ** -65, dtype=torch.float32, device=DEV)
    c = torch.empty((40, 33), dtype=torch.float32, device=DEV)
    tt.tt_shard_gemm([a], [b], [c], 40, 33, 64, 0, 0, "f32", "f32")
    assert np.all(dev_to_np(c).astype(np.float64) == 2.0 ** -129)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
def test_bf16_large_launch_eight_wave_tiles(ta, tb):
    # enough 256 x 256 tiles for the eight-wave kernels (both tile engines, chosen by layout), ragged M, N and K
    check(8, 1000, 1016, 200, ta, tb, "bf16", "bf16", True, 39)
    check(8, 1024, 1024, 192, ta, tb, "bf16", "f32", False, 40)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
def test_bf16_persistent_engine(ta, tb, out_dt):
    # K a multiple of 64 and more 256 x 256 tiles than CUs: the persistent pipelined engine, several output tiles per
    # workgroup (prefetch runs across tile boundaries), ragged M and N, K loops of one, two and five tiles
    check(8, 1544, 1528, 128, ta, tb, "bf16", out_dt, True, 42)
    check(8, 1032, 1544, 64, ta, tb, "bf16", out_dt, False, 43)
    check(3, 2056, 1800, 320, ta, tb, "bf16", out_dt, False, 44)
    # three output tiles per workgroup and a K loop of four tiles: a full tile's write-out rides along the next one
    check(8, 2056, 2312, 256, ta, tb, "bf16", out_dt, True, 48)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
def test_bf16_two_workgroups_per_cu_engine(ta, tb, out_dt):
    # launches with few 256 x 256 tiles, K a multiple of 32: the 256 x 128 engine (three-stage ring of 32-deep K tiles);
    # ragged M and N, K loops of 3 (the ring is deeper than one of the loops is long) and 16 tiles
    check(2, 520, 520, 96, ta, tb, "bf16", out_dt, True, 45)
    check(8, 256, 1024, 512, ta, tb, "bf16", out_dt, False, 46)
    check(1, 136, 264, 32, ta, tb, "bf16", out_dt, False, 47)


@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
def test_bf16_line_wide_k_tiles_engine(out_dt):
    # skinny A B^T products with at most one 256 x 128 tile per CU and K a multiple of 64 (the data gradients at batch
    # 256): the 256 x 128 engine with K tiles of 64 (two stages of A, three of B); ragged N, ragged M, K loops of 8, 4
    # and 64 tiles, the last at the shape of the VGG-16 first data gradient
    check(16, 256, 1064, 512, 0, 1, "bf16", out_dt, True, 49)
    check(32, 200, 392, 256, 0, 1, "bf16", out_dt, False, 50)
    check(6, 256, 3136, 4096, 0, 1, "bf16", out_dt, False, 51)


@pytest.mark.parametrize("K", [256, 128, 512])
def test_bf16_panel_in_registers_engine(K):
    # weight-gradient shaped products (both operands stored K-major, K = 128 / 256, large bf16 result): the engine that
    # keeps the left operand's panel in registers; 8 shards x 5 panels (the last with 8 of 256 rows) x 52 column tiles
    # on 512 resident workgroups, so runs change panel and shard mid-way
    check(8, 1032, 3328, K, 1, 0, "bf16", "bf16", K == 128, 48)


@pytest.mark.parametrize("K", [1, 40, 64, 72, 128, 219])
def test_bf16_panel_in_registers_engine_at_other_k_and_widths(K):
    # any K inside the next of 64, 128 and 256; the last unit of a panel 8 columns wide, the last panel with 8 rows
    check(2, 2056, 4104, K, 1, 0, "bf16", "bf16", K == 72, 110)


@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
@pytest.mark.parametrize("ta,tb,K", [(0, 1, 512), (0, 1, 520), (0, 0, 1024), (0, 0, 1032), (1, 0, 2048), (1, 0, 2056), (1, 1, 2104)])
def test_bf16_k_tiles_of_64_two_on_their_way(ta, tb, K, out_dt):
    # the 256 x 128 engine with three stages of 64, every layout, whole and short last K tiles
    check(2, 264, 392, K, ta, tb, "bf16", out_dt, K % 64 == 0, 111)


@pytest.mark.parametrize("ta,tb,K", [(0, 0, 1032), (0, 1, 520), (1, 0, 2056), (1, 1, 264)])
def test_bf16_large_products_of_short_last_k_tiles(ta, tb, K):
    # more 256 x 256 tiles than CUs and K outside what the other engines take: the direct-to-LDS kernel of that size
    check(8, 1288, 1288, K, ta, tb, "bf16", "bf16", True, 112)


@pytest.mark.parametrize("M,N,K,tb", [(65, 136, 384, 1), (128, 264, 392, 0), (72, 1176, 4640, 1), (33, 136, 2056, 0), (32, 264, 1032, 0), (1, 136, 1024, 0)])
def test_bf16_few_rows_straight_into_lds(M, N, K, tb):
    # 64- and 32-row tiles with three stages: whole and short rows, columns and K tiles
    check(2, M, N, K, 0, tb, "bf16", "f32" if M % 2 else "bf16", M % 2 == 0, 113)


@pytest.mark.parametrize("count,M,N,K,ta,tb", [(1, 4104, 4096, 100, 1, 0), (1, 4104, 4096, 256, 1, 0), (1, 4096, 4104, 512, 1, 0), (2, 520, 520, 96, 1, 0),
                                               (2, 300, 520, 1032, 0, 0), (8, 1544, 1528, 128, 0, 1), (8, 1288, 1288, 1032, 0, 0), (1, 72, 136, 392, 0, 1)])
def test_values_that_are_not_finite_stay_what_they_are(count, M, N, K, ta, tb):
    # a NaN and an infinity in the left operand, an infinity in the right one, on the engines that a product can run on
    a, b = to_bf16_bits(normal_f32(97, 0, (M, K), 1.0)), to_bf16_bits(normal_f32(97, 1, (K, N), 0.05))
    a[5, 3], a[9, 7], b[2, 20] = 0x7FC0, 0x7F80, 0xFF80
    with np.errstate(invalid="ignore"):
        want = bf16_bits_to_f64(a) @ bf16_bits_to_f64(b)
    A, B = [np_to_dev(a.T if ta else a, True)] * count, [np_to_dev(b.T if tb else b, True)] * count
    C = [torch.zeros((M, N), dtype=torch.bfloat16, device=DEV) for _ in range(count)]
    tt.tt_shard_gemm(A, B, C, M, N, K, ta, tb, "bf16", "bf16")
    for c in C:
        got = bf16_bits_to_f64(dev_to_np(c))
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.isnan(got[5]).all()
        assert np.array_equal(got == np.inf, want == np.inf) and np.array_equal(got == -np.inf, want == -np.inf)


def test_k_zero_and_empty():
    C = [torch.full((8, 8), 5.0, dtype=torch.float32, device=DEV)]
    A = [torch.zeros((8, 1), dtype=torch.bfloat16, device=DEV)]
    tt.tt_shard_gemm(A, A, C, 8, 8, 0, 0, 0, "bf16", "f32")
    torch.cuda.synchronize()
    assert torch.all(C[0] == 0)
    tt.tt_shard_gemm(A, A, C, 0, 8, 4, 0, 0, "bf16", "f32")          # nothing to do


def test_vgg_shard_shape_every_element():
    # the K-split shard product of the VGG-16 first classifier layer: 256 x 3136 x 4096, fp32 partial output
    M, K, N = 256, 3136, 4096
    a = to_bf16_bits(normal_f32(41, 0, (M, K), 1.0)); b = to_bf16_bits(normal_f32(41, 1, (K, N), 0.005))
    A = [np_to_dev(a, True)]; B = [np_to_dev(b, True)]
    C = [torch.empty((M, N), dtype=torch.float32, device=DEV)]
    tt.tt_shard_gemm(A, B, C, M, N, K, 0, 0, "bf16", "f32")
    torch.cuda.synchronize()
    got = dev_to_np(C[0]).astype(np.float64)
    af, bfl = bf16_bits_to_f64(a), bf16_bits_to_f64(b)
    want = af @ bfl
    mag = ly.abs_product(af, bfl)
    assert np.all(np.abs(got - want) <= 1e-2 * mag)
    assert float(np.max(np.abs(got - want) / mag)) < 1e-4
