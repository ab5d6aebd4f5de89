"""The shard-product kernels run on the host in lock step (tests/emu/emu_lockstep.h: the threads of a workgroup as
cooperative fibers, barriers that hold, MFMA and the LDS transpose read computing what the instructions compute) and
their results compared with the oracle's, to the bar of the GPU tests.  The entry point is the library's own
(csrc/gemm.hip and csrc/gemm3.hip compiled for the host as they are), so every engine is reached the way the library
reaches it.  What this cannot show is what only the hardware decides (timing, instruction alignment rules); what it does
show without a GPU: tile and fragment indexing, LDS layouts, K tails, write-out, the K split inside a launch.
"""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import layers as ly
from synthetic import bf16_bits_to_f64, normal_f32, to_bf16_bits

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = shutil.which("clang++", path="/opt/rocm/llvm/bin") or shutil.which("clang++")
pytestmark = pytest.mark.skipif(CLANG is None, reason="no host clang++ for the emulation build")


@pytest.fixture(scope="module")
def lockstep_gemm(emulators):
    return emulators.get("shard_gemm_lockstep")


def check(exe, tmp, count, M, N, K, ta, tb, in_dt, out_dt, relu, seed, ksplit=1, env=None):
    bf = in_dt == "bf16"
    want, mags = [], []
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
        np.ascontiguousarray(a.T if ta else a).tofile(os.path.join(tmp, "a%d.bin" % s))
        np.ascontiguousarray(b.T if tb else b).tofile(os.path.join(tmp, "b%d.bin" % s))
    e = dict(os.environ)
    e.update(env or {})
    r = subprocess.run([exe] + [str(v) for v in (count, M, N, K, ta, tb, int(bf), int(out_dt == "bf16"), int(relu), ksplit, tmp)],
                       capture_output=True, text=True, env=e)
    assert r.returncode == 0, r.stdout[-400:] + r.stderr[-1500:]
    for s in range(count):
        # with a K split the launch leaves ksplit partial products per shard, to be summed
        gf = np.zeros((M, N))
        for q in range(ksplit):
            raw = np.fromfile(os.path.join(tmp, "c%d.bin" % (s * ksplit + q)), dtype=np.uint16 if out_dt == "bf16" else np.float32)
            gf += (bf16_bits_to_f64(raw) if out_dt == "bf16" else raw.astype(np.float64)).reshape(M, N)
        tol = (1e-2 if bf else 1e-5) * mags[s]
        err = np.abs(gf - want[s])
        assert np.all(np.isfinite(gf)), (s, "non-finite output")
        assert np.all(err <= tol + 1e-30), (s, float(err.max()), float((err / (tol + 1e-30)).max()), np.argwhere(err > tol + 1e-30)[:5])
        if bf and out_dt == "f32" and not relu:
            assert float(np.max(err / (mags[s] + 1e-30))) < 1e-4
    return r.stdout


LAYOUTS = [(0, 0), (0, 1), (1, 0), (1, 1)]


@pytest.mark.parametrize("ta,tb", LAYOUTS)
def test_register_staged_engine_values(lockstep_gemm, tmp_path, ta, tb):
    check(lockstep_gemm, str(tmp_path), 2, 264, 200, 104, ta, tb, "bf16", "bf16", False, 31)   # ragged on every side, K mask
    check(lockstep_gemm, str(tmp_path), 1, 136, 72, 64, ta, tb, "bf16", "f32", True, 32)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
def test_two_workgroups_per_cu_engine_values(lockstep_gemm, tmp_path, ta, tb, out_dt):
    # few 256 x 256 tiles: the 256 x 128 engine; ragged M and N, a K loop shorter than its ring and a longer one
    out = check(lockstep_gemm, str(tmp_path), 1, 264, 392, 96, ta, tb, "bf16", out_dt, True, 45)
    assert int(out.split()[3]) == 8 * 256      # 2 x 4 tiles of 256 x 128, 256 threads each
    check(lockstep_gemm, str(tmp_path), 2, 136, 264, 32, ta, tb, "bf16", out_dt, False, 47)
    check(lockstep_gemm, str(tmp_path), 1, 256, 256, 256, ta, tb, "bf16", out_dt, False, 46)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
def test_persistent_engine_values(lockstep_gemm, tmp_path, ta, tb, out_dt):
    # on a stand-in device of 16 CUs, with the engine and tile forced the way the tuning switches allow: 24 ragged
    # tiles, one or two per workgroup (the operand ring runs across tile boundaries), K loops of one and three tiles
    env = {"EMU_CUS": "16", "TT_GEMM_ENGINE": "3", "TT_GEMM_TILE": "5"}
    out = check(lockstep_gemm, str(tmp_path), 2, 520, 776, 64, ta, tb, "bf16", out_dt, True, 42, env=env)
    assert int(out.split()[3]) == 16 * 512
    check(lockstep_gemm, str(tmp_path), 1, 264, 520, 192, ta, tb, "bf16", out_dt, False, 44, env=env)


@pytest.mark.parametrize("tb", [1, 0])
@pytest.mark.parametrize("out_dt", ["bf16", "f32"])
def test_line_wide_k_tiles_engine_values(lockstep_gemm, tmp_path, out_dt, tb):
    # the 256 x 128 engine with K tiles of 64 for A B^T products (two stages of A, three of B, waits that count loads):
    # ragged M and N, K loops of one tile (shorter than either ring), three and seven tiles, a K split inside the launch
    env = {"TT_GEMM_ENGINE": "6"}
    out = check(lockstep_gemm, str(tmp_path), 1, 264, 392, 192, 0, tb, "bf16", out_dt, True, 48, env=env)
    assert int(out.split()[3]) == 8 * 256      # 2 x 4 tiles of 256 x 128, 256 threads each
    check(lockstep_gemm, str(tmp_path), 2, 136, 264, 64, 0, tb, "bf16", out_dt, False, 49, env=env)
    check(lockstep_gemm, str(tmp_path), 1, 256, 256, 448, 0, tb, "bf16", out_dt, False, 50, env=env)
    if out_dt == "f32":
        check(lockstep_gemm, str(tmp_path), 2, 256, 136, 320, 0, tb, "bf16", "f32", False, 51, ksplit=2, env=env)   # chunks of 192 and 128


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("engine", ["4", "6"])
def test_short_last_k_tile_values(lockstep_gemm, tmp_path, engine, ta, tb):
    # K ends in the first tile, after 8 of 32 or of 64 values, in the middle of a tile
    for i, K in enumerate((8, 72, 104) + ((37,) if ta and not tb else ())):
        check(lockstep_gemm, str(tmp_path), 1, 264, 264, K, ta, tb, "bf16", "bf16" if i % 2 else "f32", bool(i % 2), 55 + i, env={"TT_GEMM_ENGINE": engine})


@pytest.mark.parametrize("M,K,tb", [(65, 384, 1), (128, 392, 0), (100, 520, 1), (33, 2048, 0), (64, 2056, 0), (1, 1032, 0), (32, 1024, 0)])
def test_few_rows_straight_into_lds_values(lockstep_gemm, tmp_path, M, K, tb):
    # 64- and 32-row tiles, full and short ones, K tails; 136 columns: the second tile with 8
    out = check(lockstep_gemm, str(tmp_path), 1, M, 136, K, 0, tb, "bf16", "f32" if M % 2 else "bf16", bool(M % 2), 95)
    assert int(out.split()[3]) == 8 * 256      # two or four tiles, a multiple of eight workgroups


@pytest.mark.parametrize("K", [1, 40, 64, 72, 219, 300])
def test_panel_in_registers_engine_values_at_other_k_and_widths(lockstep_gemm, tmp_path, K):
    # K inside the next of 64, 128, 256, 512; the last unit 8 columns wide (rows of 16-byte pieces), or whole
    env = {"EMU_CUS": "1", "TT_GEMM_ENGINE": "5"}
    out = check(lockstep_gemm, str(tmp_path), 1, 264, 136, K, 1, 0, "bf16", "bf16", True, 90, env=env)
    assert int(out.split()[3]) == (1 if K > 256 else 2) * 256
    check(lockstep_gemm, str(tmp_path), 1, 256, 192, K, 1, 0, "bf16", "bf16", False, 91, env=env)


@pytest.mark.parametrize("N,K,takes", [(2 ** 27, 1, 1), (2 ** 28 - 8, 3, 1), (2 ** 28, 1, 0), (306783384, 1, 0), (2 ** 29, 1, 0), (2 ** 28 - 8, 4, 1)])
def test_panel_in_registers_engine_leaves_rows_too_long_for_its_offsets(lockstep_gemm, N, K, takes):
    # a store's eight rows are addressed with 32-bit byte offsets: 7 rows of 306783384 elements are 2^32 bytes and 80
    r = subprocess.run([lockstep_gemm, "panel", "8", str(N), str(K)], capture_output=True, text=True)
    assert r.returncode == 0 and int(r.stdout) == takes


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("env,ta,tb,K", [({"TT_GEMM_ENGINE": "5", "EMU_CUS": "1"}, 1, 0, K) for K in (64, 100, 128, 256, 512)] +
                         [({"TT_GEMM_ENGINE": "4"}, 1, 0, 104), ({"TT_GEMM_ENGINE": "6"}, 0, 1, 104),
                          ({"TT_GEMM_ENGINE": "3", "TT_GEMM_TILE": "5", "EMU_CUS": "8"}, 1, 0, 128), ({"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": "8"}, 0, 0, 104),
                          ({"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": "0"}, 0, 1, 104), ({"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": "1"}, 1, 0, 104)])
def test_values_that_are_not_finite_stay_what_they_are(lockstep_gemm, tmp_path, env, ta, tb, K, relu):
    # a NaN and an infinity in the left operand, an infinity in the right one: rows and a column of NaN and infinities of both signs,
    # also where sums are rounded to bf16; under the element-wise function NaN gives 0, as -inf does
    M, N, tmp = 264, 136, str(tmp_path)
    a, b = to_bf16_bits(normal_f32(96, 0, (M, K), 1.0)), to_bf16_bits(normal_f32(96, 1, (K, N), 0.05))
    a[5, 3], a[9, 7], b[2, 20] = 0x7FC0, 0x7F80, 0xFF80
    with np.errstate(invalid="ignore"):
        want = (bf16_bits_to_f64(a)[:, :, None] * bf16_bits_to_f64(b)[None]).sum(axis=1)
        want = np.fmax(want, 0) if relu else want
    np.ascontiguousarray(a.T if ta else a).tofile(os.path.join(tmp, "a0.bin"))
    np.ascontiguousarray(b.T if tb else b).tofile(os.path.join(tmp, "b0.bin"))
    r = subprocess.run([lockstep_gemm] + [str(v) for v in (1, M, N, K, ta, tb, 1, 1, int(relu), 1, tmp)], capture_output=True, text=True, env=dict(os.environ, **env))
    assert r.returncode == 0, r.stderr[-1500:]
    got = bf16_bits_to_f64(np.fromfile(os.path.join(tmp, "c0.bin"), dtype=np.uint16)).reshape(M, N)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got == np.inf, want == np.inf) and np.array_equal(got == -np.inf, want == -np.inf)
    assert relu or (np.isnan(want[5]).all() and np.isinf(want).any(axis=0)[30])
    assert np.count_nonzero(np.isfinite(got)) > M * N * 0.9


def test_line_wide_k_tiles_engine_as_the_library_chooses_it(lockstep_gemm, tmp_path):
    # a skinny data-gradient shaped product (one row of tiles, 128 of them for 256 CUs, K of four tiles): no switch set
    check(lockstep_gemm, str(tmp_path), 32, 256, 392, 256, 0, 1, "bf16", "bf16", False, 52)


def test_line_wide_k_tiles_engine_waits_exactly_as_long_as_it_must(lockstep_gemm, tmp_path):
    # with every wait letting two more loads stay in flight than the kernel asks for it must not get away with it; and
    # its results do not depend on which wave runs ahead
    env = {"TT_GEMM_ENGINE": "6"}
    shape = (1, 264, 392, 320, 0, 1, "bf16", "f32", False, 53)
    check(lockstep_gemm, str(tmp_path), *shape, env=env)
    with pytest.raises(AssertionError):
        check(lockstep_gemm, str(tmp_path), *shape, env=dict(env, EMU_VMCNT_SLACK="2"))
    check(lockstep_gemm, str(tmp_path), *shape, env=dict(env, EMU_ORDER="reverse"))


def test_persistent_engine_values_as_the_library_chooses_it(lockstep_gemm, tmp_path):
    # 240 tiles on 256 CUs: the weight-gradient layout, bf16 results (loads interleaved with the K steps)
    out = check(lockstep_gemm, str(tmp_path), 8, 1288, 1272, 64, 1, 0, "bf16", "bf16", False, 43)
    assert int(out.split()[3]) == 240 * 512


@pytest.mark.parametrize("relu", [False, True])
def test_panel_in_registers_engine_values(lockstep_gemm, tmp_path, relu):
    # the short-K engine of the weight gradients (left operand's panel in registers, stores left in flight over the next
    # unit's wait), forced on small products on a stand-in device of one CU (two workgroups): K = 256, two shards of two
    # panels (the second with 72 of its 256 rows: one wave full, one partly masked, two idle) by three column tiles, so
    # every workgroup changes panel and runs units behind stores that are still counted; then K = 128
    env = {"EMU_CUS": "1", "TT_GEMM_ENGINE": "5"}
    out = check(lockstep_gemm, str(tmp_path), 2, 328, 192, 256, 1, 0, "bf16", "bf16", relu, 81, env=env)
    assert int(out.split()[3]) == 2 * 256
    check(lockstep_gemm, str(tmp_path), 1, 264, 128, 128, 1, 0, "bf16", "bf16", relu, 82, env=env)
    # more workgroups than units to spare: runs of one unit, and a run that ends inside a panel
    check(lockstep_gemm, str(tmp_path), 1, 512, 320, 256, 1, 0, "bf16", "bf16", relu, 83, env={"EMU_CUS": "3", "TT_GEMM_ENGINE": "5"})


def test_panel_in_registers_engine_values_at_k_512(lockstep_gemm, tmp_path):
    # K = 512: the panel takes twice the registers and the two stages 128 KB, one workgroup per CU (stand-in device of two
    # CUs: two workgroups); two panels (the second with 40 rows) by five column tiles, so runs change panel mid-way
    env = {"EMU_CUS": "2", "TT_GEMM_ENGINE": "5"}
    out = check(lockstep_gemm, str(tmp_path), 1, 296, 320, 512, 1, 0, "bf16", "bf16", True, 85, env=env)
    assert int(out.split()[3]) == 2 * 256
    shape = (1, 256, 192, 512, 1, 0, "bf16", "bf16", False, 86)
    check(lockstep_gemm, str(tmp_path), *shape, env=dict(env, EMU_ORDER="reverse"))
    with pytest.raises(AssertionError):
        check(lockstep_gemm, str(tmp_path), *shape, env=dict(env, EMU_VMCNT_SLACK="2"))


def test_panel_in_registers_engine_counts_its_stores(lockstep_gemm, tmp_path):
    # its waits leave the previous unit's eight stores in flight; letting two more operations stay in flight than it
    # asks for must give stale operand tiles, and the order in which waves run must not matter
    env = {"EMU_CUS": "1", "TT_GEMM_ENGINE": "5"}
    shape = (1, 256, 512, 256, 1, 0, "bf16", "bf16", False, 84)
    check(lockstep_gemm, str(tmp_path), *shape, env=dict(env, EMU_ORDER="reverse"))
    with pytest.raises(AssertionError):
        check(lockstep_gemm, str(tmp_path), *shape, env=dict(env, EMU_VMCNT_SLACK="2"))


@pytest.mark.parametrize("ta,tb", LAYOUTS)
def test_direct_to_lds_engine_values(lockstep_gemm, tmp_path, ta, tb):
    # the eight-wave 256 x 256 engine that loads tiles straight into LDS, forced by the tuning switches on small
    # products: ragged M and N, a K tail that is no multiple of the tile depth
    env = {"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": "8"}
    out = check(lockstep_gemm, str(tmp_path), 2, 264, 520, 72, ta, tb, "bf16", "bf16", True, 39, env=env)
    assert int(out.split()[3]) == 16 * 512     # 12 tiles, rounded up to a multiple of the 8 XCDs
    check(lockstep_gemm, str(tmp_path), 1, 256, 264, 128, ta, tb, "bf16", "f32", False, 40, env=env)


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4, 5])
def test_register_staged_engine_every_tile_values(lockstep_gemm, tmp_path, tile):
    env = {"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": str(tile)}
    check(lockstep_gemm, str(tmp_path), 1, 264, 392, 104, 0, 0, "bf16", "bf16", False, 50 + tile, env=env)
    check(lockstep_gemm, str(tmp_path), 1, 264, 392, 96, 1, 1, "bf16", "f32", True, 60 + tile, env=env)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
def test_k_split_inside_a_launch_values(lockstep_gemm, tmp_path, ta, tb):
    # the partial products of the chunks add up to the product (chunks of 128, 128 and 64 of K = 320; on the smallest tile
    # chunks of 64, 64 and 22 of K = 150 would leave ... K must keep 16-byte rows: 152)
    check(lockstep_gemm, str(tmp_path), 2, 264, 264, 320, ta, tb, "bf16", "f32", False, 70, ksplit=3)
    check(lockstep_gemm, str(tmp_path), 1, 40, 72, 152, ta, tb, "bf16", "f32", False, 71, ksplit=3)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
def test_generic_kernel_values(lockstep_gemm, tmp_path, ta, tb):
    check(lockstep_gemm, str(tmp_path), 2, 70, 130, 65, ta, tb, "f32", "f32", True, 38)
    check(lockstep_gemm, str(tmp_path), 2, 37, 125, 50, ta, tb, "bf16", "bf16", True, 35)       # rows without 16-byte vectors
    check(lockstep_gemm, str(tmp_path), 1, 33, 10, 17, ta, tb, "bf16", "f32", False, 36, ksplit=1)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_small_kernel_waves_and_blocks_values(lockstep_gemm, tmp_path, dt, ta, tb):
    # every split of the waves (K of one, two, four and eight waves, the last with a tail that is no whole MFMA step),
    # single results, and 64 x 64 blocks with one row or column in the last one (the row pairs of bf16 operands).  (bf16
    # in the forward layout runs on kernels of its own.)
    for i, (M, N, K) in enumerate([(33, 47, 1051), (1, 1, 1), (40, 31, 263), (5, 67, 131)]):
        check(lockstep_gemm, str(tmp_path), 1, M, N, K, ta, tb, dt, "f32", False, 80 + i)
    for i, (M, N, K) in enumerate([(65, 129, 97), (66, 127, 515), (129, 65, 9)]):
        check(lockstep_gemm, str(tmp_path), 1, M, N, K, ta, tb, dt, dt, True, 90 + i, env={"TT_SMALL_T2": "1"})
    check(lockstep_gemm, str(tmp_path), 2, 35, 37, 323, ta, tb, dt, "f32", False, 99, ksplit=3)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_small_kernel_with_wide_offsets_values(lockstep_gemm, tmp_path, dt, ta, tb):
    # lane offsets of 64 bits (row pitches of 2^24 elements and more), on operands small enough to check: whole chunks of
    # every wave split, tails, K below a chunk
    for i, (M, N, K) in enumerate([(33, 47, 1051), (40, 31, 263), (65, 35, 131), (35, 33, 23), (1, 1, 1)]):
        check(lockstep_gemm, str(tmp_path), 1, M, N, K, ta, tb, dt, "f32", bool(i & 1), 150 + i, env={"TT_SMALL_PITCH": "1", "TT_PLAIN_K": "0"})


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("plain_k", ["0", "100000"])
def test_short_products_on_either_kernel_values(lockstep_gemm, tmp_path, dt, ta, tb, plain_k):
    # K below, at and past a step of the plain kernel (16) and a chunk of the small one; a round of four steps and more
    for i, (M, N, K) in enumerate([(65, 37, 17), (33, 67, 31), (1, 1, 1), (63, 129, 65), (35, 33, 16)]):
        check(lockstep_gemm, str(tmp_path), 1, M, N, K, ta, tb, dt, dt, bool(i & 1), 130 + i, env={"TT_PLAIN_K": plain_k})
    check(lockstep_gemm, str(tmp_path), 2, 35, 37, 323, ta, tb, dt, "f32", False, 139, ksplit=3, env={"TT_PLAIN_K": plain_k})


@pytest.mark.parametrize("out_dt,relu", [("bf16", True), ("f32", False)])
def test_forward_tiles_of_both_sizes_store_the_same_bits(lockstep_gemm, tmp_path, out_dt, relu):
    # both add in the order of increasing K: ragged tiles, K below, at and past a step of 16 and a round of four steps
    for i, (M, N, K) in enumerate([(65, 130, 65), (64, 64, 16), (33, 1, 1), (37, 67, 129), (63, 127, 50)]):
        stored = []
        for t64 in ("1000", "1"):
            check(lockstep_gemm, str(tmp_path), 1, M, N, K, 0, 0, "bf16", out_dt, relu, 120 + i, env={"TT_FWD_T64": t64})
            stored.append(open(os.path.join(str(tmp_path), "c0.bin"), "rb").read())
        assert stored[0] == stored[1], (M, N, K)


@pytest.mark.parametrize("ta,tb", LAYOUTS)
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("t64", ["1000", "1"])
def test_ordered_kernel_values(lockstep_gemm, tmp_path, dt, ta, tb, t64):
    # 32 x 32 and 64 x 64 tiles: a single row, column or value of K (operands without a pair along the side they are stored
    # by), the last of an odd side, K at and past a step of 64 and a round of four
    for i, (M, N, K) in enumerate([(1, 33, 5), (34, 1, 7), (33, 35, 1), (1, 1, 9), (1, 37, 1), (65, 66, 64), (35, 33, 257)]):
        check(lockstep_gemm, str(tmp_path), 1, M, N, K, ta, tb, dt, dt, bool(i & 1), 170 + i, env={"TT_PLAIN_K": "100000", "TT_FWD_T64": t64})


def test_random_products_values(lockstep_gemm, tmp_path):
    # seeded random shapes, layouts, types and tuning switches (sizes mostly multiples of eight, some odd): whatever
    # engine the launch code picks or falls back to has to give the product
    rng = np.random.default_rng(2024)
    switches = [{}, {}, {"TT_GEMM_ENGINE": "4"}, {"TT_GEMM_ENGINE": "6"}, {"TT_GEMM_ENGINE": "3", "TT_GEMM_TILE": "5", "EMU_CUS": "8"},
                {"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": "8"}] + [{"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": str(t)} for t in range(6)]

    def dim(hi):
        v = int(rng.integers(8, hi))
        return v if rng.random() < 0.15 else max(8, v // 8 * 8)

    for case in range(14):
        M, N, K = dim(560), dim(560), dim(330)
        ta, tb = (int(v) for v in rng.integers(0, 2, 2))
        in_dt = "bf16" if rng.random() < 0.85 else "f32"
        out_dt = "bf16" if rng.integers(0, 2) else "f32"
        ksplit = int(rng.choice([1, 1, 1, 2]))
        if ksplit > 1 and ((K + 1) // 2 + 63) // 64 * 64 >= K:
            ksplit = 1                                       # the second chunk would be empty: the launch refuses that
        relu = bool(rng.integers(0, 2)) and ksplit == 1
        if ksplit > 1:
            out_dt = "f32"                                   # partial products are kept in fp32, as the execute calls ask
        env = switches[int(rng.integers(0, len(switches)))]
        try:
            check(lockstep_gemm, str(tmp_path), int(rng.integers(1, 3)), M, N, K, ta, tb, in_dt, out_dt, relu, 300 + case, ksplit=ksplit, env=env)
        except AssertionError as e:
            raise AssertionError((case, M, N, K, ta, tb, in_dt, out_dt, relu, ksplit, env, str(e)[:500]))


@pytest.mark.parametrize("env", [{"EMU_CUS": "16", "TT_GEMM_ENGINE": "3", "TT_GEMM_TILE": "5"}, {"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": "8"}, {}])
def test_the_model_of_late_loads_bites(lockstep_gemm, tmp_path, env):
    # global -> LDS loads land only when a wait count lets them (see emu_lockstep.h); if every wait let two more loads
    # stay in flight than the kernel asks for, the engines that load straight into LDS must not get away with it
    shape = (2, 520, 776, 192, 0, 1, "bf16", "f32", False, 42) if env else (1, 264, 392, 96, 0, 1, "bf16", "f32", False, 45)
    check(lockstep_gemm, str(tmp_path), *shape, env=env)
    with pytest.raises(AssertionError):
        check(lockstep_gemm, str(tmp_path), *shape, env=dict(env, EMU_VMCNT_SLACK="2"))


@pytest.mark.parametrize("env", [{"EMU_CUS": "16", "TT_GEMM_ENGINE": "3", "TT_GEMM_TILE": "5"}, {"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": "8"}, {}])
def test_results_do_not_depend_on_which_wave_runs_ahead(lockstep_gemm, tmp_path, env):
    # the emulation runs the threads of a workgroup in index order between synchronisation points; with the order
    # reversed the last wave reaches every barrier first, issues its loads first and writes its results first
    shape = (2, 520, 776, 192, 1, 0, "bf16", "bf16", True, 42) if env else (1, 264, 392, 96, 1, 0, "bf16", "bf16", True, 45)
    check(lockstep_gemm, str(tmp_path), *shape, env=dict(env, EMU_ORDER="reverse"))


@pytest.mark.parametrize("M,N,K,ta,tb,launcher", [
    (136, 264, 512, 0, 1, "launch_tail6<true, true, true, false>"), (136, 264, 520, 0, 1, "launch_tail6<true, true, true, true>"),
    (136, 264, 504, 0, 1, "launch_tail4<true, true, true, true>"), (136, 264, 1032, 0, 0, "launch_tail6<true, false, true, true>"),
    (136, 264, 1016, 0, 0, "launch_tail4<true, false, true, true>"), (136, 264, 2048, 1, 0, "launch_tail6<false, false, true, false>"),
    (136, 264, 2056, 1, 0, "launch_tail6<false, false, true, true>"), (136, 264, 2040, 1, 0, "launch_tail4<false, false, true, true>"),
    (65, 136, 384, 0, 1, "launch_rows_cfg<64, true, true>"), (128, 136, 392, 0, 0, "launch_rows_cfg<64, true, false>"),
    (64, 136, 384, 0, 1, "launch_mfma_cfg"), (65, 136, 376, 0, 1, "launch_mfma_cfg"),
    (33, 136, 2048, 0, 0, "launch_rows_cfg<64, true, false>"), (32, 136, 1024, 0, 0, "launch_rows_cfg<32, true, false>")])
def test_products_run_on_the_kernels_that_their_rules_name(lockstep_gemm, tmp_path, M, N, K, ta, tb, launcher):
    # either side of the lines in K and in rows, no switch set
    out = check(lockstep_gemm, str(tmp_path), 1, M, N, K, ta, tb, "bf16", "f32", False, 97)
    name, _, args = out.split("launched by ")[1].rpartition(" [")
    values = dict(a.split(" = ") for a in args.rstrip("]\n").split(", "))
    want_name, _, want = launcher.rstrip(">").partition("<")
    assert name.split("(")[-2].split(" ")[-1].split("::")[-1] == want_name
    order = ["A_KC", "B_KC", "STAGED", "TAIL"] if "tail" in want_name else ["BM", "A_KC", "B_KC"]
    assert not want or [values[n] for n in order] == want.split(", ")


@pytest.mark.parametrize("env,shape", [({}, (1, 100, 136, 520, 0, 1)), ({}, (1, 32, 136, 1032, 0, 0)), ({"TT_GEMM_ENGINE": "4"}, (1, 264, 264, 104, 1, 0)),
                                       ({"TT_GEMM_ENGINE": "6"}, (1, 264, 264, 296, 1, 0)), ({"TT_GEMM_ENGINE": "1", "TT_GEMM_TILE": "8"}, (1, 264, 264, 72, 0, 0))])
def test_a_wait_that_is_too_short_shows_in_the_values(lockstep_gemm, tmp_path, env, shape):
    # rings of two and three stages, K tails: wrong values, not a fault of the emulation
    check(lockstep_gemm, str(tmp_path), *shape, "bf16", "f32", False, 98, env=env)
    with pytest.raises(AssertionError) as e:
        check(lockstep_gemm, str(tmp_path), *shape, "bf16", "f32", False, 98, env=dict(env, EMU_VMCNT_SLACK="2"))
    assert str(e.value).startswith("(")


@pytest.mark.parametrize("row,total,nts", [(4096, 2 ** 30, 1), (4000, 8 * 256 * 4000, 1), (4000, 2 ** 24, 1), (4000, 2 ** 24 + 4000, 0), (2000, 2 ** 26, 0), (2048, 2 ** 26, 1)])
def test_rows_that_begin_inside_a_64_byte_piece_are_stored_for_the_caches_from_16_mb_on(lockstep_gemm, row, total, nts):
    # smaller results would push the operands of the launches behind them out
    assert int(subprocess.run([lockstep_gemm, "store", str(row), str(total)], capture_output=True, text=True, check=True).stdout) == nts


@pytest.mark.parametrize("M,N,K,blocks,shards,runs", [(512, 8192, 512, 1, 16, 4), (2048, 2048, 1024, 1, 8, 4), (2048, 8192, 2048, 1, 4, 1), (520, 8192, 2048, 1, 4, 2),
                                                      (384, 12288, 1024, 1, 8, 2), (520, 12288, 1024, 1, 4, 1), (264, 4096, 4096, 1, 4, 0), (256, 8192, 4096, 2, 4, 0)])
def test_shards_that_add_up_are_cut_into_the_runs_that_measured_fastest(lockstep_gemm, M, N, K, blocks, shards, runs):
    r = subprocess.run([lockstep_gemm, "runs"] + [str(v) for v in (M, N, K, blocks, shards)], capture_output=True, text=True, check=True)
    assert int(r.stdout) == runs
