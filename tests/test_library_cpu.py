"""CPU-side checks of the product library: exported symbols, host planner against the oracle's brute force and
Algorithm 1, geometry, and host-side argument errors.  No kernel is launched."""
import ctypes
import itertools
import os
import re

import numpy as np
import pytest

import paper_1805_04170_amd as tt
from oracle import cost as oc
from oracle import execute as ex
from oracle import tiling as tl
from synthetic import CONFIGS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def fc_layers(widths, relu=False):
    L = len(widths) - 1
    return [tt.layer("fc", "relu" if (relu and l < L - 1) else "none", widths[l], widths[l + 1]) for l in range(L)]


def test_every_declared_symbol_is_exported():
    header = open(os.path.join(ROOT, "include", "tensor_tiling.h")).read()
    declared = set(re.findall(r"\b(tt_[a-z0-9_]+)\s*\(", header))
    assert declared == set(tt.binding.EXPORTS)
    L = ctypes.CDLL(tt.binding.LIB_PATH)
    for name in declared:
        assert hasattr(L, name), name


def test_no_oracle_in_product():
    # the product never imports or calls the oracle
    for dirpath, _, files in os.walk(os.path.join(ROOT, "paper_1805_04170_amd")):
        for f in files:
            if f.endswith((".py", ".cpp", ".hip", ".h")):
                text = open(os.path.join(dirpath, f)).read()
                assert "oracle" not in text.lower(), (dirpath, f)


def test_shard_shape_matches_oracle_and_rejects_uneven():
    for t in tl.all_tilings(3):
        assert tt.tt_shard_shape(64, 1000, t) == tl.shard_shape(64, 1000, t)
    with pytest.raises(tt.TilingError) as e:
        tt.tt_shard_shape(10, 6, "RR")
    assert e.value.status == 2
    with pytest.raises(tt.TilingError) as e:
        tt.tt_shard_shape(8, 8, "RX")
    assert e.value.status == 1


@pytest.mark.parametrize("k", [1, 2])
def test_exact_plan_equals_bruteforce(k):
    rng = np.random.default_rng(100 + k)
    for trial in range(8):
        L = int(rng.integers(1, 3))
        b = int(rng.choice([4, 6, 8, 12, 16, 48]))
        widths = [int(v) for v in rng.choice([2, 4, 6, 8, 10, 12, 24, 32, 112], size=L + 1)]
        chain = oc.make_chain(b, widths)
        ref = oc.bruteforce(chain, k)
        if ref[0] == oc.INF:
            with pytest.raises(tt.TilingError):
                tt.tt_plan_chain(fc_layers(widths), b, k, tt.TT_PLAN_EXACT)
            continue
        p = tt.tt_plan_chain(fc_layers(widths), b, k, tt.TT_PLAN_EXACT)
        assert p.cost == ref[0], (b, widths)
        # the returned tiling is valid: the oracle prices it at the same cost
        assert oc.chain_cost(chain, k, p.x(), p.g(), p.w())[0] == p.cost
        assert p.cost == sum(p.delta(j) << j for j in range(k))          # Theorem 1


def test_exact_plan_three_cuts_single_layer():
    chain = oc.make_chain(16, [24, 40])
    ref = oc.bruteforce(chain, 3)
    p = tt.tt_plan_chain(fc_layers([24, 40]), 16, 3, tt.TT_PLAN_EXACT)
    assert p.cost == ref[0]


def test_exact_plan_with_pins():
    widths, b, k = [8, 24, 12], 16, 2
    chain = oc.make_chain(b, widths)
    for pins in [dict(pin_x0="RR", pin_g0="RR"), dict(pin_xL="RR", pin_gL="rr"), dict(pin_x0="Cr")]:
        p = tt.tt_plan_chain(fc_layers(widths), b, k, tt.TT_PLAN_EXACT, **pins)
        assert p.cost == oc.bruteforce(chain, k, **pins)[0]
        if "pin_x0" in pins:
            assert p.x()[0] == pins["pin_x0"]
        if "pin_gL" in pins:
            assert p.g()[-1] == pins["pin_gL"]


def test_tiny_config_plan_is_the_bruteforce_optimum():
    cfg = CONFIGS["tiny_mlp"]
    p = tt.tt_plan_chain(fc_layers(cfg.widths), cfg.batch, cfg.k, tt.TT_PLAN_EXACT)
    assert p.cost == oc.bruteforce(oc.make_chain(cfg.batch, list(cfg.widths)), cfg.k)[0] == 57984


@pytest.mark.parametrize("name", ["tiny_mlp", "alexnet_fc", "vgg16_fc"])
def test_recursive_plan_equals_algorithm1_oracle(name):
    cfg = CONFIGS[name]
    chain = oc.make_chain(cfg.batch, list(cfg.widths))
    ref = oc.recursive(chain, cfg.k)
    p = tt.tt_plan_chain(fc_layers(cfg.widths), cfg.batch, cfg.k, tt.TT_PLAN_RECURSIVE)
    assert p.cost == ref[0]
    assert (p.x(), p.g(), p.w()) == (ref[1], ref[2], ref[3])
    assert [p.delta(j) for j in range(cfg.k)] == ref[4]
    exact = tt.tt_plan_chain(fc_layers(cfg.widths), cfg.batch, cfg.k, tt.TT_PLAN_EXACT)
    assert exact.cost <= p.cost
    assert oc.chain_cost(chain, cfg.k, exact.x(), exact.g(), exact.w())[0] == exact.cost


def test_recursive_random_chains_and_pins():
    rng = np.random.default_rng(9)
    for _ in range(10):
        b = int(rng.choice([4, 8, 12, 16, 48])); widths = [int(v) for v in rng.choice([4, 8, 10, 12, 24, 32], size=3)]
        chain = oc.make_chain(b, widths)
        pins = dict(pin_x0="RR") if rng.random() < 0.5 else {}
        ref = oc.recursive(chain, 2, **pins)
        if ref[0] == oc.INF:
            continue
        p = tt.tt_plan_chain(fc_layers(widths), b, 2, tt.TT_PLAN_RECURSIVE, **pins)
        assert (p.cost, p.x(), p.g(), p.w()) == (ref[0], ref[1], ref[2], ref[3])


def test_plan_eval_equals_oracle_on_random_tilings():
    rng = np.random.default_rng(3)
    widths, b, k = [8, 16, 10], 12, 2
    chain = oc.make_chain(b, widths)
    ts = tl.all_tilings(k)
    for _ in range(300):
        x = [ts[i] for i in rng.integers(0, 9, 3)]; g = [ts[i] for i in rng.integers(0, 9, 3)]
        w = [ts[i] for i in rng.integers(0, 9, 2)]
        ref = oc.chain_cost(chain, k, x, g, w)
        if ref[0] == oc.INF:
            with pytest.raises(tt.TilingError) as e:
                tt.tt_plan_eval(fc_layers(widths), b, k, x, g, w)
            assert e.value.status == 2
        else:
            cost, delta, forms = tt.tt_plan_eval(fc_layers(widths), b, k, x, g, w)
            assert (cost, delta, forms) == (ref[0], ref[2], ref[1])


def test_conv_chain_plan():
    # areas carry the image / filter-tap multipliers (Sec. 4.5); 1x1 images reduce to FC
    conv = [tt.layer("conv", "none", 4, 8, H=1, W=1, R=1, S=1, pad=0), tt.layer("conv", "none", 8, 4, H=1, W=1, R=1, S=1, pad=0)]
    assert tt.tt_plan_chain(conv, 8, 2).cost == tt.tt_plan_chain(fc_layers([4, 8, 4]), 8, 2).cost
    big = [tt.layer("conv", "none", 4, 8, H=8, W=8, R=3, S=3, pad=1), tt.layer("conv", "none", 8, 4, H=8, W=8, R=3, S=3, pad=1)]
    p = tt.tt_plan_chain(big, 8, 1)
    ref = oc.bruteforce(oc.make_chain(8, [4, 8, 4], xmult=[64, 64, 64], wmult=[0, 9, 9]), 1)
    assert p.cost == ref[0] and p.w() == ["r", "r"] and p.x() == ["R"] * 3      # large images: data parallel wins


def conv_layer(c, k_, hw, rs, pad):
    return tt.layer("conv", "none", c, k_, H=hw, W=hw, R=rs, S=rs, pad=pad)


def test_mixed_chain_flatten_and_pooling_against_oracle():
    # conv (4 -> 8 channels, 8 x 8) | pool to 4 x 4 | conv (8 -> 6, 4 x 4) | flatten | fc (6*16 -> 10) | fc (10 -> 4)
    layers = [conv_layer(4, 8, 8, 3, 1), conv_layer(8, 6, 4, 3, 1), tt.layer("fc", "none", 96, 10), tt.layer("fc", "none", 10, 4)]
    # the same graph written out for the oracle: cuttable widths, area multipliers of x_0..x_L and of W_1..W_L
    # (x_1 is charged at the pooled size, x_2 at 16 pixels per channel, the first fc weight is 6 x 10 times 16 pixels)
    chain = oc.make_chain(8, [4, 8, 6, 10, 4], xmult=[64, 16, 16, 1, 1], wmult=[0, 9, 9, 16, 1])
    for k in (1, 2):
        p = tt.tt_plan_chain(layers, 8, k)
        cost, forms, delta = oc.chain_cost(chain, k, p.x(), p.g(), p.w())     # the oracle prices the planner's tiling
        assert cost == p.cost and delta == [p.delta(j) for j in range(k)]
        rec = tt.tt_plan_chain(layers, 8, k, tt.TT_PLAN_RECURSIVE)
        assert rec.cost == oc.recursive(chain, k)[0] and rec.cost >= p.cost
    # one cut: the planner's optimum is the oracle's exhaustive optimum over the whole mixed graph (9^... tilings)
    sub = layers[1:3]
    sub_chain = oc.make_chain(8, [8, 6, 10], xmult=[16, 16, 1], wmult=[0, 9, 16])
    for k in (1, 2):
        assert tt.tt_plan_chain(sub, 8, k).cost == oc.bruteforce(sub_chain, k)[0]
    # flatten + fc is the convolution whose filter covers the whole image
    as_conv = [conv_layer(8, 6, 4, 3, 1), conv_layer(6, 10, 4, 4, 0)]
    assert tt.tt_plan_chain(sub, 8, 2).cost == tt.tt_plan_chain(as_conv, 8, 2).cost


def alexnet_layers():
    # public AlexNet layer dimensions (single tower); stride and pooling appear as the smaller image the next layer reads
    return [conv_layer(3, 96, 227, 11, 0), conv_layer(96, 256, 27, 5, 2), conv_layer(256, 384, 13, 3, 1),
            conv_layer(384, 384, 13, 3, 1), conv_layer(384, 256, 13, 3, 1), tt.layer("fc", "none", 9216, 4096),
            tt.layer("fc", "none", 4096, 4096), tt.layer("fc", "none", 4096, 1000)]


def vgg16_layers():
    cfg = [(3, 64, 224), (64, 64, 224), (64, 128, 112), (128, 128, 112), (128, 256, 56), (256, 256, 56), (256, 256, 56),
           (256, 512, 28), (512, 512, 28), (512, 512, 28), (512, 512, 14), (512, 512, 14), (512, 512, 14)]
    return [conv_layer(c, k_, hw, 3, 1) for c, k_, hw in cfg] + [tt.layer("fc", "none", 25088, 4096),
                                                                 tt.layer("fc", "none", 4096, 4096), tt.layer("fc", "none", 4096, 1000)]


def pinned_cost(layers, b, k, x_letter, g_letter, w_letter):
    L = len(layers)
    return tt.tt_plan_eval(layers, b, k, [x_letter * k] * (L + 1), [g_letter * k] * (L + 1), [w_letter * k] * L)[0]


@pytest.mark.parametrize("net", [alexnet_layers, vgg16_layers])
def test_whole_network_plans_and_the_batch_size_crossover(net):
    layers, k = net(), 3
    costs = {}
    for b in (32, 256, 2048):
        p = tt.tt_plan_chain(layers, b, k)
        # a returned tiling re-prices to the returned cost, and Algorithm 1 can only be worse
        assert tt.tt_plan_eval(layers, b, k, p.x(), p.g(), p.w())[0] == p.cost
        assert tt.tt_plan_chain(layers, b, k, tt.TT_PLAN_RECURSIVE).cost >= p.cost
        data = pinned_cost(layers, b, k, "R", "R", "r")      # data parallelism: batch cut, weights replicated
        costs[b] = (p.cost, data)
        assert p.cost <= data
    # data parallelism moves weight gradients, not activations (Sec. 2.2): its cost hardly depends on the batch (it is not
    # exactly constant: Eq. 2 takes the cheapest form per product, and for small batches that is not always F1)
    assert costs[32][1] <= costs[256][1] <= costs[2048][1] <= 1.3 * costs[32][1]
    # the gain of the optimum over data parallelism shrinks as the batch grows (Sec. 6.1: larger batches favour
    # data parallelism) ...
    gain = {b: costs[b][1] / costs[b][0] for b in costs}
    assert gain[32] > gain[256] > gain[2048] >= 1.0
    # ... and the convolution layers, with their large images, are data parallel in the optimum already: every
    # activation and gradient among them is cut along the batch only, forward products run as F1 (Sec. 6.1: "with the
    # larger image size, data parallelism has better performance than model parallelism")
    p = tt.tt_plan_chain(layers, 256, k)
    n_conv = sum(1 for lay in layers if lay.kind == tt.TT_CONV2D)
    assert all(t == "RRR" for t in p.x()[:n_conv]) and all(t == "RRR" for t in p.g()[:n_conv])
    assert all(p.forms(l, tt.TT_OP_FWD) == "111" for l in range(1, n_conv + 1))
    # the fully-connected tail is not: its first weight matrix is cut, never replicated
    assert "r" not in p.w()[n_conv]


def test_planner_argument_errors():
    with pytest.raises(tt.TilingError) as e:
        tt.tt_plan_chain(fc_layers([8, 8]), 8, 7)
    assert e.value.status == 1
    with pytest.raises(tt.TilingError) as e:
        tt.tt_plan_chain([tt.layer("fc", "none", 8, 4), tt.layer("fc", "none", 5, 4)], 8, 1)
    assert e.value.status == 1
    with pytest.raises(tt.TilingError) as e:                    # flatten must be channels x pixels
        tt.tt_plan_chain([conv_layer(4, 8, 4, 3, 1), tt.layer("fc", "none", 8 * 16 + 1, 4)], 8, 1)
    assert e.value.status == 1
    with pytest.raises(tt.TilingError) as e:                    # an image cannot grow between layers
        tt.tt_plan_chain([conv_layer(4, 8, 4, 3, 1), conv_layer(8, 8, 8, 3, 1)], 8, 1)
    assert e.value.status == 1
    with pytest.raises(tt.TilingError) as e:                    # convolution after fully-connected
        tt.tt_plan_chain([tt.layer("fc", "none", 8, 16), conv_layer(16, 8, 1, 1, 0)], 8, 1)
    assert e.value.status == 3
    with pytest.raises(tt.TilingError) as e:
        tt.tt_plan_chain(fc_layers([8, 8]), 8, 5, tt.TT_PLAN_EXACT)
    assert e.value.status == 3
    with pytest.raises(tt.TilingError) as e:
        tt.tt_plan_chain(fc_layers([3, 5]), 7, 1)       # nothing can be cut evenly
    assert e.value.status == 2


def test_host_side_errors_of_device_calls_need_no_gpu():
    # detected before any launch: bad letters, uneven cuts, bad element size, NULL shards
    import ctypes as C
    L = tt.binding.lib()
    null = (C.c_void_p * 4)(0, 0, 0, 0)
    one = (C.c_void_p * 4)(256, 256, 256, 256)
    assert L.tt_retile(one, tt.tiling("RR"), one, tt.tiling("CC"), 2, 6, 8, 2, None) == 2      # 6 rows cut twice
    assert L.tt_retile(one, tt.tiling("RR"), one, tt.tiling("CC"), 2, 8, 8, 3, None) == 1      # element size
    assert L.tt_retile(null, tt.tiling("RR"), one, tt.tiling("CC"), 2, 8, 8, 2, None) == 1     # NULL shard
    assert L.tt_retile(one, tt.tiling("RX"), one, tt.tiling("CC"), 2, 8, 8, 2, None) == 1      # bad letter
    assert L.tt_retile(one, tt.tiling("RR"), one, tt.tiling("CC"), 2, 0, 8, 2, None) == 0      # empty tensor: no-op
    lay = tt.layer("fc", "none", 10, 6)
    f = tt.forms("22")
    assert L.tt_fc_forward(C.byref(lay), 8, 2, tt.TT_BF16, tt.tiling("RR"), tt.tiling("rr"), tt.tiling("RR"), f,
                           one, one, one, None, 0, None) == 2                                # 6 columns, two N-splits
    conv = tt.layer("conv", "none", 8, 8, H=4, W=4, R=3, S=3, pad=1)
    assert L.tt_fc_forward(C.byref(conv), 8, 2, tt.TT_BF16, tt.tiling("RR"), tt.tiling("rr"), tt.tiling("RR"), None,
                           one, one, one, None, 0, None) == 1                                # wrong layer kind


def test_workspace_query_runs_on_host():
    lay = tt.layer("fc", "relu", 64, 32)
    assert tt.tt_fc_workspace_bytes(lay, 16, 2, "bf16", tt.TT_OP_FWD, "RR", "rr", "RR", forms_a="11") == 0
    n = tt.tt_fc_workspace_bytes(lay, 16, 2, "bf16", tt.TT_OP_FWD, "CC", "RR", "RR", forms_a="33")
    assert n == 4 * 16 * 32 * 4                               # four fp32 partial blocks
    assert tt.tt_fc_workspace_bytes(lay, 16, 2, "bf16", tt.TT_OP_DGRAD, "CC", "RR", "RR", "rr", "CC") > 0


# ---- counted cross-shard elements (what an execution moves) against explicit index sets

def _sets(rows, cols, t, s):
    rs, cs = tl.shard_slices(rows, cols, t, s)
    return {(i, j) for i in range(rs.start, rs.stop) for j in range(cs.start, cs.stop)}


def _moved_conversion(rows, cols, frm, to):
    k = len(frm)
    return sum(len(_sets(rows, cols, to, s) - _sets(rows, cols, frm, s)) for s in range(1 << k))


def _moved_reduction(rows, cols, form_seq, to):
    """every device fetches, for every element it is to store, the partial sums that other devices computed (two
    devices never hold the same value of an output element: an R or C cut puts them on different blocks, a form-3 cut
    gives them different partial sums)"""
    k = len(form_seq)
    grid = ex.output_grid_tiling(form_seq)           # where each device's partial sums lie
    made = [_sets(rows, cols, grid, q) for q in range(1 << k)]
    moved = 0
    for s in range(1 << k):
        for e in _sets(rows, cols, to, s):
            moved += sum(1 for q in range(1 << k) if q != s and e in made[q])
    return moved


def test_counted_conversion_elements_are_ghost_minus_held():
    rng = np.random.default_rng(21)
    for k in (1, 2, 3):
        ts = tl.all_tilings(k)
        for _ in range(40):
            a, b = ts[rng.integers(len(ts))], ts[rng.integers(len(ts))]
            rows, cols = 8 * int(rng.integers(1, 3)), 8 * int(rng.integers(1, 4))
            assert tt.tt_conversion_cross_elems(rows, cols, a, b) == _moved_conversion(rows, cols, a, b), (a, b)
    assert tt.tt_conversion_cross_elems(8, 8, "", "", 0) == 0
    with pytest.raises(tt.TilingError) as e:
        tt.tt_conversion_cross_elems(6, 8, "RR", "CC")
    assert e.value.status == 2


def test_counted_product_elements_against_index_sets_and_the_one_cut_cost():
    rng = np.random.default_rng(22)
    M, K, N = 8, 16, 8
    # one cut: the count is Eq. 2's term, for every stored tiling and every form
    for tx, ty, tz in itertools.product("RCr", repeat=3):
        for f in "123":
            got = sum(tt.tt_product_cross_elems(M, K, N, tx, ty, tz, f))
            assert got == oc.eq2_term(int(f) - 1, tx, ty, tz, M * K, K * N, M * N)
    # several cuts: explicit sets
    for k in (2, 3):
        ts = tl.all_tilings(k)
        for _ in range(25):
            tx, ty, tz = (ts[rng.integers(len(ts))] for _ in range(3))
            f = "".join(rng.choice(list("123")) for _ in range(k))
            if not ex.forms_feasible(f, M, K, N):
                continue
            aX, aY = ex.aligned_tilings(f)
            want_out = _moved_reduction(M, N, f, tz) if "3" in f else _moved_conversion(M, N, ex.output_grid_tiling(f), tz)
            got = tt.tt_product_cross_elems(M, K, N, tx, ty, tz, f)
            assert got == [_moved_conversion(M, K, tx, aX), _moved_conversion(K, N, ty, aY), want_out], (tx, ty, tz, f)
    assert tt.tt_product_cross_elems(8, 8, 8, "R", "r", "R", "1", mult=(3, 5, 7)) == [0, 0, 0]
    assert tt.tt_product_cross_elems(8, 8, 8, "C", "C", "r", "1", mult=(3, 5, 7)) == [3 * 32, 5 * 64, 7 * 64]


def test_counted_elements_of_a_whole_step_equal_the_plan_cost_at_one_cut():
    batch, widths = 16, [24, 16, 8]
    layers = fc_layers(widths)
    p = tt.tt_plan_chain(layers, batch, 1)
    forms = [[p.forms(l, op) for op in range(3)] for l in range(1, 3)]
    assert tt.tt_fc_chain_cross_elems(layers, batch, 1, p.x(), p.g(), p.w(), forms) == p.cost
    # data parallelism at one cut: both weight gradients are all-reduced, nothing else moves
    x = g = ["R"] * 3
    w = ["r"] * 2
    cost, _, f = tt.tt_plan_eval(layers, batch, 1, x, g, w)
    assert tt.tt_fc_chain_cross_elems(layers, batch, 1, x, g, w, f) == cost == 2 * (24 * 16 + 16 * 8)
    # more cuts: the recursive model and the flat count part ways (two row cuts of a large batch, weights replicated:
    # the model charges 2|W| (2^k - 1), every one of the four devices really fetches three foreign partial sums of |W|)
    k, big = 2, 256
    x = g = ["RR"] * 3
    w = ["rr"] * 2
    cost, _, f = tt.tt_plan_eval(layers, big, k, x, g, w)
    counted = tt.tt_fc_chain_cross_elems(layers, big, k, x, g, w, f)
    assert cost == 2 * (24 * 16 + 16 * 8) * 3 and counted == 4 * 3 * (24 * 16 + 16 * 8)


@pytest.mark.parametrize("net", [alexnet_layers, vgg16_layers])
def test_whole_network_strategies_rank_as_in_the_paper(net):
    # Sec. 2.2 / Sec. 6: data parallelism, model parallelism, the hand-made hybrid (convolutions data parallel,
    # fully-connected layers model parallel) and the searched tiling, priced by the same cost model at three cuts
    layers, k = net(), 3
    L = len(layers)
    fc = [l.kind == tt.TT_FC for l in layers]
    first_fc = fc.index(True)
    for b in (32, 256, 2048):
        dp = tt.tt_plan_eval(layers, b, k, ["R" * k] * (L + 1), ["R" * k] * (L + 1), ["r" * k] * L)[0]
        mp = tt.tt_plan_eval(layers, b, k, ["r" * k] * (L + 1), ["r" * k] * (L + 1), ["C" * k] * L)[0]
        act = ["R" * k if l <= first_fc else "r" * k for l in range(L + 1)]
        hybrid = tt.tt_plan_eval(layers, b, k, act, act, ["C" * k if fc[l] else "r" * k for l in range(L)])[0]
        best = tt.tt_plan_chain(layers, b, k).cost
        assert best < hybrid < min(dp, mp)
        # model parallelism moves activations: it grows with the batch, data parallelism hardly does
        if b > 32:
            assert mp > dp


def test_counted_traffic_argument_errors():
    def status(fn):
        with pytest.raises(tt.TilingError) as e:
            fn()
        return e.value.status

    assert status(lambda: tt.tt_conversion_cross_elems(0, 8, "R", "C")) == 1
    assert status(lambda: tt.tt_conversion_cross_elems(8, 8, "RRRRRRR", "CCCCCCC")) == 1           # more than six cuts
    assert status(lambda: tt.tt_product_cross_elems(8, 8, 8, "R", "r", "R", "4")) == 1              # no such form
    assert status(lambda: tt.tt_product_cross_elems(6, 8, 8, "RR", "rr", "RR", "11")) == 2          # M = 6 cannot be halved twice
    assert status(lambda: tt.tt_product_cross_elems(8, 8, 8, "R", "r", "R", "1", k=7)) == 1
    conv = [conv_layer(4, 8, 8, 3, 1)]
    assert status(lambda: tt.tt_fc_chain_cross_elems(conv, 8, 1, ["R"] * 2, ["R"] * 2, ["r"], [["1", "1", "3"]])) == 3
    two = fc_layers([8, 6, 4])
    bad = [tt.layer("fc", "none", 8, 6), tt.layer("fc", "none", 5, 4)]                                # widths do not chain
    assert status(lambda: tt.tt_fc_chain_cross_elems(bad, 8, 1, ["R"] * 3, ["R"] * 3, ["r"] * 2, [["1", "1", "3"]] * 2)) == 1
    assert tt.tt_fc_chain_cross_elems(two, 8, 0, [""] * 3, [""] * 3, [""] * 2, [["", "", ""]] * 2) == 0   # one device: nothing moves


def test_the_product_build_reads_no_environment():
    # launch decisions are functions of the call's arguments alone: the library as built for use imports no getenv
    # (tuning overrides exist only in builds with -DTT_TUNING, which the tests' host builds are)
    import shutil
    import subprocess
    nm = shutil.which("nm")
    if nm is None or not os.path.exists(tt.binding.LIB_PATH):
        pytest.skip("no nm, or the library is not built")
    syms = subprocess.run([nm, "-D", "--undefined-only", tt.binding.LIB_PATH], capture_output=True, text=True).stdout
    assert "getenv" not in syms


def test_layer_calls_take_what_the_binding_documents(monkeypatch):
    # nothing is launched: every call is refused, or fails before it reaches the library
    import torch
    monkeypatch.setattr(tt.binding, "_stream", lambda stream: 0)
    lay, x = tt.layer("fc", "none", 8, 8), [torch.zeros(8) for _ in range(2)]

    def fwd(*, X=x, Y=x, batch=5, dtype="bf16", tX="R", f="1"):
        tt.tt_fc_forward(lay, batch, 1, dtype, tX, "r", "R", f, X, x, Y)

    for ok in (dict(), dict(X=tuple(x)), dict(X=iter(x)), dict(X=[1 << 20, 2 << 20]), dict(X=[x[0], 1 << 20]), dict(dtype=tt.TT_F32),
               dict(tX=tt.tiling("R")), dict(f=tt.binding.forms("1")), dict(f=None)):
        with pytest.raises(tt.TilingError) as e:      # a batch of five under one row cut
            fwd(**ok)
        assert e.value.status == 2, ok
    for bad, status in ((dict(X=None), 1), (dict(X=x[:1]), 1), (dict(tX="X"), 1), (dict(tX="RRRRRRR"), 1), (dict(f="4"), 2), (dict(f=""), 2)):
        with pytest.raises(tt.TilingError) as e:
            fwd(**bad)
        assert e.value.status == status, bad
    for bad, error in ((dict(dtype="bf17"), KeyError), (dict(X=[None, 1]), TypeError), (dict(X=5), TypeError), (dict(batch=4.5), TypeError),
                       (dict(f="a"), ValueError)):
        with pytest.raises(error):
            fwd(**bad)


def test_form_sequences_shorter_than_the_cuts_are_refused(monkeypatch):
    # nothing past the end of what was given is read, whatever it was given as (nothing is launched: every call is refused)
    import torch
    monkeypatch.setattr(tt.binding, "_stream", lambda stream: 0)
    lay, x = tt.layer("fc", "none", 8, 8), [torch.zeros(8) for _ in range(4)]
    t = ("RR", "rr", "RR")
    for short in ("1", "", [1], (1,), [], b"", [1, 9]):
        for call in (lambda: tt.tt_fc_forward(lay, 8, 2, "bf16", *t, short, x, x, x),
                     lambda: tt.tt_fc_forward_static(lay, 8, 2, "bf16", *t, short, x, x, x),
                     lambda: tt.tt_fc_backward(lay, 8, 2, "bf16", *t, "RR", "RR", short, "11", x, x, x, x, x, x),
                     lambda: tt.tt_fc_backward(lay, 8, 2, "bf16", *t, "RR", "RR", "11", short, x, x, x, x, None, x),
                     lambda: tt.tt_fc_backward_overlapped(lay, 8, 2, "bf16", *t, "RR", "RR", short, "11", x, x, x, x, x, x),
                     lambda: tt.tt_fc_workspace_bytes(lay, 8, 2, "bf16", tt.TT_OP_FWD, *t, forms_a=short),
                     lambda: tt.tt_product_cross_elems(8, 8, 8, *t, short, k=2),
                     lambda: tt.tt_fc_chain_cross_elems([lay], 8, 2, ["RR", "RR"], ["RR", "RR"], ["rr"], [["11", "11", short]]),
                     lambda: tt.tt_reduce(x, "rr", "f32", x, short, 8, 8, k=2)):
            with pytest.raises(tt.TilingError) as e:
                call()
            assert e.value.status in (1, 2), short
    assert tt.tt_product_cross_elems(8, 8, 8, *t, "11") == tt.tt_product_cross_elems(8, 8, 8, *t, [1, 1])


def test_the_library_is_built_before_the_binding_s_module(monkeypatch):
    # the C library knows nothing of Python: where the extension module cannot be compiled (no headers), it is still linked
    import subprocess as sp
    from paper_1805_04170_amd import build as b
    ran = []

    def check_call(cmd, *a, **kw):
        ran.append(cmd)
        if any("calls.cpp" in str(x) for x in cmd):
            raise sp.CalledProcessError(1, cmd)

    monkeypatch.setattr(b, "_compile", lambda src: src + ".o")
    monkeypatch.setattr(b.subprocess, "check_call", check_call)
    with pytest.raises(sp.CalledProcessError):
        b.build()
    assert any("-shared" in c and b.LIB in c for c in ran)


def test_shard_lists_shorter_than_the_shards_are_refused(monkeypatch):
    # entries that were not given are NULL addresses, in every call (nothing is launched: every call is refused)
    import torch
    monkeypatch.setattr(tt.binding, "_stream", lambda stream: 0)
    lay, x = tt.layer("fc", "none", 8, 8), [torch.zeros(64) for _ in range(4)]
    few = x[:1]
    for call in (lambda: tt.tt_shard_gemm(few, x, x, 8, 8, 8), lambda: tt.tt_shard_gemm(x, few, x, 8, 8, 8), lambda: tt.tt_reduce(x, "rr", "f32", few, "33", 8, 8),
                 lambda: tt.tt_reduce(few, "rr", "f32", x, "33", 8, 8), lambda: tt.tt_retile_gate(x, "RR", few, "RR", x, "RR", 8, 8, "f32"),
                 lambda: tt.tt_retile_gate(x, "RR", x, "CC", few, "RR", 8, 8, "f32"), lambda: tt.tt_retile_gate(few, "RR", x, "CC", x, "RR", 8, 8, "f32"),
                 lambda: tt.tt_fc_backward_overlapped(lay, 8, 2, "bf16", "RR", "rr", "RR", "RR", "RR", "11", "33", x, few, x, x, x, x),
                 lambda: tt.tt_fc_backward(lay, 8, 2, "bf16", "RR", "rr", "RR", "RR", "RR", "11", "33", x, few, x, x, x, x)):
        with pytest.raises(tt.TilingError) as e:
            call()
        assert e.value.status == 1
    assert list(tt.binding.ptrs(few)[1:]) == [None] * 63 and tt.binding.ptrs(None) is None
