"""GPU kernels and dispatch branches at the sizes where they can go wrong:
edges of tiles, remainders, the smallest and largest of a range.  Whole
layers at the usual sizes are in test_gpu_parity.py."""
import numpy as np
import pytest

import oracle
from parity import GAP_TOL, compare_out, compare_routing, near_tie_tokens
from test_gpu_parity import _layer_in_batches, dev, host, small_layer

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sw():
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2609_34117_amd import slimwise

    return slimwise


# --------------------------------------------------------------------------
# routing mass: waves without a token, uneven token runs, every experts-a-lane
# count, experts past the last full lane, the block cap set by the workspace
# (few pairs: m 1000, k 1), fewer eligible experts than k

@pytest.mark.parametrize("hidden,m,k,tokens,eligible", [
    (64, 64, 8, 1, 64),
    (128, 65, 3, 33, 65),
    (256, 128, 32, 130, 40),
    (256, 300, 4, 97, 300),
    (256, 1000, 1, 1300, 1000),
    (512, 256, 8, 4097, 256),
    (256, 96, 8, 50, 5),
])
def test_routing_mass_edges(sw, hidden, m, k, tokens, eligible):
    cfg, L, D = small_layer(hidden, m, k, 32, tokens, seed=31)
    mask = None
    if eligible < m:
        mask = np.zeros(m, np.uint8)
        mask[np.random.default_rng(5).permutation(m)[:eligible]] = 1
    start = np.linspace(0.5, 2.0, m).astype(np.float32)
    mass = (dev(start), dev(start))
    sw.sw_moe_routing_mass(D["x"], D["wr"], k, keep_mask=None if mask is None else dev(mask),
                           mass=mass)
    ms, mt = host(mass[0]) - start, host(mass[1]) - start
    z = oracle.route(L["x"], L["wr"], min(k, eligible), keep_mask=mask, want_logits=True)[3]
    z = z.astype(np.float64)
    if mask is not None:
        z[:, mask == 0] = -np.inf
    p = np.exp(z - z.max(1, keepdims=True))
    o_ms = (p / p.sum(1, keepdims=True)).sum(0)
    # a logit off by GAP_TOL moves a share by twice that; the sums round at
    # 2^-24 of the running mass, here and in `start` + mass
    tol = 2 * GAP_TOL * o_ms + 2.0 ** -22 * (o_ms + 2.0)
    assert np.all(np.abs(ms - o_ms) <= tol)
    if eligible < k:
        assert np.array_equal(host(mass[1]), start)
        return
    o_mt = np.zeros(m)
    order = np.argsort(-z, axis=1, kind="stable")[:, :k]
    w = np.exp(np.take_along_axis(z, order, 1) - z.max(1, keepdims=True))
    np.add.at(o_mt, order, w / w.sum(1, keepdims=True))
    n_near = int(near_tie_tokens(z, mask, k).sum())
    assert np.all(np.abs(mt - o_mt) <= 2 * GAP_TOL * o_mt + 2.0 ** -22 * (o_mt + 2.0) + n_near)


# one array for both masses takes the sum of what two would

def test_routing_mass_into_one_array(sw):
    cfg, L, D = small_layer(256, 96, 4, 32, 200, seed=33)
    two = sw.sw_moe_routing_mass(D["x"], D["wr"], 4)
    one = torch.zeros(96, device="cuda")
    for _ in range(3):
        one.zero_()
        sw.sw_moe_routing_mass(D["x"], D["wr"], 4, mass=(one, one))
        assert torch.equal(one, two[0] + two[1])


# --------------------------------------------------------------------------
# selection and plan: one wave a token and one plan wave up to 16 tokens and 64
# pairs; a row of 16 lanes a token and one plan block past either edge, up to 32
# tokens over 64 experts; else the separate kernels; 1 to 16 experts a lane,
# pools that end inside a wave or a row, masks and biases

def plan_of(ids, m):
    """(counts, offsets, perm, active) of the pairs' ids, by a stable sort."""
    flat = np.asarray(ids).reshape(-1)
    counts = np.bincount(flat, minlength=m)
    return (counts, np.concatenate([[0], np.cumsum(counts)]), np.argsort(flat, kind="stable"),
            np.nonzero(counts)[0])


def check_plan(plan, ids, m):
    counts, offsets, perm, active = plan_of(ids, m)
    assert int(plan.n_active.item()) == len(active)
    assert np.array_equal(host(plan.counts), counts)
    assert np.array_equal(host(plan.offsets), offsets)
    assert np.array_equal(host(plan.perm)[: len(perm)], perm)
    assert np.array_equal(host(plan.active)[: len(active)], active)


@pytest.mark.parametrize("m,k,tokens,masked,biased", [
    (256, 4, 16, True, True),     # 64 pairs on 16 waves
    (256, 8, 8, False, False),    # 64 pairs on 8
    (256, 16, 4, True, False),    # 64 pairs on 4
    (16, 16, 1, False, False),    # k = m: an infinite gap
    (65, 3, 16, False, True),     # the pool ends inside the second expert a lane
    (256, 8, 9, True, True),      # 72 pairs
    (128, 1, 17, False, False),   # 17 tokens
    (257, 8, 2, False, True),     # past the fused pool
    (1000, 2, 5, True, True),     # 16 experts a lane
    (16, 1, 17, False, True),     # rows: one expert a lane, 17 tokens
    (17, 16, 5, True, False),     # two experts a lane, 80 pairs
    (33, 4, 32, True, True),      # four
    (64, 16, 32, False, False),   # the largest: 512 pairs
    (65, 4, 32, False, True),     # past the row pool
    (64, 4, 33, True, False),     # past the row tokens
])
def test_selection_and_plan_edges(sw, m, k, tokens, masked, biased):
    cfg, L, D = small_layer(512, m, k, 32, tokens, seed=41)
    rng = np.random.default_rng([41, m, k])
    mask = None
    if masked:
        mask = np.zeros(m, np.uint8)
        mask[rng.permutation(m)[: max(k, m // 2)]] = 1
    bias = (0.5 * rng.standard_normal(m)).astype(np.float32) if biased else None
    ids, w, gap, plan = sw.sw_moe_route_dispatch(
        D["x"], D["wr"], k, keep_mask=None if mask is None else dev(mask),
        bias=None if bias is None else dev(bias))
    o_ids, o_w, o_gap, o_z = oracle.route(L["x"], L["wr"], k, keep_mask=mask, bias=bias,
                                          want_logits=True)
    compare_routing(host(ids), host(w), o_ids, o_w, o_z, mask, k, g_gap=host(gap), o_gap=o_gap)
    check_plan(plan, host(ids), m)


# the row form against route, then dispatch, bit for bit: ties, a NaN and
# infinite logits, fewer eligible experts than k; and, with a shared expert, against
# batches of 3 tokens, which take the wave form

@pytest.mark.parametrize("m,k,tokens", [(16, 8, 32), (50, 16, 17), (64, 2, 32)])
def test_row_selection_equals_separate_kernels(sw, m, k, tokens):
    cfg, L, D = small_layer(512, m, k, 32, tokens, seed=43)
    bias = np.zeros(m, np.float32)
    bias[1], bias[3], bias[5] = np.inf, -np.inf, np.nan
    D["wr"][7] = D["wr"][9]  # equal logits
    few = np.zeros(m, np.uint8)
    few[: k - 1] = 1
    for b, mask in ((None, None), (dev(bias), None), (None, dev(few))):
        ids, w, gap, plan = sw.sw_moe_route_dispatch(D["x"], D["wr"], k, keep_mask=mask, bias=b)
        r_ids, r_w, r_gap = sw.sw_moe_route(D["x"], D["wr"], k, keep_mask=mask, bias=b)
        r_plan = sw.sw_moe_dispatch(r_ids, m)
        assert torch.equal(ids, r_ids)
        for a, r in ((w, r_w), (gap, r_gap)):
            assert torch.equal(a.view(torch.int32), r.view(torch.int32))
        n = int(r_plan.n_active.item())
        assert int(plan.n_active.item()) == n and (n < 0) == (mask is not None)
        for name in ("counts", "offsets", "perm"):
            assert torch.equal(getattr(plan, name), getattr(r_plan, name))
        assert torch.equal(plan.active[: max(n, 0)], r_plan.active[: max(n, 0)])


@pytest.mark.parametrize("m,k,n_shared,groups,tokens", [(60, 4, 2, 2, 32), (16, 14, 2, 1, 17)])
def test_row_selection_with_shared_expert(sw, m, k, n_shared, groups, tokens):
    cfg, L, D = small_layer(512, m + 1, k, 32, tokens, seed=44)  # the last router row: its gate
    ids, w, gap, plan = sw.sw_moe_route_dispatch_shared(D["x"], D["wr"], k, n_shared,
                                                        n_groups=groups)
    pool = m + groups * n_shared
    for t0 in range(0, tokens, 3):
        part = sw.sw_moe_route_dispatch_shared(D["x"][t0:t0 + 3].contiguous(), D["wr"], k, n_shared)
        assert torch.equal(ids[t0:t0 + 3, :k], part[0][:, :k])
        assert torch.equal(w[t0:t0 + 3], part[1]) and torch.equal(gap[t0:t0 + 3], part[2])
    g = np.arange(tokens) * groups // tokens
    assert np.array_equal(host(ids)[:, k:], m + g[:, None] * n_shared + np.arange(n_shared))
    check_plan(plan, host(ids), pool)


# the one-block plan: one pair, part of a run, both block sizes at their largest
# pools and pair counts, every pair on one expert, then the first size past it;
# an id out of range on the last pair

@pytest.mark.parametrize("m,pairs,spread", [
    (1, 1, 1), (7, 63, 7), (512, 1024, 512), (513, 1024, 513), (512, 1025, 3), (1024, 2048, 1024),
    (300, 2047, 1), (300, 2049, 300),
])
def test_dispatch_plan_edges(sw, m, pairs, spread):
    rng = np.random.default_rng([43, m, pairs])
    ids = (rng.integers(0, spread, (pairs, 1)) + (m - spread)).astype(np.int32)
    check_plan(sw.sw_moe_dispatch(dev(ids), m), ids, m)
    for bad in (m, -1):
        ids[-1] = bad
        plan = sw.sw_moe_dispatch(dev(ids), m)
        assert int(plan.n_active.item()) == -1
        assert not host(plan.counts).any() and not host(plan.offsets).any()
        assert np.array_equal(host(plan.perm), np.arange(pairs))


# --------------------------------------------------------------------------
# prefill-sized router logits: token tiles and expert tiles that end inside a
# block, experts that are not a multiple of four (scalar stores), one to three
# slices of H, a slice of two chunks and one that ends in the middle of the ring;
# one expert, whose row the loads past the end of the slice must not leave

@pytest.mark.parametrize("hidden,m,tokens,k", [
    (128, 1000, 261, 4), (256, 129, 1900, 4), (1152, 64, 4100, 4), (3072, 250, 1025, 4),
    (128, 1, 16400, 1), (384, 2, 16400, 2),
])
def test_wide_logits_edges(sw, hidden, m, tokens, k):
    cfg, L, D = small_layer(hidden, m, k, 32, tokens, seed=47)
    ids, w, gap = sw.sw_moe_route(D["x"], D["wr"], k)
    o_ids, o_w, o_gap, o_z = oracle.route(L["x"], L["wr"], k, want_logits=True)
    compare_routing(host(ids), host(w), o_ids, o_w, o_z, None, k, g_gap=host(gap), o_gap=o_gap)


# --------------------------------------------------------------------------
# the prefill kernels: K of one round of the rings, the last that is too short
# to look up the next pass (H 384), the first that does (H 512), longer ones;
# row tiles that end inside a unit (H 128, 384; I 128, 384); more units than
# blocks (300 experts), experts of several passes, from 1 to 10 column blocks;
# units that start inside the row (H 2048, row-major); tiled rows past the ring
# of the down projection (I 640, 768)

@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("hidden,inter,m,k,tokens", [
    (128, 128, 16, 1, 256), (384, 256, 16, 4, 700), (512, 128, 300, 8, 640),
    (512, 384, 16, 8, 330), (1152, 256, 24, 4, 450), (2048, 384, 16, 2, 300),
    (384, 640, 16, 8, 330), (1152, 768, 24, 4, 700),
])
def test_prefill_kernel_edges(sw, hidden, inter, m, k, tokens, tiled):
    cfg, L, D = small_layer(hidden, m, k, inter, tokens, seed=53)
    bias = np.linspace(1.0, -1.0, m).astype(np.float32)  # graded loads
    layout = sw.ROW_MAJOR
    if tiled:
        D = dict(D)
        D["w13"], D["w2"] = sw.sw_moe_pack_experts(D["w13"], D["w2"])
        layout = sw.TILED
    d = sw.dims(hidden, inter, m, k)
    assert sw.sw_moe_forward_kernels(d, tokens, layout) == ("prefill", "prefill")
    g = sw.moe_layer(D["x"], D["wr"], D["w13"], D["w2"], k, bias=dev(bias), layout=layout)
    g_ids, g_w = host(g["topk_ids"]), host(g["topk_w"])
    compare_out(host(g["out"]), oracle.forward(L["x"], L["w13"], L["w2"], g_ids, g_w))
    # the wave kernels accumulate every output over K in the same order (the
    # split-K ones, which small batches of the deeper layers take, do not; row-major
    # rows of H 2048: test_prefill_order_of_sums)
    same_order = tiled or hidden % 2048 != 0
    if same_order and sw.sw_moe_forward_kernels(d, 16, layout) == ("wave", "wave"):
        small = _layer_in_batches(sw, D, k, 16, layout, bias=dev(bias))
        assert torch.equal(g["out"], small)


# --------------------------------------------------------------------------
# where the families' order of summation over K shows (sw_kernel_family): rows a
# multiple of 4 KiB apart make the row-major prefill gate/up start inside the row.
# h is rounded to two bf16 planes, 2^-17 of it at most, whatever the order; the sums
# before it differ by less (64 roundings of 2^-25 of about the sum, at random), so
# two orders give outputs within 2^-16 of each other in the 2-norm.  Everything
# else here, and all of it in the tiled layout, is the same bits.

def _rel(a, b):
    return float(torch.linalg.vector_norm((a - b).double()) / torch.linalg.vector_norm(b.double()))


@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("hidden", [1920, 2048])
def test_prefill_order_of_sums(sw, hidden, tiled):
    inter, m, k, tokens = 512, 96, 8, 96  # 768 pairs: 16 an expert of half the pool, 8 of all
    cfg, L, D = small_layer(hidden, m, k, inter, tokens, seed=61)
    g = sw.sw_moe_prune_compact(D["importance"], m // 2, k, w13=D["w13"], w2=D["w2"], wr=D["wr"])
    layout, pack = sw.ROW_MAJOR, lambda w13, w2: (w13, w2)
    if tiled:
        layout, pack = sw.TILED, sw.sw_moe_pack_experts
    full = dict(D, w13=pack(D["w13"], D["w2"])[0], w2=pack(D["w13"], D["w2"])[1])
    comp = dict(x=D["x"], wr=g["wr"], w13=pack(g["w13"], g["w2"])[0],
                w2=pack(g["w13"], g["w2"])[1])
    families = [sw.sw_moe_forward_kernels(sw.dims(hidden, inter, e, k), t, layout)
                for e, t in ((m, tokens), (m // 2, tokens), (m // 2, 32))]
    assert families == [("wave", "wave"), ("prefill", "prefill"), ("wave", "wave")]

    def layer(d, **kw):
        return sw.moe_layer(d["x"], d["wr"], d["w13"], d["w2"], k, layout=layout, **kw)

    whole = layer(comp)
    others = {
        "masked": layer(full, keep_mask=g["keep_mask"])["out"],
        "batches": _layer_in_batches(sw, comp, k, 32, layout),
        "layouts": sw.moe_layer(D["x"], g["wr"], *sw.sw_moe_pack_experts(g["w13"], g["w2"]), k,
                                layout=sw.TILED)["out"],
    }
    assert torch.equal(layer(comp)["out"], whole["out"])
    for name, out in others.items():
        if tiled or hidden % 2048 != 0:
            assert torch.equal(out, whole["out"]), name
        else:
            assert _rel(out, whole["out"]) <= 2.0 ** -16, name
    g_ids, g_w = host(whole["topk_ids"]), host(whole["topk_w"])
    compare_out(host(whole["out"]), oracle.forward(L["x"], host(g["w13"]), host(g["w2"]), g_ids, g_w))


@pytest.mark.parametrize("hidden", [1920, 2048])
def test_token_groups_across_families(sw, hidden):
    # 640 pairs: the pool of 24 experts and one copy of the shared expert's two
    # parts is prefill-sized (16 pairs an expert), with nine copies it is not
    inter, m, k, S, tokens = 512, 24, 8, 2, 64
    cfg, L, D = small_layer(hidden, m + 1 + S, k, inter, tokens, seed=67)
    wr = D["wr"][: m + 1].contiguous()
    out, families = [], []
    for groups in (1, 9):
        w13 = torch.cat([D["w13"][:m]] + [D["w13"][m + 1:]] * groups)
        w2 = torch.cat([D["w2"][:m]] + [D["w2"][m + 1:]] * groups)
        families.append(sw.sw_moe_forward_kernels(
            sw.dims(hidden, inter, m + groups * S, k + S), tokens, sw.ROW_MAJOR))
        out.append(sw.sw_moe_layer(D["x"], wr, k, w13, w2, n_shared=S, n_groups=groups)[4])
    assert families == [("prefill", "prefill"), ("wave", "wave")]
    if hidden % 2048 != 0:
        assert torch.equal(out[0], out[1])
    else:
        assert _rel(out[0], out[1]) <= 2.0 ** -16


# --------------------------------------------------------------------------
# row-major weights, read as operands (the wave kernels) or in runs of rows that
# are transposed into operands (the generic ones): a contraction that ends
# inside a group of four steps and inside a step, output rows that end inside a
# tile, several column blocks and passes; against the oracle, and (wave) the
# tiled layout's bits

@pytest.mark.parametrize("hidden,inter,m,k,tokens,family", [
    (32, 64, 8, 1, 5, "wave"), (160, 96, 8, 1, 30, "wave"), (288, 64, 64, 2, 300, "wave"),
    (2080, 1056, 32, 2, 40, "generic"), (2568, 1544, 16, 2, 70, "generic"),
    (4096, 1096, 32, 2, 100, "generic"), (2112, 1088, 16, 2, 70, "generic"),
])
def test_row_major_operand_edges(sw, hidden, inter, m, k, tokens, family):
    cfg, L, D = small_layer(hidden, m, k, inter, tokens, seed=59)
    fams = sw.sw_moe_forward_kernels(sw.dims(hidden, inter, m, k), tokens, sw.ROW_MAJOR)
    assert fams[0] == family
    g = sw.moe_layer(D["x"], D["wr"], D["w13"], D["w2"], k, layout=sw.ROW_MAJOR)
    g_ids, g_w = host(g["topk_ids"]), host(g["topk_w"])
    compare_out(host(g["out"]), oracle.forward(L["x"], L["w13"], L["w2"], g_ids, g_w))
    if family == "wave":
        w13, w2 = sw.sw_moe_pack_experts(D["w13"], D["w2"])
        t = sw.moe_layer(D["x"], D["wr"], w13, w2, k, layout=sw.TILED)
        assert torch.equal(g["out"], t["out"])
