"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on the
same seeded inputs.  Tolerances and the near-tie rule are in parity.py."""
import dataclasses
import functools

import numpy as np
import pytest

import oracle
from paper_2609_34117_amd import inputs as I
from guard import Guards
from parity import compare_out, compare_routing, oracle_forward_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sw():
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2609_34117_amd import slimwise

    return slimwise


def dev(a):
    a = np.ascontiguousarray(a)
    if a.dtype == np.uint16:
        a = a.view(np.int16)
    return torch.from_numpy(a).cuda()


def host(t):
    a = t.cpu().numpy()
    return a.view(np.uint16) if a.dtype == np.int16 else a


@functools.lru_cache(maxsize=2)
def layer_inputs(name, layer=0):
    cfg = I.CONFIGS[name]
    L = I.make_layer(cfg, layer=layer)
    D = {k: dev(v) for k, v in L.items() if isinstance(v, np.ndarray)}
    return cfg, L, D


def small_layer(hidden, n_experts, top_k, inter, tokens, seed=0):
    cfg = I.MoEConfig("edge", 200 + seed, hidden=hidden, n_experts=n_experts, top_k=top_k,
                      inter=inter, tokens=tokens)
    L = I.make_layer(cfg)
    D = {k: dev(v) for k, v in L.items() if isinstance(v, np.ndarray)}
    return cfg, L, D


def mask_for(cfg, L, pruning):
    if pruning == 0:
        return None
    return oracle.prune_compact(L["importance"], cfg.n_keep(pruning), cfg.top_k)[2]


def run_gpu_layer(sw, D, k, mask=None, x=None, bias=None):
    xm = D["x"] if x is None else x
    keep = None if mask is None else dev(mask)
    return sw.moe_layer(xm, D["wr"], D["w13"], D["w2"], k, keep_mask=keep, bias=bias)


def guarded_layer(sw, D, k, mask=None, bias=None, layout=None, one_call=False):
    """Route + dispatch and forward (or, with `one_call`, sw_moe_layer) with
    every output and workspace inside a canaried allocation (poisoned
    interiors: an unwritten output shows as -7 or NaN); the margins are
    checked after the call."""
    x, wr = D["x"], D["wr"]
    t, m = x.shape[0], wr.shape[0]
    G = Guards()
    out3 = (G.empty((t, k), torch.int32, poison=-7), G.empty((t, k), torch.float32, poison=float("nan")),
            G.empty(t, torch.float32, poison=float("nan")))
    plan = sw.Plan(G.empty(m, torch.int32, poison=-7), G.empty(m + 1, torch.int32, poison=-7),
                   G.empty(max(t * k, 1), torch.int32, poison=-7), G.empty(m, torch.int32, poison=-7),
                   G.empty(1, torch.int32, poison=-7))
    lay = sw.ROW_MAJOR if layout is None else layout
    keep = None if mask is None else dev(mask)
    out = G.empty((t, x.shape[1]), torch.float32, poison=float("nan"))
    if one_call:
        ld = sw.dims(x.shape[1], D["w13"].shape[1] // 2, m, k)
        ids, w, gap, plan, out = sw.sw_moe_layer(
            x, wr, k, D["w13"], D["w2"], layout=lay, keep_mask=keep, bias=bias, route_out=out3,
            plan=plan, out=out, ws=G.workspace(sw.sw_moe_layer_workspace_bytes(ld, t)))
        G.check()
        return dict(topk_ids=ids, topk_w=w, gap=gap, plan=plan, out=out)
    rd = sw.dims(x.shape[1], 8, m, k)
    ids, w, gap, plan = sw.sw_moe_route_dispatch(
        x, wr, k, keep_mask=keep, bias=bias, out=out3, plan=plan,
        ws=G.workspace(sw.sw_moe_route_workspace_bytes(rd, t)))
    fd = sw.dims(x.shape[1], D["w13"].shape[1] // 2, D["w13"].shape[0], k)
    sw.sw_moe_forward(x, D["w13"], D["w2"], w, plan, layout=lay, out=out,
                      ws=G.workspace(sw.sw_moe_forward_workspace_bytes(fd, t)))
    G.check()
    return dict(topk_ids=ids, topk_w=w, gap=gap, plan=plan, out=out)


def bits(t):
    """A tensor's bit patterns (NaN-safe bitwise comparison)."""
    return t.view(torch.int32) if t.dtype == torch.float32 else t


def assert_same_layer(a, b):
    """Two runs of the layer wrote the same bits to every output (the active
    list up to n_active: the plan leaves the rest unwritten)."""
    for key in ("topk_ids", "topk_w", "gap", "out"):
        if a[key] is not None or b[key] is not None:
            assert torch.equal(bits(a[key]), bits(b[key])), key
    for f in ("counts", "offsets", "perm", "n_active"):
        assert torch.equal(getattr(a["plan"], f), getattr(b["plan"], f)), f
    n = max(int(a["plan"].n_active.item()), 0)
    assert torch.equal(a["plan"].active[:n], b["plan"].active[:n])


def check_layer(sw, cfg, L, D, mask, bias=None, rows=None, layout=None, what=None, out_scale=1.0):
    """Route, dispatch and forward on the GPU vs the oracle; returns stats.
    The forward is compared on every token unless `rows` names a subset;
    both outputs are divided by `out_scale` first (inputs scaled up by s
    scale the output by about s^2, and the absolute bound is for unit
    scale)."""
    k = cfg.top_k
    b_dev = None if bias is None else dev(bias)
    g = guarded_layer(sw, D, k, mask=mask, bias=b_dev, layout=layout)
    # the one-call layer (its gate/up launch builds the plan on decode
    # batches) writes the same bits
    assert_same_layer(g, guarded_layer(sw, D, k, mask=mask, bias=b_dev, layout=layout,
                                       one_call=True))
    g_ids, g_w, g_gap = host(g["topk_ids"]), host(g["topk_w"]), host(g["gap"])
    o_ids, o_w, o_gap, o_z = oracle.route(L["x"], L["wr"], k, keep_mask=mask, bias=bias,
                                          want_logits=True)
    r = compare_routing(g_ids, g_w, o_ids, o_w, o_z, mask, k, g_gap=g_gap, o_gap=o_gap,
                        what=what or cfg.name)
    # dispatch: bit-exact against the oracle's dispatch of the GPU's own ids
    counts, offsets, perm, active, n_active = oracle.dispatch(g_ids, cfg.n_experts)
    plan = g["plan"]
    np.testing.assert_array_equal(host(plan.counts), counts)
    np.testing.assert_array_equal(host(plan.offsets), offsets)
    np.testing.assert_array_equal(host(plan.perm)[: g_ids.size], perm)
    assert int(host(plan.n_active)[0]) == n_active
    np.testing.assert_array_equal(host(plan.active)[:n_active], active)
    # forward: against the oracle on the GPU's routing
    rows = np.arange(g_ids.shape[0]) if rows is None else np.asarray(rows)
    o_out = oracle_forward_rows(oracle.forward, L["x"], L["w13"], L["w2"], g_ids, g_w, rows)
    err, rel = compare_out(host(g["out"])[rows] / out_scale, o_out / out_scale)
    return dict(n_near=r["near_ties"], routing=r, n_active=n_active, err=err, rel=rel, gpu=g,
                counts=counts)


# --------------------------------------------------------------------------
# route / dispatch / forward on the named workloads

@pytest.mark.parametrize("name,pruning", [("tiny", 0.0), ("tiny", 0.5), ("decode_b64", 0.0),
                                          ("decode_b64", 0.5)])
def test_layer_parity(sw, name, pruning):
    cfg, L, D = layer_inputs(name)
    mask = mask_for(cfg, L, pruning)
    s = check_layer(sw, cfg, L, D, mask, what=f"{name} p={pruning}")
    print(f"{name} p={pruning}: n_active={s['n_active']} near_ties={s['n_near']} "
          f"max|err|={s['err']:.3g} rel={s['rel']:.3g}")


@pytest.mark.parametrize("name,batch,pruning,family", [("decode_b64", 64, 0.5, "wave"),
                                                       ("decode_b64", 1, 0.0, "split_k"),
                                                       ("decode_sweep", 256, 0.75, "prefill")])
def test_layer_parity_with_saturating_gates(sw, name, batch, pruning, family):
    # Gate/up weights scaled by 32 (exact in bf16), so that the SwiGLU gate g
    # runs far past the range of the exponential both ways (g > 88: silu(g)
    # = g to fp32 precision; g < -88: silu(g) * u vanishes), on each kernel
    # family's epilogue; the router and its tolerances are untouched.  The
    # outputs (32^2 times larger) are compared at unit scale.
    cfg, L, D = layer_inputs(name)
    s = 32.0
    x = I.make_x(cfg, tokens=batch, rep=300 + batch)
    mask = mask_for(cfg, L, pruning)
    w13, w2, wr = L["w13"], L["w2"], L["wr"]
    if pruning:  # the compacted pool, as the benchmark runs it
        n_keep = cfg.n_keep(pruning)
        _, _, _, w13, w2, wr, _ = oracle.prune_compact(L["importance"], n_keep, cfg.top_k,
                                                       w13=w13, w2=w2, wr=wr)
        cfg = dataclasses.replace(cfg, n_experts=n_keep)
        mask = None
    w13 = I.to_bf16_bits(I.bf16_bits_to_f32(w13) * np.float32(s))
    L2 = dict(L, x=x, w13=w13, w2=w2, wr=wr)
    D2 = dict(D, x=dev(x), w13=dev(w13), w2=dev(w2), wr=dev(wr))
    d = sw.dims(cfg.hidden, cfg.inter, cfg.n_experts, cfg.top_k)
    assert sw.sw_moe_forward_kernels(d, batch, sw.ROW_MAJOR)[0] == family
    st = check_layer(sw, cfg, L2, D2, mask, what=f"saturating {name} B={batch}",
                     out_scale=s * s)
    # the gates of the routed pairs do reach both saturated ranges
    ids = host(st["gpu"]["topk_ids"])
    xf = I.bf16_bits_to_f32(x).astype(np.float64)
    g = np.concatenate([I.bf16_bits_to_f32(w13[ids[t, j], :cfg.inter]).astype(np.float64) @ xf[t]
                        for t in range(ids.shape[0]) for j in range(ids.shape[1])])
    assert (g > 88).any() and (g < -88).any(), (g.min(), g.max())
    print(f"saturating {name} B={batch}: g in [{g.min():.0f}, {g.max():.0f}] "
          f"max|err|={st['err']:.3g} rel={st['rel']:.3g} (unit scale)")


@pytest.mark.parametrize("batch", I.SWEEP_BATCHES)
@pytest.mark.parametrize("pruning", I.SWEEP_PRUNING)
def test_decode_sweep_parity(sw, batch, pruning):
    # every batch of the sweep at 0/25/50/75% pruning, every token compared
    cfg, L, D = layer_inputs("decode_sweep")
    mask = mask_for(cfg, L, pruning)
    x = I.make_x(cfg, tokens=batch, rep=batch)
    L2 = dict(L, x=x)
    D2 = dict(D, x=dev(x))
    s = check_layer(sw, cfg, L2, D2, mask, what=f"sweep B={batch} p={pruning}")
    # the router mask keeps the full pool: at most 8 pairs per expert on
    # average, the decode kernels
    d = sw.dims(cfg.hidden, cfg.inter, cfg.n_experts, cfg.top_k)
    fam = sw.sw_moe_forward_kernels(d, batch, sw.ROW_MAJOR)
    if batch >= 64:
        assert fam == ("wave", "wave")
    if batch == 256 and pruning == 0.75:
        # 2048 pairs over 64 experts: experts with more pairs than a whole-K
        # pass holds (sliced passes, double-buffered)
        assert s["counts"].max() > 32
    print(f"sweep B={batch} p={pruning}: kernels={fam} n_active={s['n_active']} "
          f"max pairs/expert={s['counts'].max()} near_ties={s['n_near']} "
          f"max|err|={s['err']:.3g} rel={s['rel']:.3g}")
    n_keep = cfg.n_keep(pruning)
    if pruning and batch * cfg.top_k >= 16 * n_keep:
        # the compacted pool (the one the benchmark times) has 16 or more
        # pairs per expert here: the prefill kernels, against the oracle on
        # the compacted layer
        _, _, _, w13c, w2c, wrc, _ = oracle.prune_compact(L["importance"], n_keep, cfg.top_k,
                                                          w13=L["w13"], w2=L["w2"], wr=L["wr"])
        cc = dataclasses.replace(cfg, n_experts=n_keep)
        dc = sw.dims(cfg.hidden, cfg.inter, n_keep, cfg.top_k)
        assert sw.sw_moe_forward_kernels(dc, batch, sw.ROW_MAJOR) == ("prefill", "prefill")
        sc = check_layer(sw, cc, dict(L2, w13=w13c, w2=w2c, wr=wrc),
                         dict(D2, w13=dev(w13c), w2=dev(w2c), wr=dev(wrc)), None,
                         what=f"sweep compacted B={batch} p={pruning}")
        print(f"  compacted pool ({n_keep} experts): kernels=prefill max pairs/expert="
              f"{sc['counts'].max()} max|err|={sc['err']:.3g} rel={sc['rel']:.3g}")


def test_prefill_shape_parity(sw):
    # 4096 tokens through the full pool of the sweep's layer shape, every token
    cfg, L, D = layer_inputs("decode_sweep")
    pcfg = I.CONFIGS["prefill"]
    x = I.make_x(pcfg)
    d = sw.dims(cfg.hidden, cfg.inter, cfg.n_experts, cfg.top_k)
    assert sw.sw_moe_forward_kernels(d, pcfg.tokens, sw.ROW_MAJOR) == ("prefill", "prefill")
    s = check_layer(sw, cfg, dict(L, x=x), dict(D, x=dev(x)), None, what="prefill T=4096")
    assert s["n_active"] == cfg.n_experts
    print(f"prefill T=4096: near_ties={s['n_near']} max|err|={s['err']:.3g} rel={s['rel']:.3g}")


@pytest.mark.parametrize("pruning", [0.0, 0.5])
def test_skew_routed_batch256_parity(sw, pruning):
    # the skewed stack's routing (Zipf(1.1) logit bias, kept set = the most
    # popular half) on the sweep layer's host-drawn experts at batch 256:
    # popular experts take up to ~80 pairs (sliced passes, the cost-weighted
    # walk); every token is compared
    cfg, L, D = layer_inputs("decode_sweep")
    scfg = I.CONFIGS["skewed_stack"]
    S = I.make_layer(scfg, layer=0, experts=False)
    mask = None if pruning == 0 else oracle.prune_compact(S["importance"], scfg.n_keep(pruning),
                                                          scfg.top_k)[2]
    L2 = dict(L, x=S["x"], wr=S["wr"])
    D2 = dict(D, x=dev(S["x"]), wr=dev(S["wr"]))
    s = check_layer(sw, cfg, L2, D2, mask, bias=S["bias"], what=f"skew-routed B=256 p={pruning}")
    assert s["counts"].max() > 64
    print(f"skew-routed B=256 p={pruning}: n_active={s['n_active']} max pairs/expert="
          f"{s['counts'].max()} near_ties={s['n_near']} max|err|={s['err']:.3g} rel={s['rel']:.3g}")


# --------------------------------------------------------------------------
# the prefill-sized path (16 or more pairs per expert)

def _layer_in_batches(sw, D, k, nb, layout, mask=None, bias=None):
    """The layer over the tokens in batches of nb (small enough for the
    decode kernels), concatenated."""
    outs = []
    for t0 in range(0, D["x"].shape[0], nb):
        g = sw.moe_layer(D["x"][t0:t0 + nb], D["wr"], D["w13"], D["w2"], k, keep_mask=mask,
                         bias=bias, layout=layout)
        outs.append(g["out"])
    return torch.cat(outs)


@pytest.mark.parametrize("tiled", [False, True])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("hidden", [256, 384])
def test_prefill_path_parity_and_equal_to_decode_path(sw, tiled, masked, hidden):
    # 512 tokens, 16 experts, top-4: ~128 tokens per expert, the prefill
    # kernels (4 and 6 gate/up chunks of K, 2 down chunks)
    cfg, L, D = small_layer(hidden, 16, 4, 128, 512, seed=7)
    mask = mask_for(cfg, L, 0.25) if masked else None
    layout = sw.ROW_MAJOR
    if tiled:
        D = dict(D)
        D["w13"], D["w2"] = sw.sw_moe_pack_experts(D["w13"], D["w2"])
        layout = sw.TILED
    d = sw.dims(cfg.hidden, cfg.inter, cfg.n_experts, cfg.top_k)
    assert sw.sw_moe_forward_kernels(d, 512, layout) == ("prefill", "prefill")
    assert sw.sw_moe_forward_kernels(d, 16, layout) == ("wave", "wave")
    keep = None if mask is None else dev(mask)
    g = sw.moe_layer(D["x"], D["wr"], D["w13"], D["w2"], cfg.top_k, keep_mask=keep, layout=layout)
    g_ids, g_w = host(g["topk_ids"]), host(g["topk_w"])
    o_ids, o_w, o_gap, o_z = oracle.route(L["x"], L["wr"], cfg.top_k, keep_mask=mask, want_logits=True)
    compare_routing(g_ids, g_w, o_ids, o_w, o_z, mask, cfg.top_k, g_gap=host(g["gap"]), o_gap=o_gap)
    o_out = oracle.forward(L["x"], L["w13"], L["w2"], g_ids, g_w)
    compare_out(host(g["out"]), o_out)
    # each output accumulates in the same order on both paths: bit for bit
    small = _layer_in_batches(sw, D, cfg.top_k, 16, layout, mask=keep)
    assert torch.equal(g["out"], small)


def test_prefill_path_uneven_experts(sw):
    # graded router biases: expert loads from ~460 tokens (passes of 160,
    # 160 and ~140) down to one, so every pass shape of the prefill kernels
    # (4, 8 and 10 column blocks) runs, several with only 1-3 blocks used
    cfg, L, D = small_layer(256, 16, 4, 128, 512, seed=9)
    bias = np.linspace(1.0, -1.0, 16).astype(np.float32)
    layout = sw.TILED
    D = dict(D)
    D["w13"], D["w2"] = sw.sw_moe_pack_experts(D["w13"], D["w2"])
    d = sw.dims(cfg.hidden, cfg.inter, cfg.n_experts, cfg.top_k)
    assert sw.sw_moe_forward_kernels(d, 512, layout) == ("prefill", "prefill")
    g = sw.moe_layer(D["x"], D["wr"], D["w13"], D["w2"], 4, bias=dev(bias), layout=layout)
    counts = host(g["plan"].counts)
    last = [c % 160 for c in counts if c > 0]
    assert counts.max() > 320 and any(0 < r <= 64 for r in last) and any(64 < r <= 128 for r in last)
    g_ids, g_w = host(g["topk_ids"]), host(g["topk_w"])
    o_ids, o_w, o_gap, o_z = oracle.route(L["x"], L["wr"], 4, bias=bias, want_logits=True)
    compare_routing(g_ids, g_w, o_ids, o_w, o_z, None, 4, g_gap=host(g["gap"]), o_gap=o_gap)
    compare_out(host(g["out"]), oracle.forward(L["x"], L["w13"], L["w2"], g_ids, g_w))
    small = _layer_in_batches(sw, D, 4, 16, layout, bias=dev(bias))
    assert torch.equal(g["out"], small)


@pytest.mark.parametrize("tiled", [False, True])
def test_prefill_path_expert_with_several_passes(sw, tiled):
    # a bias makes expert 3 every token's first choice: 400 pairs on one
    # expert (passes of 160, 160 and 80 tokens); 16 experts keep the layer
    # on the prefill kernels
    cfg, L, D = small_layer(256, 16, 2, 128, 400, seed=8)
    bias = np.zeros(16, np.float32)
    bias[3] = 50.0
    layout = sw.ROW_MAJOR
    if tiled:
        D = dict(D)
        D["w13"], D["w2"] = sw.sw_moe_pack_experts(D["w13"], D["w2"])
        layout = sw.TILED
    d = sw.dims(cfg.hidden, cfg.inter, cfg.n_experts, cfg.top_k)
    assert sw.sw_moe_forward_kernels(d, 400, layout) == ("prefill", "prefill")
    assert sw.sw_moe_forward_kernels(d, 16, layout) == ("wave", "wave")
    g = sw.moe_layer(D["x"], D["wr"], D["w13"], D["w2"], 2, bias=dev(bias), layout=layout)
    assert int(host(g["plan"].counts)[3]) == 400
    g_ids, g_w = host(g["topk_ids"]), host(g["topk_w"])
    o_ids, o_w, o_gap, o_z = oracle.route(L["x"], L["wr"], 2, bias=bias, want_logits=True)
    compare_routing(g_ids, g_w, o_ids, o_w, o_z, None, 2, g_gap=host(g["gap"]), o_gap=o_gap)
    compare_out(host(g["out"]), oracle.forward(L["x"], L["w13"], L["w2"], g_ids, g_w))
    small = _layer_in_batches(sw, D, 2, 16, layout, bias=dev(bias))
    assert torch.equal(g["out"], small)


# --------------------------------------------------------------------------
# pruning: masked full pool == compacted pool, 0% == full, GPU compaction

@pytest.mark.parametrize("name,pruning", [("tiny", 0.5), ("decode_b64", 0.5), ("decode_sweep", 0.25)])
def test_prune_compact_parity_and_masked_equals_compacted(sw, name, pruning):
    cfg, L, D = layer_inputs(name)
    n_keep = cfg.n_keep(pruning)
    g = sw.sw_moe_prune_compact(D["importance"], n_keep, cfg.top_k, w13=D["w13"], w2=D["w2"], wr=D["wr"])
    kept, remap, mask, w13c, w2c, wrc, _ = oracle.prune_compact(L["importance"], n_keep, cfg.top_k,
                                                                w13=L["w13"], w2=L["w2"], wr=L["wr"])
    np.testing.assert_array_equal(host(g["kept"]), kept)
    np.testing.assert_array_equal(host(g["remap"]), remap)
    np.testing.assert_array_equal(host(g["keep_mask"]), mask)
    np.testing.assert_array_equal(host(g["wr"]), wrc)
    assert torch.equal(g["w13"], dev(w13c)) and torch.equal(g["w2"], dev(w2c))
    # Eq. 2: the masked router over the full pool picks exactly what the
    # pruned checkpoint picks, with identical gates and outputs
    masked = run_gpu_layer(sw, D, cfg.top_k, mask=mask)
    comp = sw.moe_layer(D["x"], g["wr"], g["w13"], g["w2"], cfg.top_k)
    kept_t = g["kept"].long()
    assert torch.equal(masked["topk_ids"].long(), kept_t[comp["topk_ids"].long()])
    assert torch.equal(masked["topk_w"], comp["topk_w"])
    assert torch.equal(masked["out"], comp["out"])


def test_zero_pruning_is_the_full_model_and_deterministic(sw):
    cfg, L, D = layer_inputs("decode_b64")
    a = run_gpu_layer(sw, D, cfg.top_k)
    b = run_gpu_layer(sw, D, cfg.top_k, mask=np.ones(cfg.n_experts, np.uint8))
    c = run_gpu_layer(sw, D, cfg.top_k)
    for key in ("topk_ids", "topk_w", "out"):
        assert torch.equal(a[key], b[key]), key
        assert torch.equal(a[key], c[key]), key


def test_pruned_experts_never_selected_and_gates_ignore_them(sw):
    cfg, L, D = layer_inputs("decode_b64")
    mask = mask_for(cfg, L, 0.5)
    a = run_gpu_layer(sw, D, cfg.top_k, mask=mask)
    ids = host(a["topk_ids"])
    assert np.all(mask[ids] == 1)
    wr2 = D["wr"].clone()
    wr2[torch.from_numpy(mask == 0).cuda()] = 5.0
    b = sw.moe_layer(D["x"], wr2, D["w13"], D["w2"], cfg.top_k, keep_mask=dev(mask))
    for key in ("topk_ids", "topk_w", "out"):
        assert torch.equal(a[key], b[key]), key


# --------------------------------------------------------------------------
# edge cases

@pytest.mark.parametrize("hidden,n_experts,top_k,inter,tokens", [
    (72, 5, 5, 8, 3),         # every expert selected; H not a multiple of 32; I = 8
    (64, 16, 1, 32, 17),      # top-1: gates are exactly 1
    (256, 1024, 32, 16, 9),   # largest pool and k
    (128, 3, 2, 24, 1),       # a single token
    (520, 12, 4, 40, 70),     # ragged H and I tails
])
def test_edge_shapes(sw, hidden, n_experts, top_k, inter, tokens):
    cfg, L, D = small_layer(hidden, n_experts, top_k, inter, tokens)
    s = check_layer(sw, cfg, L, D, None)
    if top_k == 1:
        assert np.all(host(s["gpu"]["topk_w"]) == 1.0)


# the split-K path (few tiles: each tile's K spread over the waves of a block)

@pytest.mark.parametrize("name,batch,pruning", [("decode_sweep", 1, 0.0), ("decode_sweep", 2, 0.5),
                                                ("decode_sweep", 3, 0.25), ("decode_b64", 1, 0.0),
                                                ("decode_b64", 2, 0.5)])
def test_split_k_decode_parity_and_layouts_agree(sw, name, batch, pruning):
    cfg, L, D = layer_inputs(name)
    mask = mask_for(cfg, L, pruning)
    x = I.make_x(cfg, tokens=batch, rep=100 + batch)
    s = check_layer(sw, cfg, dict(L, x=x), dict(D, x=dev(x)), mask)
    assert s["n_active"] <= batch * cfg.top_k
    t13, t2 = sw.sw_moe_pack_experts(D["w13"], D["w2"])
    keep = None if mask is None else dev(mask)
    tl = sw.moe_layer(dev(x), D["wr"], t13, t2, cfg.top_k, keep_mask=keep, layout=sw.TILED)
    assert torch.equal(tl["out"], s["gpu"]["out"])
    print(f"split-K {name} B={batch} p={pruning}: n_active={s['n_active']} "
          f"max|err|={s['err']:.3g} rel={s['rel']:.3g}")


@pytest.mark.parametrize("hidden,n_experts,top_k,inter,tokens,popular", [
    (1056, 24, 2, 296, 5, False),   # 37 gate/up tiles per expert: tile pairs span two experts
    (1056, 24, 3, 288, 7, False),   # 66 down tiles per expert, 8 per block: groups span experts
    (1024, 30, 4, 288, 20, True),   # 20 tokens on expert 0: two 16-token blocks in its pass;
                                    # down on one wave per tile over 9 K steps
])
def test_split_k_ragged_shapes(sw, hidden, n_experts, top_k, inter, tokens, popular):
    cfg, L, D = small_layer(hidden, n_experts, top_k, inter, tokens, seed=11)
    bias = None
    if popular:
        bias = np.zeros(n_experts, np.float32)
        bias[0] = 50.0
    s = check_layer(sw, cfg, L, D, None, bias=bias)
    if popular:
        assert int(host(s["gpu"]["plan"].counts)[0]) == tokens


def test_popular_expert_spans_several_token_passes(sw):
    # a bias makes expert 3 every token's first choice: 200 pairs on one
    # expert (two passes of 100 tokens over its weights)
    cfg, L, D = small_layer(256, 16, 2, 64, 200, seed=1)
    bias = np.zeros(16, np.float32)
    bias[3] = 50.0
    s = check_layer(sw, cfg, L, D, None, bias=bias)
    assert int(host(s["gpu"]["plan"].counts)[3]) == 200


@pytest.mark.parametrize("hidden,n_experts,top_k,inter,tokens,popular", [
    (512, 16, 2, 96, 300, (3, 7)),   # two experts take every token: 3 passes each,
                                     # 2 of 16 experts active (first segment guessed, redone)
    (256, 64, 2, 64, 100, (5,)),     # one expert with a 100-token pass among ~50 light
                                     # ones (no guess: many idle experts expected)
])
def test_weighted_walk_over_popular_experts(sw, hidden, n_experts, top_k, inter, tokens, popular):
    # popular experts with sliced or several passes: the decode kernels'
    # blocks take equal runs of estimated cost instead of equal tile ranges
    cfg, L, D = small_layer(hidden, n_experts, top_k, inter, tokens, seed=13)
    bias = np.zeros(n_experts, np.float32)
    bias[list(popular)] = 50.0
    s = check_layer(sw, cfg, L, D, None, bias=bias)
    counts = host(s["gpu"]["plan"].counts)
    assert all(int(counts[e]) == tokens for e in popular)


@pytest.mark.parametrize("hidden,n_experts,top_k,inter,tokens,popular", [
    (2048, 64, 4, 512, 64, (3,)),      # 64-token batch: 32-token passes, the popular expert
                                       # in two (each tile streamed twice)
    (1056, 48, 4, 384, 80, (2,)),      # H 1056 (5 chunks, the last one K step): one-chunk slices
    (2048, 32, 4, 1024, 120, (0, 1)),  # 120 pairs: gate/up 8 one-chunk slices; down 2 passes of
                                       # 60 tokens over 4 h slices (I 1024)
    (2048, 48, 4, 768, 100, (5,)),     # gate/up 8 one-chunk slices; down 2 passes of 50 tokens,
                                       # h slices of one chunk
    (2048, 40, 4, 512, 90, (7,)),      # down: 90 tokens, one LDS buffer (two do not fit): h slices
                                       # of one chunk staged at each slice's start
])
@pytest.mark.parametrize("tiled", [False, True])
def test_sliced_passes_stream_each_tile_once(sw, hidden, n_experts, top_k, inter, tokens, popular,
                                             tiled):
    # experts whose tokens do not fit in LDS with the whole contraction take
    # sliced passes (K in slices, every token staged per slice); each output
    # still accumulates over K in the same order, so it equals the same
    # tokens run in small batches (whole-K passes) bit for bit
    cfg, L, D = small_layer(hidden, n_experts, top_k, inter, tokens, seed=17)
    bias = np.zeros(n_experts, np.float32)
    bias[list(popular)] = 50.0
    layout = sw.ROW_MAJOR
    if tiled:
        D = dict(D)
        D["w13"], D["w2"] = sw.sw_moe_pack_experts(D["w13"], D["w2"])
        layout = sw.TILED
    d = sw.dims(hidden, inter, n_experts, top_k)
    assert sw.sw_moe_forward_kernels(d, tokens, layout) == ("wave", "wave")
    # reference batches that divide the tokens and run whole-K passes of the
    # same kernels (a ragged last batch could take the split-K kernels)
    nb = next(b for b in (16, 20, 24, 30) if tokens % b == 0)
    assert sw.sw_moe_forward_kernels(d, nb, layout) == ("wave", "wave")
    s = check_layer(sw, cfg, L, D, None, bias=bias, layout=layout,
                    what=f"sliced H={hidden} I={inter} T={tokens}")
    assert all(int(s["counts"][e]) == tokens for e in popular)
    small = _layer_in_batches(sw, D, top_k, nb, layout, bias=dev(bias))
    assert torch.equal(s["gpu"]["out"], small)


def test_bias_and_mask_together(sw):
    cfg = I.CONFIGS["skewed_stack"]
    small = I.MoEConfig("skew_small", cfg.config_id, hidden=256, n_experts=cfg.n_experts,
                        top_k=cfg.top_k, inter=64, tokens=96, zipf_s=cfg.zipf_s,
                        zipf_beta=cfg.zipf_beta)
    L = I.make_layer(small)
    D = {k: dev(v) for k, v in L.items() if isinstance(v, np.ndarray)}
    mask = oracle.prune_compact(L["importance"], 128, small.top_k)[2]
    check_layer(sw, small, L, D, mask, bias=L["bias"])


def test_empty_batch(sw):
    cfg, L, D = small_layer(64, 8, 2, 32, 1)
    x0 = D["x"][:0]
    ids, w, gap = sw.sw_moe_route(x0, D["wr"], 2)
    plan = sw.sw_moe_dispatch(ids, 8)
    out = sw.sw_moe_forward(x0, D["w13"], D["w2"], w, plan)
    assert out.shape == (0, 64)
    assert int(plan.n_active.item()) == 0
    assert torch.all(plan.counts == 0) and torch.all(plan.offsets == 0)


def test_invalid_ids_flag_the_dispatch_and_poison_the_output(sw):
    cfg, L, D = small_layer(64, 8, 2, 32, 4)
    ids = torch.tensor([[0, 1], [2, 9], [3, 4], [5, 6]], dtype=torch.int32, device="cuda")
    w = torch.full((4, 2), 0.5, device="cuda")
    plan = sw.sw_moe_dispatch(ids, 8)
    assert int(plan.n_active.item()) == -1
    assert torch.all(plan.counts == 0)
    assert torch.equal(plan.perm.cpu(), torch.arange(8, dtype=torch.int32))
    out = sw.sw_moe_forward(D["x"], D["w13"], D["w2"], w, plan)
    assert torch.all(torch.isnan(out))


def test_too_few_eligible_experts_in_band(sw):
    cfg, L, D = small_layer(64, 8, 3, 32, 2)
    mask = np.zeros(8, np.uint8)
    mask[[1, 6]] = 1
    ids, w, gap = sw.sw_moe_route(D["x"], D["wr"], 3, keep_mask=dev(mask))
    ids = host(ids)
    assert np.all(ids[:, 2] == -1) and np.all(host(w)[:, 2] == 0)
    assert np.all(np.isnan(host(gap)))
    assert set(ids[:, :2].ravel().tolist()) <= {1, 6}


def test_dispatch_skewed_and_large(sw):
    g = np.random.default_rng(5)
    for t, m, k in [(4096, 256, 8), (3, 1024, 32), (700, 64, 1), (333, 256, 8)]:
        rows = []
        for i in range(t):
            if i % 2 == 0 and k > 1:  # every other token also picks the popular expert 7
                rest = g.choice(np.delete(np.arange(m), 7), size=k - 1, replace=False)
                rows.append(np.insert(rest, i % k, 7))
            else:
                rows.append(g.choice(m, size=k, replace=False))
        ids = np.stack(rows).astype(np.int32)
        plan = sw.sw_moe_dispatch(dev(ids), m)
        counts, offsets, perm, active, n_active = oracle.dispatch(ids, m)
        np.testing.assert_array_equal(host(plan.counts), counts)
        np.testing.assert_array_equal(host(plan.offsets), offsets)
        np.testing.assert_array_equal(host(plan.perm)[: t * k], perm)
        assert int(host(plan.n_active)[0]) == n_active
        np.testing.assert_array_equal(host(plan.active)[:n_active], active)


@pytest.mark.parametrize("tokens,m,k", [
    (64, 512, 8),    # 512 pairs over 512 experts: the half-size plan block at both limits
    (57, 512, 9),    # 513 pairs: the full block
    (64, 513, 8),    # 513 experts: the full block
    (1, 1, 1),       # one pair, one expert
    (73, 7, 7),      # 511 pairs, every token picks every expert
])
def test_dispatch_plan_block_size_boundaries(sw, tokens, m, k):
    g = np.random.default_rng(tokens * 1000 + m)
    ids = np.stack([g.choice(m, size=k, replace=False) for _ in range(tokens)]).astype(np.int32)
    plan = sw.sw_moe_dispatch(dev(ids), m)
    counts, offsets, perm, active, n_active = oracle.dispatch(ids, m)
    np.testing.assert_array_equal(host(plan.counts), counts)
    np.testing.assert_array_equal(host(plan.offsets), offsets)
    np.testing.assert_array_equal(host(plan.perm)[: tokens * k], perm)
    assert int(host(plan.n_active)[0]) == n_active
    np.testing.assert_array_equal(host(plan.active)[:n_active], active)


@pytest.mark.parametrize("n_experts,top_k,tokens", [
    (64, 8, 32), (40, 3, 32),     # the row form (a token per 16-lane row, the plan by the block)
    (128, 8, 8), (256, 16, 4),    # the wave form with the plan (64 pairs)
    (128, 8, 33), (256, 16, 63),  # the top-k kernel itself on part of the batch
])
def test_selection_forms_agree_bit_for_bit(sw, n_experts, top_k, tokens):
    # sw_moe_route of 64 tokens takes the top-k kernel (a token per wave); the
    # first tokens' logits are the same in a smaller batch, so whatever form
    # selects there, ids, gates and gaps must be
    cfg, L, D = small_layer(2048, n_experts, top_k, 32, 64, seed=13)
    ids64, w64, gap64 = sw.sw_moe_route(D["x"], D["wr"], top_k)
    ids, w, gap, _ = sw.sw_moe_route_dispatch(D["x"][:tokens].contiguous(), D["wr"], top_k)
    assert torch.equal(ids64[:tokens], ids)
    assert torch.equal(w64[:tokens], w)
    assert torch.equal(gap64[:tokens], gap)


def test_exact_logit_ties_break_to_smaller_id(sw):
    # identical router rows give bit-identical logits on both sides
    cfg, L, D = small_layer(256, 40, 6, 32, 33, seed=2)
    wr = L["wr"].copy()
    for dup in (7, 19, 33):
        wr[dup] = wr[3]
    wr[39] = wr[0]
    ids, w, gap = sw.sw_moe_route(D["x"], dev(wr), 6)
    o_ids, o_w, o_gap = oracle.route(L["x"], wr, 6)
    np.testing.assert_array_equal(host(ids), o_ids)
    np.testing.assert_allclose(host(w), o_w, atol=1e-5)
    np.testing.assert_allclose(host(gap), o_gap, atol=1e-5)
    for r in host(ids):
        pos = {int(e): j for j, e in enumerate(r)}
        if 3 in pos and 7 in pos:
            assert pos[3] < pos[7]


def test_dispatch_every_pair_on_one_expert(sw):
    for t, k in [(300, 1), (64, 1), (2000, 1)]:
        ids = np.full((t, k), 5, np.int32)
        plan = sw.sw_moe_dispatch(dev(ids), 9)
        counts, offsets, perm, active, n_active = oracle.dispatch(ids, 9)
        np.testing.assert_array_equal(host(plan.counts), counts)
        np.testing.assert_array_equal(host(plan.offsets), offsets)
        np.testing.assert_array_equal(host(plan.perm)[: t * k], perm)
        assert int(host(plan.n_active)[0]) == n_active == 1


# --------------------------------------------------------------------------
# tiled (fragment-major) weight layout

def np_tile(rows16):
    """[16, K] -> [K/32 * 64 * 8]: fragment s, lane l = 16*kg + row, 8 values."""
    k = rows16.shape[1]
    return rows16.reshape(16, k // 32, 4, 8).transpose(1, 2, 0, 3).reshape(-1)


def np_tile_w13(w13):
    m, two_i, h = w13.shape
    inter = two_i // 2
    out = []
    for e in range(m):
        for b in range(inter // 8):
            rows = np.concatenate([w13[e, 8 * b:8 * b + 8], w13[e, inter + 8 * b:inter + 8 * b + 8]])
            out.append(np_tile(rows))
    return np.concatenate(out).reshape(w13.shape)


def np_tile_w2(w2):
    m, h, inter = w2.shape
    return np.concatenate([np_tile(w2[e, 16 * b:16 * b + 16]) for e in range(m)
                           for b in range(h // 16)]).reshape(w2.shape)


@pytest.mark.parametrize("hidden,inter,m", [(64, 32, 3), (256, 128, 5), (2048, 96, 2)])
def test_pack_matches_layout_definition(sw, hidden, inter, m):
    cfg, L, D = small_layer(hidden, m, 1, inter, 1, seed=3)
    t13, t2 = sw.sw_moe_pack_experts(D["w13"], D["w2"])
    np.testing.assert_array_equal(host(t13), np_tile_w13(L["w13"]))
    np.testing.assert_array_equal(host(t2), np_tile_w2(L["w2"]))


@pytest.mark.parametrize("name,pruning,batch", [("tiny", 0.5, None), ("decode_b64", 0.0, None),
                                                ("decode_b64", 0.5, None), ("decode_sweep", 0.5, 64),
                                                ("decode_sweep", 0.0, 256), ("decode_sweep", 0.5, 1)])
def test_tiled_forward_parity_and_bitwise_equal_to_row_major(sw, name, pruning, batch):
    cfg, L, D = layer_inputs(name)
    mask = mask_for(cfg, L, pruning)
    x_np = L["x"] if batch is None else I.make_x(cfg, tokens=batch, rep=7)
    x = dev(x_np)
    t13, t2 = sw.sw_moe_pack_experts(D["w13"], D["w2"])
    keep = None if mask is None else dev(mask)
    rm = sw.moe_layer(x, D["wr"], D["w13"], D["w2"], cfg.top_k, keep_mask=keep)
    tl = sw.moe_layer(x, D["wr"], t13, t2, cfg.top_k, keep_mask=keep, layout=sw.TILED)
    assert torch.equal(rm["out"], tl["out"])
    ids, w = host(tl["topk_ids"]), host(tl["topk_w"])
    o_out = oracle_forward_rows(oracle.forward, x_np, L["w13"], L["w2"], ids, w)
    compare_out(host(tl["out"]), o_out)


def test_benchmark_configuration_parity(sw):
    # The configuration the decode benchmark times: the batch-64 layer pruned
    # to 64 of its 128 experts by the library's own compaction of the tiled
    # pool, one sw_moe_layer call (the gate/up launch builds the plan and,
    # every kept expert being active, takes the fully-active guess), against
    # the oracle on the oracle's compacted layer, every token.
    cfg, L, D = layer_inputs("decode_b64")
    n_keep = cfg.n_keep(0.5)
    t13, t2 = sw.sw_moe_pack_experts(D["w13"], D["w2"])
    c = sw.sw_moe_prune_compact(D["importance"], n_keep, cfg.top_k, w13=t13, w2=t2, wr=D["wr"])
    kept, _, _, w13c, w2c, wrc, _ = oracle.prune_compact(L["importance"], n_keep, cfg.top_k,
                                                         w13=L["w13"], w2=L["w2"], wr=L["wr"])
    np.testing.assert_array_equal(host(c["kept"]), kept)
    cc = dataclasses.replace(cfg, n_experts=n_keep)
    d = sw.dims(cfg.hidden, cfg.inter, n_keep, cfg.top_k)
    assert sw.sw_moe_gate_up_builds_plan(d, cfg.tokens, sw.TILED)
    assert sw.sw_moe_forward_kernels(d, cfg.tokens, sw.TILED) == ("wave", "wave")
    Lc = dict(L, w13=w13c, w2=w2c, wr=wrc)
    Dc = dict(D, w13=c["w13"], w2=c["w2"], wr=c["wr"])
    st = check_layer(sw, cc, Lc, Dc, None, layout=sw.TILED, what="benchmark configuration")
    assert st["n_active"] == n_keep  # the fully-active guess holds
    print(f"benchmark configuration: n_active={st['n_active']} near_ties={st['n_near']} "
          f"max|err|={st['err']:.3g} rel={st['rel']:.3g}")


def test_compacting_a_tiled_pool_equals_tiling_the_compacted_pool(sw):
    cfg, L, D = layer_inputs("decode_b64")
    n_keep = cfg.n_keep(0.5)
    t13, t2 = sw.sw_moe_pack_experts(D["w13"], D["w2"])
    a = sw.sw_moe_prune_compact(D["importance"], n_keep, cfg.top_k, w13=t13, w2=t2, wr=D["wr"])
    b = sw.sw_moe_prune_compact(D["importance"], n_keep, cfg.top_k, w13=D["w13"], w2=D["w2"], wr=D["wr"])
    bt13, bt2 = sw.sw_moe_pack_experts(b["w13"], b["w2"])
    assert torch.equal(a["w13"], bt13) and torch.equal(a["w2"], bt2)


# --------------------------------------------------------------------------
# fused route + dispatch: bitwise the separate calls

def _route_then_dispatch(sw, x, wr, k, m, **kw):
    ids, w, gap = sw.sw_moe_route(x, wr, k, **kw)
    plan = sw.sw_moe_dispatch(ids, m)
    return ids, w, gap, plan


def _assert_same_route_dispatch(a, b):
    ids_a, w_a, gap_a, pa = a
    ids_b, w_b, gap_b, pb = b
    assert torch.equal(ids_a, ids_b)
    # gates and gaps bit for bit (NaN gaps compared as bits)
    assert torch.equal(w_a.view(torch.int32), w_b.view(torch.int32))
    assert torch.equal(gap_a.view(torch.int32), gap_b.view(torch.int32))
    n = int(pa.n_active.item())
    assert n == int(pb.n_active.item())
    for f in ("counts", "offsets", "perm"):
        assert torch.equal(getattr(pa, f), getattr(pb, f)), f
    if n > 0:
        assert torch.equal(pa.active[:n], pb.active[:n])


@pytest.mark.parametrize("hidden,n_experts,top_k,tokens,masked,biased", [
    (256, 16, 2, 8, False, False),        # tiny shape, one logit slice
    (2048, 64, 8, 32, False, False),      # the row form's largest batch and pool
    (2048, 128, 8, 21, True, False),      # a 50% mask; separate kernels, ragged last block
    (2048, 256, 8, 1, False, True),       # one token, 256 experts, with bias
    (2048, 64, 8, 4, True, False),        # 4 tokens: a wave each, one wave's plan of 32 pairs
    (2048, 128, 16, 4, False, True),      # 64 pairs: the one-wave plan at its limit
    (512, 256, 1, 3, False, False),       # k = 1 on the one-wave plan
    (256, 16, 2, 5, False, False),        # 5 tokens, 10 pairs
    (2048, 256, 16, 32, True, True),      # k = 16 over 256 experts: separate kernels
    (2048, 128, 8, 33, True, False),      # 33 tokens: top-k, then dispatch
    (2048, 128, 8, 64, False, False),     # 64 tokens: the same
    (2048, 64, 16, 64, True, True),       # 1024 pairs, k = 16
    (2048, 256, 8, 256, False, True),     # 2048 pairs: the largest one-block dispatch
    (2048, 512, 8, 256, False, False),    # 2048 pairs over 512 experts (8 per lane)
    (1024, 200, 16, 100, True, False),    # k = 16, ragged last top-k block
    (2048, 256, 8, 600, False, False),    # 4800 pairs: chunked multi-block dispatch
    (2048, 256, 8, 4096, True, False),    # prefill: wide logit tiles, 32 dispatch chunks
    (1536, 100, 6, 700, False, True),     # wide logit tiles with ragged token and expert tiles
    (512, 300, 8, 40, False, False),      # m > 256
    (1024, 600, 4, 40, False, False),     # m > 512: 10 experts per lane
    (256, 64, 17, 20, False, False),      # k > 16: separate kernels over a small pool
    (520, 12, 4, 70, True, False),        # ragged H
])
def test_route_dispatch_equals_route_then_dispatch(sw, hidden, n_experts, top_k, tokens, masked,
                                                   biased):
    cfg, L, D = small_layer(hidden, n_experts, top_k, 32, tokens, seed=3)
    kw = {}
    if masked:
        kw["keep_mask"] = dev(oracle.prune_compact(L["importance"], n_experts // 2, top_k)[2])
    if biased:
        g = np.random.default_rng(11)
        kw["bias"] = dev((0.5 * g.standard_normal(n_experts)).astype(np.float32))
    a = _route_then_dispatch(sw, D["x"], D["wr"], top_k, n_experts, **kw)
    b = sw.sw_moe_route_dispatch(D["x"], D["wr"], top_k, **kw)
    _assert_same_route_dispatch(a, b)
    # and the routing itself against the oracle
    mask_np = host(kw["keep_mask"]) if masked else None
    bias_np = host(kw["bias"]) if biased else None
    ids_o, w_o, gap_o, z_o = oracle.route(L["x"], L["wr"], top_k, keep_mask=mask_np, bias=bias_np,
                                          want_logits=True)
    compare_routing(host(b[0]), host(b[1]), ids_o, w_o, z_o, mask_np, top_k, g_gap=host(b[2]),
                    o_gap=gap_o)


def test_route_dispatch_in_band_errors_and_empty_batch(sw):
    cfg, L, D = small_layer(64, 8, 3, 32, 2)
    mask = np.zeros(8, np.uint8)
    mask[[1, 6]] = 1
    a = _route_then_dispatch(sw, D["x"], D["wr"], 3, 8, keep_mask=dev(mask))
    b = sw.sw_moe_route_dispatch(D["x"], D["wr"], 3, keep_mask=dev(mask))
    _assert_same_route_dispatch(a, b)
    assert int(b[3].n_active.item()) == -1      # the missing third choice flags the batch
    # the same flag from the row form (30 tokens, 90 pairs) and after the
    # separate top-k (70 tokens)
    for tokens in (30, 70):
        cfg, L, D = small_layer(64, 8, 3, 32, tokens, seed=5)
        a = _route_then_dispatch(sw, D["x"], D["wr"], 3, 8, keep_mask=dev(mask))
        b = sw.sw_moe_route_dispatch(D["x"], D["wr"], 3, keep_mask=dev(mask))
        _assert_same_route_dispatch(a, b)
        assert int(b[3].n_active.item()) == -1
    # the same in-band flag from the chunked dispatch (3000 pairs)
    cfg, L, D = small_layer(64, 8, 3, 32, 1000, seed=4)
    a = _route_then_dispatch(sw, D["x"], D["wr"], 3, 8, keep_mask=dev(mask))
    b = sw.sw_moe_route_dispatch(D["x"], D["wr"], 3, keep_mask=dev(mask))
    _assert_same_route_dispatch(a, b)
    assert int(b[3].n_active.item()) == -1
    assert torch.equal(b[3].perm, torch.arange(3000, dtype=torch.int32, device=b[3].perm.device))
    ids, w, gap, plan = sw.sw_moe_route_dispatch(D["x"][:0], D["wr"], 3)
    assert ids.shape == (0, 3)
    assert int(plan.n_active.item()) == 0
    assert torch.all(plan.counts == 0) and torch.all(plan.offsets == 0)


# --------------------------------------------------------------------------
# the one-call layer: on decode batches its gate/up launch builds the plan

@pytest.mark.parametrize("hidden,n_experts,top_k,inter,tokens,tiled,popular,builds", [
    (512, 64, 8, 256, 64, True, False, True),     # fully active guess
    (512, 128, 8, 256, 64, True, False, True),    # idle experts expected: no guess
    (512, 64, 8, 256, 33, False, False, True),    # row-major weights
    (512, 256, 8, 256, 8, True, False, True),     # 8 tokens over 256 experts
    (256, 16, 2, 128, 3, False, False, True),     # the smallest batch of the wave kernels
    (512, 512, 8, 256, 48, True, False, True),    # 512 experts: the plan's scan limit
    (512, 512, 16, 256, 64, True, False, False),  # 1024 pairs over 512 experts: LDS too small
    (512, 64, 8, 256, 64, True, True, True),      # one expert takes every token: two passes
    (512, 64, 8, 256, 2, True, False, False),     # 2 tokens: split-K kernels
    (512, 64, 8, 256, 65, True, False, False),    # 65 tokens: the 128-token variants
    (256, 480, 16, 128, 63, True, False, True),   # 2450 plan words: just within the LDS plan
    (256, 480, 16, 128, 64, True, False, False),  # 2466 plan words: just past it
    (256, 512, 14, 128, 64, False, False, True),  # 512 experts and 896 pairs: 2434 plan words
])
def test_layer_call_against_oracle_and_separate_calls(sw, hidden, n_experts, top_k, inter, tokens,
                                                      tiled, popular, builds):
    cfg, L, D = small_layer(hidden, n_experts, top_k, inter, tokens, seed=31)
    layout = sw.ROW_MAJOR
    if tiled:
        D = dict(D)
        D["w13"], D["w2"] = sw.sw_moe_pack_experts(D["w13"], D["w2"])
        layout = sw.TILED
    bias = None
    if popular:
        bias = np.zeros(n_experts, np.float32)
        bias[5] = 30.0
    # check_layer runs the separate calls against the oracle and the one-call
    # layer against them, bit for bit
    s = check_layer(sw, cfg, L, D, None, bias=bias, layout=layout,
                    what=f"layer call T={tokens} m={n_experts}")
    if popular:
        assert s["counts"][5] == tokens
    # where the plan is built in the gate/up launch, a second call gives the
    # same bits (every block builds the same plan)
    a = guarded_layer(sw, D, top_k, bias=None if bias is None else dev(bias), layout=layout,
                      one_call=True)
    b = guarded_layer(sw, D, top_k, bias=None if bias is None else dev(bias), layout=layout,
                      one_call=True)
    assert_same_layer(a, b)
    pairs = tokens * top_k
    fam = sw.sw_moe_forward_kernels(sw.dims(hidden, inter, n_experts, top_k), tokens, layout)
    print(f"layer call T={tokens} m={n_experts} k={top_k}: kernels={fam} builds plan={builds} "
          f"({3 * n_experts + 2 + pairs} plan words) max|err|={s['err']:.3g}")


@pytest.mark.parametrize("hidden,n_experts,top_k,inter,tokens", [
    (512, 64, 8, 256, 64),    # gate/up builds the plan, the pool fully active
    (512, 256, 8, 256, 40),   # gate/up builds the plan, idle experts expected
    (512, 64, 8, 256, 100),   # routing + dispatch, then the forward's launches
])
def test_layer_phases_in_order_are_the_layer_call(sw, hidden, n_experts, top_k, inter, tokens):
    cfg, L, D = small_layer(hidden, n_experts, top_k, inter, tokens, seed=41)
    w13, w2 = sw.sw_moe_pack_experts(D["w13"], D["w2"])
    whole = sw.sw_moe_layer(D["x"], D["wr"], top_k, w13, w2, layout=sw.TILED)
    d = sw.dims(hidden, inter, n_experts, top_k)
    bufs = ((torch.empty_like(whole[0]), torch.empty_like(whole[1]), torch.empty_like(whole[2])),
            sw.alloc_plan(tokens, n_experts, top_k, "cuda"), torch.empty_like(whole[4]),
            sw.workspace(sw.sw_moe_layer_workspace_bytes(d, tokens), "cuda"))
    for phase in range(4):
        res = sw.sw_moe_layer(D["x"], D["wr"], top_k, w13, w2, layout=sw.TILED, route_out=bufs[0],
                              plan=bufs[1], out=bufs[2], ws=bufs[3], phase=phase)
    names = ("topk_ids", "topk_w", "gap", "plan", "out")
    assert_same_layer(dict(zip(names, whole)), dict(zip(names, res)))


def test_layer_call_in_band_flag_and_empty_batch(sw):
    # two eligible experts for top-3: the third slot is -1 on every token,
    # the plan built in the gate/up launch flags the batch (n_active -1, perm
    # the identity) and the output is NaN, as with the separate calls
    mask = np.zeros(8, np.uint8)
    mask[[1, 6]] = 1
    for tokens in (3, 40):
        cfg, L, D = small_layer(64, 8, 3, 32, tokens, seed=5)
        a = guarded_layer(sw, D, 3, mask=mask)
        b = guarded_layer(sw, D, 3, mask=mask, one_call=True)
        assert_same_layer(a, b)
        assert int(b["plan"].n_active.item()) == -1
        assert torch.equal(b["plan"].perm.cpu(), torch.arange(3 * tokens, dtype=torch.int32))
        assert bool(torch.all(torch.isnan(b["out"])))
    cfg, L, D = small_layer(64, 8, 2, 32, 4)
    ids, w, gap, plan, out = sw.sw_moe_layer(D["x"][:0], D["wr"], 2, D["w13"], D["w2"])
    assert ids.shape == (0, 2) and out.shape == (0, 64)
    assert int(plan.n_active.item()) == 0
    assert torch.all(plan.counts == 0) and torch.all(plan.offsets == 0)


# --------------------------------------------------------------------------
# the shared expert (Section 3.3)

def _shared_inputs(hidden, inter, tokens, seed):
    g = np.random.default_rng([301, seed])
    x = I.to_bf16_bits(g.standard_normal((tokens, hidden), dtype=np.float32))
    w13 = I.to_bf16_bits(0.02 * g.standard_normal((2 * inter, hidden), dtype=np.float32))
    w2 = I.to_bf16_bits(0.02 * g.standard_normal((hidden, inter), dtype=np.float32))
    gate = (0.05 * g.standard_normal(hidden)).astype(np.float32)
    base = g.standard_normal((tokens, hidden)).astype(np.float32)
    return x, w13, w2, gate, base


@pytest.mark.parametrize("hidden,inter,tokens", [(256, 128, 8), (2048, 1024, 64), (2048, 1024, 1),
                                                 (512, 256, 200), (2048, 1024, 17),
                                                 (2048, 1536, 100), (1024, 512, 300)])
def test_shared_expert_parity(sw, hidden, inter, tokens):
    x, w13, w2, gate, base = _shared_inputs(hidden, inter, tokens, hidden + tokens)
    out = dev(base)
    sw.sw_moe_shared_expert(dev(x), dev(w13[None]), dev(w2[None]), dev(gate), out)
    want = oracle.shared_expert(x, w13, w2, gate, out=base)
    err, rel = compare_out(host(out) - base, want - base, "shared expert term")
    print(f"shared H={hidden} I_s={inter} T={tokens}: max|err|={err:.3g} rel={rel:.3g}")
    if hidden <= 2048 and inter <= 1024:
        t13, t2 = sw.sw_moe_pack_experts(dev(w13[None]), dev(w2[None]))
        out_t = dev(base)
        sw.sw_moe_shared_expert(dev(x), t13, t2, dev(gate), out_t, layout=sw.TILED)
        assert torch.equal(out_t, out)


def test_shared_expert_zero_initialised_se2_is_se1_bit_for_bit(sw):
    x, w13a, w2a, gate, base = _shared_inputs(512, 128, 16, 5)
    _, w13b, _, _, _ = _shared_inputs(512, 128, 16, 6)
    i = 128
    w13 = np.concatenate([w13a[:i], w13b[:i], w13a[i:], w13b[i:]])
    w2 = np.concatenate([w2a, np.zeros_like(w2a)], axis=1)
    one = dev(base)
    sw.sw_moe_shared_expert(dev(x), dev(w13a[None]), dev(w2a[None]), dev(gate), one)
    merged = dev(base)
    sw.sw_moe_shared_expert(dev(x), dev(w13[None]), dev(w2[None]), dev(gate), merged)
    assert torch.equal(one, merged)


def _shared_parts(w13s, w2s, inter, n_shared):
    """The shared expert of width n_shared * I as n_shared experts of width I
    in the pool layout: part s = the gate and up rows of its intermediate
    units s*I .. (s+1)*I - 1, and the matching columns of its down
    projection."""
    isz = n_shared * inter
    p13 = np.stack([np.concatenate([w13s[s * inter:(s + 1) * inter],
                                    w13s[isz + s * inter:isz + (s + 1) * inter]])
                    for s in range(n_shared)])
    p2 = np.stack([np.ascontiguousarray(w2s[:, s * inter:(s + 1) * inter]) for s in range(n_shared)])
    return p13, p2


def _folded_layer(sw, L, w13s, w2s, gate, top_k, n_shared, mask, tiled, n_groups=1):
    inter = L["w2"].shape[2]
    p13, p2 = _shared_parts(w13s, w2s, inter, n_shared)
    # the pool: the routed experts, then n_groups copies of the parts
    w13 = dev(np.concatenate([L["w13"]] + [p13] * n_groups))
    w2 = dev(np.concatenate([L["w2"]] + [p2] * n_groups))
    layout = sw.ROW_MAJOR
    if tiled:
        w13, w2 = sw.sw_moe_pack_experts(w13, w2)
        layout = sw.TILED
    wr = dev(np.concatenate([L["wr"], gate[None]]))
    ids, w, gap, plan = sw.sw_moe_route_dispatch_shared(
        dev(L["x"]), wr, top_k, n_shared, n_groups=n_groups,
        keep_mask=None if mask is None else dev(mask))
    out = sw.sw_moe_forward(dev(L["x"]), w13, w2, w, plan, layout=layout)
    # the one-call layer with the folded expert writes the same bits
    one = sw.sw_moe_layer(dev(L["x"]), wr, top_k, w13, w2, layout=layout, n_shared=n_shared,
                          n_groups=n_groups, keep_mask=None if mask is None else dev(mask))
    assert_same_layer(dict(topk_ids=ids, topk_w=w, gap=gap, plan=plan, out=out),
                      dict(topk_ids=one[0], topk_w=one[1], gap=one[2], plan=one[3], out=one[4]))
    return ids, w, gap, plan, out


@pytest.mark.parametrize("hidden,n_experts,top_k,inter,tokens,n_shared,masked,tiled,groups", [
    (2048, 64, 8, 512, 64, 2, False, True, 1),    # batch 64: top-k, then dispatch;
                                                  # parts with every token (two passes)
    (2048, 64, 8, 512, 64, 2, False, True, 2),    # the same in two groups of 32 tokens
    (2048, 128, 8, 512, 1, 2, True, False, 1),    # one token: selection + plan in one block
    (2048, 128, 8, 512, 3, 2, True, False, 3),    # 3 groups of one token: the same
    (2048, 64, 8, 768, 17, 1, False, False, 1),   # 17 tokens: the row form, one part
    (2048, 64, 8, 768, 17, 1, False, True, 2),    # the row form, groups of 8 and 9
    (2048, 256, 8, 512, 100, 2, False, True, 1),  # 100 tokens: top-k, then dispatch
    (2048, 256, 8, 512, 100, 2, False, True, 4),  # four groups of 25 tokens
    (1024, 200, 14, 256, 40, 2, True, False, 3),  # k + parts = 16, 3 groups of 13 and 14
    (2048, 96, 6, 512, 200, 4, False, False, 1),  # 4 parts: 200-token parts over gate/up passes
    (2048, 128, 8, 512, 64, 2, False, True, 4),   # the shared-expert benchmark's shape: 128
                                                  # experts, 2 parts in 4 groups of 16 tokens
])
def test_shared_expert_folded_into_the_plan(sw, hidden, n_experts, top_k, inter, tokens, n_shared,
                                            masked, tiled, groups):
    # Section 3.3: the always-on shared expert behind a sigmoid gate, run as
    # n_shared extra experts every token routes to (token t to the parts of
    # copy t * groups // T)
    cfg, L, D = small_layer(hidden, n_experts, top_k, inter, tokens, seed=23)
    g = np.random.default_rng([401, hidden, tokens])
    isz = n_shared * inter
    w13s = I.to_bf16_bits(0.02 * g.standard_normal((2 * isz, hidden), dtype=np.float32))
    w2s = I.to_bf16_bits(0.02 * g.standard_normal((hidden, isz), dtype=np.float32))
    gate = (0.05 * g.standard_normal(hidden)).astype(np.float32)
    mask = mask_for(cfg, L, 0.5) if masked else None
    ids, w, gap, plan, out = _folded_layer(sw, L, w13s, w2s, gate, top_k, n_shared, mask, tiled,
                                           n_groups=groups)
    ids, w, gap = host(ids), host(w), host(gap)
    m, k = n_experts, top_k
    # routed slots: the oracle's routing rule; shared slots: every part, with
    # the sigmoid of the gate logit
    o_ids, o_w, o_gap, o_z = oracle.route(L["x"], L["wr"], k, keep_mask=mask, want_logits=True)
    compare_routing(ids[:, :k], w[:, :k], o_ids, o_w, o_z, mask, k, g_gap=gap, o_gap=o_gap,
                    what=f"folded shared T={tokens}")
    xf = I.bf16_bits_to_f32(L["x"]).astype(np.float64)
    sig = 1.0 / (1.0 + np.exp(-(xf @ gate.astype(np.float64))))
    copy = np.arange(tokens) * groups // tokens
    for s in range(n_shared):
        assert np.all(ids[:, k + s] == m + copy * n_shared + s)
        np.testing.assert_allclose(w[:, k + s], sig, rtol=0, atol=1e-6)
    counts, offsets, perm, active, n_active = oracle.dispatch(ids, m + groups * n_shared)
    np.testing.assert_array_equal(host(plan.counts), counts)
    np.testing.assert_array_equal(host(plan.offsets), offsets)
    np.testing.assert_array_equal(host(plan.perm)[: ids.size], perm)
    assert int(host(plan.n_active)[0]) == n_active
    np.testing.assert_array_equal(host(plan.active)[:n_active], active)
    # output: the routed layer plus the shared expert, as the oracle defines it
    o_out = oracle_forward_rows(oracle.forward, L["x"], L["w13"], L["w2"],
                                np.ascontiguousarray(ids[:, :k]), np.ascontiguousarray(w[:, :k]))
    o_out = oracle.shared_expert(L["x"], w13s, w2s, gate, out=o_out)
    err, rel = compare_out(host(out), o_out)
    print(f"folded shared H={hidden} m={m} k={k} I={inter} T={tokens} parts={n_shared} "
          f"groups={groups}: max|err|={err:.3g} rel={rel:.3g}")
    if groups > 1:
        # every copy holds the same weights: the output equals one copy's
        one = _folded_layer(sw, L, w13s, w2s, gate, top_k, n_shared, mask, tiled)
        assert torch.equal(out, one[4])


def test_folded_shared_expert_zero_se2_is_se1_bit_for_bit(sw):
    # SE2's down projection starts at zero (Section 3.3): its part adds +0 to
    # every output, so the folded SE1 + SE2 equals the folded SE1 alone
    cfg, L, D = small_layer(2048, 64, 8, 512, 48, seed=29)
    g = np.random.default_rng(31)
    w13s = I.to_bf16_bits(0.02 * g.standard_normal((2 * 1024, 2048), dtype=np.float32))
    w2s = I.to_bf16_bits(0.02 * g.standard_normal((2048, 1024), dtype=np.float32))
    w2s[:, 512:] = 0
    gate = (0.05 * g.standard_normal(2048)).astype(np.float32)
    se1_13 = np.concatenate([w13s[:512], w13s[1024:1536]])
    two = _folded_layer(sw, L, w13s, w2s, gate, 8, 2, None, True)
    one = _folded_layer(sw, L, se1_13, np.ascontiguousarray(w2s[:, :512]), gate, 8, 1, None, True)
    assert torch.equal(two[4], one[4])


# --------------------------------------------------------------------------
# routing-mass statistics (Section 2.3)

@pytest.mark.parametrize("hidden,m,k,tokens,masked,biased", [
    (256, 16, 2, 8, False, False),
    (2048, 64, 8, 64, False, False),
    (2048, 256, 8, 256, True, True),
    (512, 300, 8, 40, False, True),     # separate route + dispatch kernels
    (2048, 256, 8, 1024, False, False),
])
def test_routing_mass_parity(sw, hidden, m, k, tokens, masked, biased):
    cfg, L, D = small_layer(hidden, m, k, 32, tokens, seed=11)
    mask = mask_for(cfg, L, 0.5) if masked else None
    bias = (0.3 * np.random.default_rng(12).standard_normal(m)).astype(np.float32) if biased else None
    kw = dict(keep_mask=None if mask is None else dev(mask), bias=None if bias is None else dev(bias))
    ms, mt = sw.sw_moe_routing_mass(D["x"], D["wr"], k, **kw)
    o_ms, o_mt = oracle.routing_mass(L["x"], L["wr"], k, keep_mask=mask, bias=bias)
    np.testing.assert_allclose(host(ms), o_ms, rtol=1e-4, atol=1e-5)
    # near-tie tokens may route their k-th slot differently: allow their gates
    _, _, _, o_z = oracle.route(L["x"], L["wr"], k, keep_mask=mask, bias=bias, want_logits=True)
    from parity import near_tie_tokens
    n_near = int(near_tie_tokens(o_z, mask, k).sum())
    assert np.abs(host(mt) - o_mt).max() <= 1e-4 + n_near * 1.0
    assert abs(float(host(mt).sum()) - tokens) < 1e-3 * tokens
    # accumulation over a second batch
    sw.sw_moe_routing_mass(D["x"], D["wr"], k, mass=(ms, mt), **kw)
    np.testing.assert_allclose(host(ms), 2 * o_ms, rtol=2e-4, atol=2e-5)


def test_gpu_kept_sets_nest_and_match_the_oracle(sw):
    cfg, L, D = layer_inputs("decode_sweep")
    prev = None
    for p in (0.75, 0.5, 0.25):
        g = sw.sw_moe_prune_compact(D["importance"], cfg.n_keep(p), cfg.top_k, compact=False,
                                    hidden=cfg.hidden)
        kept = set(host(g["kept"]).tolist())
        assert kept == set(oracle.prune_compact(L["importance"], cfg.n_keep(p), cfg.top_k)[0].tolist())
        if prev is not None:
            assert prev < kept
        prev = kept
