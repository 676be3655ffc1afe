"""GPU parity: the HIP path, called through the C ABI, against the fp64 CPU oracle on the
same seeded inputs.  Index sets must match exactly (a position may differ only where the
oracle's scores tie within 1e-4 relative); bf16 outputs must satisfy
|gpu - oracle| <= 2e-2 + 1e-2 * |oracle|."""
import numpy as np
import pytest
import torch

from oracle import lychee_oracle as lo
from paper_2602_04541_amd import workloads as wl
from tests import gpu_harness as H
from tests.test_launch_plan import plan  # noqa: F401  (a fixture: the rules that lay out a launch)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def _shared_ctx():
    lb = H.binding()
    c = lb.Context(0)
    yield c
    c.close()


@pytest.fixture
def ctx(_shared_ctx):
    """One context for the module; every test starts from, and leaves behind, the library's
    default options (the ones bench.py runs with)."""
    lb = H.binding()
    _shared_ctx.set_option(lb.OPT_DEFAULTS, 0)
    yield _shared_ctx
    _shared_ctx.set_option(lb.OPT_DEFAULTS, 0)


@pytest.fixture
def own_ctx():
    """A context for one test: its counts of waits that gave up and of rows ranked whole start at zero."""
    c = H.binding().Context(0)
    yield c
    c.close()


def _say(msg):
    print(msg, flush=True)


# ------------------------------------------------------------------ configuration 1
def test_c1_small_layer(ctx):
    w = wl.WORKLOADS["c1"]
    inp = wl.make_layer(w)
    idx_in = H.previous_layer_sets(inp, w.k)
    _say("c1: B1 8q/2kv L4096 k256 mask=%s" % inp.mask.tolist())
    _, _, idx_gpu, _, _, _ = H.check_layer(ctx, inp, inp.mask, w.k, idx_in, "c1")
    for g in range(w.n_kv_heads):
        assert np.isin(inp.planted_pos[0, g], idx_gpu[0, g]).all()


# -------------------------------------------------- tiles, ragged tails, edge sizes
EDGE = [
    # (B, Hq, Hkv, L_cap, lengths, k, mask-kind)
    (1, 4, 1, 1, [1], 1, "all_r"),
    (1, 4, 1, 5, [5], 3, "mixed"),
    (2, 8, 2, 80, [17, 80], 16, "mixed"),
    (1, 8, 2, 63, [63], 63, "mixed"),          # k == L
    (1, 8, 2, 64, [64], 100, "mixed"),         # k > L: -1 padding
    (3, 4, 4, 300, [65, 300, 129], 32, "mixed"),   # G = 1
    (2, 4, 2, 1000, [999, 1000], 128, "all_s"),    # G = 2, no retrieval head at all
    (1, 8, 2, 1537, [1537], 257, "all_r"),
    (2, 8, 2, 2100, [2049, 1], 300, "one_r"),      # a length-1 sequence in the batch
    (1, 12, 4, 777, [700], 64, "mixed"),           # G = 3, cache longer than the sequence
]


def _mask(kind, Hq, rng):
    if kind == "all_r":
        return np.ones(Hq, np.uint8)
    if kind == "all_s":
        return np.zeros(Hq, np.uint8)
    if kind == "one_r":
        m = np.zeros(Hq, np.uint8)
        m[int(rng.integers(0, Hq))] = 1
        return m
    m = (rng.random(Hq) < 0.4).astype(np.uint8)
    m[0], m[-1] = 1, 0
    return m


@pytest.mark.parametrize("case", EDGE, ids=lambda c: "B%d_Hq%d_Hkv%d_L%d_k%d_%s" % (c[0], c[1], c[2], c[3], c[5], c[6]))
def test_edge_shapes(ctx, case):
    B, Hq, Hkv, l_cap, lens, k, kind = case
    rng = np.random.default_rng(l_cap * 31 + k)
    w = wl.scaled(wl.WORKLOADS["c1"], batch=B, n_q_heads=Hq, n_kv_heads=Hkv, max_len=l_cap, k=k,
                  planted=min(8, min(lens)), retrieval_heads=())
    mask = _mask(kind, Hq, rng)
    inp = wl.make_layer(w, mask=mask, lens=np.asarray(lens, np.int32), l_cap=l_cap)
    idx_in = None if kind == "all_r" else H.previous_layer_sets(inp, k)
    _say("edge %s mask=%s" % (case, mask.tolist()))
    H.check_layer(ctx, inp, mask, k, idx_in, "edge%s" % (case,))


@pytest.mark.parametrize("block", [1, 64])
@pytest.mark.parametrize("n_wg", [0, 2])
@pytest.mark.parametrize("Hkv,G", [(2, 1), (1, 2), (2, 3), (1, 4)])
def test_pieces_of_a_few_tiles(ctx, Hkv, G, n_wg, block):
    """Layer calls whose streamed and gathered pieces end at the edges of a wavefront's tile of 16 rows and of one
    and two blocks of 64 (on a grid of two workgroups a segment is a piece), with a set of which some entries name
    nothing."""
    rng = np.random.default_rng(100 * Hkv + G)
    ctx.set_option(H.binding().OPT_N_WG, n_wg)
    for L, k in ((1, 1), (15, 15), (16, 3), (17, 16), (31, 17), (48, 47), (49, 33), (63, 64), (64, 64), (65, 63), (129, 65),
                 (150, 80), (200, 81), (128, 127), (128, 128), (300, 129)):
        k = -(-k // block)
        w = wl.scaled(wl.WORKLOADS["c1"], n_q_heads=Hkv * G, n_kv_heads=Hkv, max_len=L, k=k, planted=min(8, L),
                      retrieval_heads=())
        mask = (rng.random(Hkv * G) < 0.5).astype(np.uint8)
        mask[0], mask[-1] = 1, 0
        inp = wl.make_layer(w, mask=mask, lens=np.asarray([L], np.int32), l_cap=L)
        idx_in = H.previous_layer_sets(inp, k, block=block)
        _say("short pieces %dx%d L=%d k=%d block %d" % (Hkv, G, L, k, block))
        H.check_layer(ctx, inp, mask, k, idx_in, "L=%d k=%d" % (L, k), block=block)
        if block == 1 and k > 2:  # (entries that name nothing leave the outputs of the set without them)
            few = idx_in[:, :, :k - 2].copy()
            junk = idx_in.copy()
            junk[:, :, k - 2:] = (-1, 10 ** 6)
            out_few, _ = H.run_hybrid(ctx, H.DeviceLayer(inp, k - 2, few), mask)
            out_junk, _ = H.run_hybrid(ctx, H.DeviceLayer(inp, k, junk), mask)
            H.assert_outputs_close(out_junk, out_few, "ignored entries, L=%d k=%d" % (L, k))
        if block == 1:
            H.check_prob_rule_layer(ctx, inp, mask, k, 2, 0.8, "top-p L=%d k=%d" % (L, k), idx_in)


def test_inherited_sets_in_any_order_and_with_ignored_entries(ctx):
    """idx_in need not be sorted; negative and out-of-range entries are skipped."""
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=900, k=96, planted=8)
    inp = wl.make_layer(w, l_cap=900)
    rng = np.random.default_rng(5)
    idx_sorted = H.previous_layer_sets(inp, w.k)
    idx_in = idx_sorted[:, :, rng.permutation(w.k)].copy()
    idx_in[0, 0, 90:] = -1
    mask = np.zeros(w.n_q_heads, np.uint8)
    dl, out_gpu, idx_gpu, out_ref, _, _ = H.check_layer(ctx, inp, mask, w.k, idx_in, "unsorted")
    # the same set with junk entries appended behaves like the clean set
    junk = np.concatenate([idx_in, np.full((1, w.n_kv_heads, 32), 10 ** 6, np.int32)], axis=2)
    junk[0, 1, -5:] = -3
    dl2 = H.DeviceLayer(inp, w.k + 32, junk)
    out2, idx2 = H.run_hybrid(ctx, dl2, mask)
    assert (out2 == out_gpu).all()
    assert (idx2 == junk).all()


def test_token_major_cache_layout(ctx):
    """Strides are honoured: the same cache stored as [B][L][H_kv][128]."""
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=1300, k=64, planted=8)
    inp = wl.make_layer(w, l_cap=1300)
    idx_in = H.previous_layer_sets(inp, w.k)
    dl = H.DeviceLayer(inp, w.k, idx_in)
    out_a, idx_a = H.run_hybrid(ctx, dl, inp.mask)
    lb = H.binding()
    k_tm = dl.k_cache.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)   # same values, token-major
    v_tm = dl.v_cache.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    assert k_tm.stride(2) == w.n_kv_heads * 128
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 1300, w.k, kv=k_tm)
    out_b = torch.zeros_like(dl.out)
    idx_b = torch.zeros_like(dl.idx_out)
    ctx.decode_attn(shape, dl.q, k_tm, v_tm, inp.mask, dl.idx_in, out_b, idx_b, dl.lengths,
                    dl.workspace)
    torch.cuda.synchronize()
    assert (H.bf16_tensor_to_f64(out_b) == out_a).all() and (idx_b.cpu().numpy() == idx_a).all()


# ------------------------------------------------------------------ ties (duplicated keys)
def test_duplicated_key_rows_break_ties_towards_the_lower_position(ctx):
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=6000, k=300, planted=16)
    inp = wl.make_layer(w, l_cap=6000)
    # sources: planted rows, and rows whose score straddles the k-th score
    _, idx0, sel0 = H.oracle_layer(inp, np.ones(w.n_q_heads, np.uint8), w.k, None)
    src = np.zeros((1, w.n_kv_heads, 12), np.int64)
    for g in range(w.n_kv_heads):
        order = np.argsort(-sel0[0, g, :6000], kind="stable")
        src[0, g] = np.concatenate([inp.planted_pos[0, g, :4], order[w.k - 4:w.k + 4]])
    wl.plant_ties(inp, 1500, src)
    mask = inp.mask
    idx_in = H.previous_layer_sets(inp, w.k)
    _say("ties: 1500 duplicated key rows per KV head")
    H.check_layer(ctx, inp, mask, w.k, idx_in, "ties", exact_sets=True)
    H.check_layer(ctx, inp, np.ones(w.n_q_heads, np.uint8), w.k, None, "ties_all_r", exact_sets=True)


def test_all_keys_identical(ctx):
    """Every score ties: the set is the first k positions, the output the mean of V."""
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=5000, k=77, planted=0)
    inp = wl.make_layer(w, l_cap=5000)
    inp.k_cache[:] = inp.k_cache[:, :, :1, :]
    mask = np.ones(w.n_q_heads, np.uint8)
    _, _, idx_gpu, _, _, _ = H.check_layer(ctx, inp, mask, w.k, None, "identical", exact_sets=True)
    assert (idx_gpu[0, 0] == np.arange(77)).all()


# ------------------------------------------------------------------ dense baseline
@pytest.mark.parametrize("lens", [[4096], [1], [333, 2048, 31]])
def test_dense_kernel_matches_oracle(ctx, lens):
    B = len(lens)
    w = wl.scaled(wl.WORKLOADS["c1"], batch=B, max_len=max(lens), planted=min(8, min(lens)))
    inp = wl.make_layer(w, lens=np.asarray(lens, np.int32), l_cap=max(lens))
    dl = H.DeviceLayer(inp, w.k, None)
    got = H.run_dense(ctx, dl)
    ref = lo.dense_attn(wl.bf16_bits(inp.q), wl.bf16_bits(inp.k_cache), wl.bf16_bits(inp.v_cache),
                        inp.lengths)
    H.assert_outputs_close(got, ref, "dense%s" % lens)


def test_sparse_with_full_set_equals_dense_kernel(ctx):
    """Eq. 3 with the set of all positions is Eq. 1: gather path == streaming path."""
    L = 3000
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=L, k=L, planted=8)
    inp = wl.make_layer(w, l_cap=L)
    full = np.tile(np.arange(L, dtype=np.int32), (1, w.n_kv_heads, 1))
    dl = H.DeviceLayer(inp, L, full)
    sparse, _ = H.run_hybrid(ctx, dl, np.zeros(w.n_q_heads, np.uint8))
    dense = H.run_dense(ctx, dl)
    ref = lo.dense_attn(wl.bf16_bits(inp.q), wl.bf16_bits(inp.k_cache), wl.bf16_bits(inp.v_cache),
                        inp.lengths)
    H.assert_outputs_close(sparse, ref, "sparse_full")
    H.assert_outputs_close(dense, ref, "dense")
    assert np.abs(sparse - dense).max() <= 2 ** -6     # both are bf16 roundings of the same value


# ------------------------------------------------------------------ splits and determinism
def test_result_does_not_depend_on_the_grid_size_and_is_deterministic(ctx):
    lb = H.binding()
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=5000, k=700, planted=16)
    inp = wl.make_layer(w, l_cap=5000)
    idx_in = H.previous_layer_sets(inp, w.k)
    out_ref, idx_ref, sel_ref = H.oracle_layer(inp, inp.mask, w.k, idx_in)
    dl = H.DeviceLayer(inp, w.k, idx_in)
    results = []
    try:
        for wg_per_cu, n_wg, gb, tail in [(2, 0, 48, 250), (1, 0, 48, 0), (3, 0, 16, 1000), (2, 37, 128, 500),
                                          (2, 1, 64, 150), (2, 0, 48, 250)]:
            ctx.set_option(lb.OPT_WG_PER_CU, wg_per_cu)
            ctx.set_option(lb.OPT_N_WG, n_wg)
            ctx.set_option(lb.OPT_GATHER_BLOCK, gb)
            ctx.set_option(lb.OPT_TAIL_PERMILLE, tail)
            out, idx = H.run_hybrid(ctx, dl, inp.mask)
            what = "wg_per_cu=%d n_wg=%d gather_block=%d tail=%d" % (wg_per_cu, n_wg, gb, tail)
            H.assert_outputs_close(out, out_ref, what)
            H.assert_sets_match(idx, idx_ref, sel_ref, inp.mask, inp, w.k, idx_in, what)
            results.append((out, idx))
    finally:
        ctx.set_option(lb.OPT_DEFAULTS, 0)
    for out, idx in results[1:]:
        assert (idx == results[0][1]).all()              # scores do not depend on the split
        assert np.abs(out - results[0][0]).max() <= 2 ** -6
    assert (results[0][0] == results[-1][0]).all()       # same configuration: bit-identical


# ------------------------------------------------------------------ configuration 2
def test_c2_llama_shaped_layer(ctx):
    w = wl.WORKLOADS["c2"]
    inp = wl.make_layer(w, device="cuda")
    idx_in = H.previous_layer_sets(inp, w.k)
    _say("c2: 32q/8kv L32768 k2048 retrieval heads %s" % np.flatnonzero(inp.mask).tolist())
    _, _, idx_gpu, _, _, _ = H.check_layer(ctx, inp, inp.mask, w.k, idx_in, "c2")
    G = w.group
    for g in range(w.n_kv_heads):
        if inp.mask[g * G:(g + 1) * G].any():
            assert np.isin(inp.planted_pos[0, g], idx_gpu[0, g]).all()


# ------------------------------------------------------------------ configuration 4
def test_c4_batched_ragged(ctx):
    w = wl.WORKLOADS["c4"]
    inp = wl.make_layer(w, device="cuda")
    _say("c4: lengths %s" % inp.lengths.tolist())
    idx_in = H.previous_layer_sets(inp, w.k)
    H.check_layer(ctx, inp, inp.mask, w.k, idx_in, "c4")


# ------------------------------------------------------------------ decode step (chaining)
@pytest.mark.parametrize("mode", ["phased", "layerwise"])
def test_decode_step_chains_sets_through_layers(ctx, mode):
    lb = H.binding()
    n_layers = 6
    w = wl.scaled(wl.WORKLOADS["c3"], max_len=4096, k=256, n_layers=n_layers, planted=64)
    layers = [wl.make_layer(w, layer=l, device="cuda", l_cap=4096) for l in range(n_layers)]
    masks = np.stack([ly.mask for ly in layers])
    assert masks[0].all() and masks[1:].sum(1).tolist() == [3] * (n_layers - 1)
    # oracle chain
    idx = None
    refs = []
    for ly in layers:
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, w.k, idx)
        refs.append((out_ref, idx, sel_ref))
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 4096, w.k, kv=layers[0].k_cache)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    idx_final = torch.full((w.batch, w.n_kv_heads, w.k), -9, dtype=torch.int32, device="cuda")
    lens = torch.from_numpy(layers[0].lengths).cuda()
    ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED if mode == "phased" else lb.STEP_LAYERWISE)
    try:
        for rep in range(2):    # the second step reuses a workspace full of the first one's data
            ctx.decode_step(shape, [ly.q for ly in layers], [ly.k_cache for ly in layers],
                            [ly.v_cache for ly in layers], masks, None, outs, idx_final, lens, ws)
            torch.cuda.synchronize()
    finally:
        ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED)
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "step layer %d" % l)
    # the final sets: groups that selected in the last layer are checked against its scores,
    # the others must equal the oracle chain's sets (which came from earlier layers)
    last = layers[-1]
    G = w.group
    got = idx_final.cpu().numpy()
    for g in range(w.n_kv_heads):
        if last.mask[g * G:(g + 1) * G].any():
            ok, _, msg = H.index_sets_match(got[0, g], refs[-1][1][0, g], refs[-1][2][0, g, :4096],
                                            w.k, H.TIE_REL)
            assert ok, msg
        else:
            assert (got[0, g] == refs[-1][1][0, g]).all()


def test_decode_step_with_given_sets_and_ragged_batch(ctx):
    """Layer 0 is a hybrid layer fed by caller-supplied sets; batch of 3 ragged sequences."""
    lb = H.binding()
    n_layers = 5
    w = wl.scaled(wl.WORKLOADS["c4"], batch=3, max_len=3000, k=200, n_layers=n_layers, planted=32,
                  len_lo=700, len_hi=3000)
    lens_h = wl.lengths(w)
    layers = [wl.make_layer(w, layer=l, device="cuda", lens=lens_h, l_cap=3000) for l in range(n_layers)]
    masks = np.stack([ly.mask for ly in layers])
    idx0 = H.previous_layer_sets(layers[0], w.k)
    idx = idx0
    refs = []
    for ly in layers:
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, w.k, idx)
        refs.append((out_ref, idx, sel_ref))
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 3000, w.k, kv=layers[0].k_cache)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    lens = torch.from_numpy(lens_h).cuda()
    ctx.decode_step(shape, [ly.q for ly in layers], [ly.k_cache for ly in layers],
                    [ly.v_cache for ly in layers], masks, torch.from_numpy(idx0).cuda(), outs, None,
                    lens, ws)
    torch.cuda.synchronize()
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "ragged step layer %d" % l)


def test_phased_step_skips_partials_without_a_row(ctx):
    """A piece whose set entries are all -1 has no row and weight 0.  The rows it re-reads in their place hold
    an infinity, and must not reach the output of heads whose sets do not name them."""
    lb = H.binding()
    n_layers, L, k, used = 2, 3000, 1024, 256
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=L, k=k, n_layers=n_layers, planted=8)
    mask = np.zeros(w.n_q_heads, np.uint8)
    inp = wl.make_layer(w, mask=mask, l_cap=L)
    idx = np.full((1, w.n_kv_heads, k), -1, np.int32)
    rng = np.random.default_rng(4)
    for g in range(w.n_kv_heads):
        idx[0, g, :used] = np.sort(rng.choice(np.arange(1, L), size=used, replace=False))
    out_ref, _, _ = H.oracle_layer(inp, mask, used, np.ascontiguousarray(idx[:, :, :used]))
    dl = H.DeviceLayer(inp, k, idx)
    dl.v_cache[:, :, 0, ::3] = float("inf")
    ws = lb.alloc_workspace(dl.shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs = [torch.full_like(dl.out, float("nan")) for _ in range(n_layers)]
    _say("phased step: sets of %d entries of which %d name a row" % (k, used))
    ctx.set_option(lb.OPT_GATHER_BLOCK, 128)      # (whole spans: the pieces with rows re-read nothing)
    ctx.decode_step(dl.shape, [dl.q] * n_layers, [dl.k_cache] * n_layers, [dl.v_cache] * n_layers,
                    np.stack([mask] * n_layers), dl.idx_in, outs, None, dl.lengths, ws)
    torch.cuda.synchronize()
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), out_ref, "layer %d" % l)


@pytest.mark.parametrize("G,n_wg,l_cap,split", [(4, 52, 400, 2), (4, 51, 400, 1), (4, 28, 400, 1), (4, 27, 400, 0), (4, 16, 50000, 2),
                                                (4, 15, 50000, 0), (3, 28, 400, 1), (2, 7, 400, 0), (1, 5, 400, 2)])
def test_phased_steps_on_either_side_of_how_their_merges_are_dealt(ctx, plan, G, n_wg, l_cap, split):
    """Three layers of two sequences and two KV heads: a head, a kind of heads or a KV head a unit, in one round and in
    several, and the dense step beside it."""
    lb = H.binding()
    n_layers, B, Hkv, k = 3, 2, 2, 40
    slots = -(-l_cap // 64) // max(8, -(-(-(-l_cap // 64)) // 192)) + 2
    assert plan.merge_split(n_layers * B * Hkv, G, 1, B * Hkv, slots, n_wg) == split
    rng = np.random.default_rng(G)
    masks = np.concatenate([np.ones((1, Hkv * G), np.uint8), (rng.random((n_layers - 1, Hkv * G)) < 0.4).astype(np.uint8)])
    lens = np.asarray([300, 50], np.int32)
    w = wl.scaled(wl.WORKLOADS["c4"], batch=B, n_q_heads=Hkv * G, n_kv_heads=Hkv, max_len=l_cap, k=k, n_layers=n_layers, planted=6)
    layers = [wl.make_layer(w, layer=l, device="cuda", mask=masks[l], lens=lens, l_cap=l_cap) for l in range(n_layers)]
    shape = lb.make_shape(B, Hkv * G, Hkv, l_cap, k, kv=layers[0].k_cache)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs, dense = ([torch.full_like(ly.q, float("nan")) for ly in layers] for _ in range(2))
    idx_final = torch.full((B, Hkv, k), -9, dtype=torch.int32, device="cuda")
    args = [[getattr(ly, name) for ly in layers] for name in ("q", "k_cache", "v_cache")]
    lens_d = torch.from_numpy(lens).cuda()
    ctx.set_option(lb.OPT_N_WG, n_wg)
    _say("phased step, groups of %d heads, %d workgroups" % (G, n_wg))
    ctx.decode_step(shape, *args, masks, None, outs, idx_final, lens_d, ws)
    ctx.dense_decode_step(shape, *args, dense, lens_d, ws)
    torch.cuda.synchronize()
    idx = None
    for l, ly in enumerate(layers):
        out_ref, idx, _ = H.oracle_layer(ly, masks[l], k, idx)
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), out_ref, "layer %d" % l)
        H.assert_outputs_close(H.bf16_tensor_to_f64(dense[l]), H.oracle_layer(ly, np.ones_like(masks[l]), k, None)[0], "dense %d" % l)


# ------------------------------------------------------------------ boundary behaviour
def test_error_codes_and_index_validator(ctx):
    lb = H.binding()
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=512, k=32, planted=4)
    inp = wl.make_layer(w, l_cap=512)
    idx_in = H.previous_layer_sets(inp, w.k)
    dl = H.DeviceLayer(inp, w.k, idx_in)

    def code(fn):
        try:
            fn()
        except lb.LycheeError as e:
            return e.code
        return 0

    args = lambda **kw: dict(dict(shape=dl.shape, q=dl.q, k_cache=dl.k_cache, v_cache=dl.v_cache,
                                  head_type_mask=inp.mask, idx_in=dl.idx_in, out=dl.out,
                                  idx_out=dl.idx_out, lengths=dl.lengths, workspace=dl.workspace), **kw)
    assert code(lambda: ctx.decode_attn(**args())) == 0
    assert code(lambda: ctx.decode_attn(**args(idx_in=None))) == lb.EINVAL        # sparse heads, no set
    assert code(lambda: ctx.decode_attn(**args(idx_out=dl.idx_in))) == lb.EINVAL  # aliasing
    assert code(lambda: ctx.decode_attn(**args(workspace=dl.workspace[:1024]))) == lb.EWORKSPACE
    assert code(lambda: ctx.decode_attn(**args(workspace=dl.workspace[3:]))) == lb.EWORKSPACE
    assert code(lambda: ctx.decode_attn(**args(q=dl.q.view(-1)[1:]))) == lb.EINVAL  # misaligned
    bad = lb.make_shape(1, 8, 2, 512, 32, head_dim=64)
    assert code(lambda: ctx.decode_attn(**args(shape=bad))) == lb.EUNSUPPORTED
    torch.cuda.synchronize()
    _, idx_gpu = H.run_hybrid(ctx, dl, inp.mask)
    assert ctx.validate_idx(dl.shape, dl.idx_out, dl.lengths) == 0
    broken = dl.idx_out.clone()
    broken[0, 0, 3] = broken[0, 0, 2]      # a duplicate
    broken[0, 1, 0] = 512                  # out of range
    assert ctx.validate_idx(dl.shape, broken, dl.lengths) == 2


# ------------------------------------------------------------------ configuration 3, full size
@pytest.mark.parametrize("layer", [0, 1, 17, 35])
def test_c3_full_size_single_layers(ctx, layer):
    """Teacher-forced: a 128K Qwen3-8B-shaped layer with the oracle's sets as idx_in."""
    w = wl.WORKLOADS["c3"]
    inp = wl.make_layer(w, layer=layer, device="cuda")
    idx_in = None if inp.mask.all() else H.previous_layer_sets(inp, w.k)
    _say("c3 layer %d: retrieval heads %s" % (layer, np.flatnonzero(inp.mask).tolist()))
    _, _, idx_gpu, _, _, _ = H.check_layer(ctx, inp, inp.mask, w.k, idx_in, "c3 layer %d" % layer)
    G = w.group
    for g in range(w.n_kv_heads):
        if inp.mask[g * G:(g + 1) * G].any():       # k = 4096 holds all 1024 planted rows
            assert np.isin(inp.planted_pos[0, g], idx_gpu[0, g]).all()


def test_c3_full_decode_step_in_the_benchmarked_configuration(ctx):
    """The whole 36-layer 128K step with the library's default options, against ONE oracle chain:
    (a) exactly as bench.py times it - lychee_decode_step layer after layer, one launch per layer -,
        every layer's output and the final sets;
    (b) the same free-running chain as 36 lychee_decode_attn_deferred calls and a flush, which
        expose EVERY layer's sets: each is compared with the oracle's set of that layer, and a
        difference is only accepted where the oracle's scores tie (none is expected);
    (c) the phased step (all queries given before the step), outputs and final sets."""
    lb = H.binding()
    w = wl.WORKLOADS["c3"]
    n_layers = w.n_layers
    layers = [wl.make_layer(w, layer=l, device="cuda") for l in range(n_layers)]
    masks = np.stack([ly.mask for ly in layers])
    lens_h = layers[0].lengths
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, w.max_len, w.k, kv=layers[0].k_cache)
    lens = torch.from_numpy(lens_h).cuda()
    G = w.group
    # the oracle chain, one layer on the host at a time
    refs = []
    idx = None
    for l, ly in enumerate(layers):
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, w.k, idx)
        refs.append((out_ref, idx.copy(), {g: sel_ref[0, g, :w.max_len].copy() for g in range(w.n_kv_heads)
                                           if ly.mask[g * G:(g + 1) * G].any()}))
    last_sel = {}
    for l in range(n_layers):
        last_sel.update(refs[l][2])

    def check_outputs(outs, what):
        worst = 0.0
        for l in range(n_layers):
            worst = max(worst, H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "%s layer %d" % (what, l)))
        _say("c3 %s: worst abs output error %.4g" % (what, worst))

    def check_final(got, what):
        for g in range(w.n_kv_heads):
            ok, n_diff, msg = H.index_sets_match(got[0, g], refs[-1][1][0, g], last_sel[g], w.k, H.TIE_REL)
            assert ok, "%s: final set of KV head %d: %s" % (what, g, msg)
            assert (np.diff(got[0, g]) > 0).all()

    qs, ks, vs = [ly.q for ly in layers], [ly.k_cache for ly in layers], [ly.v_cache for ly in layers]
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    for mode, what in ((lb.STEP_LAYERWISE, "step, layer after layer"), (lb.STEP_PHASED, "phased step")):
        outs = [torch.zeros_like(ly.q) for ly in layers]
        idx_final = torch.full((w.batch, w.n_kv_heads, w.k), -9, dtype=torch.int32, device="cuda")
        ctx.set_option(lb.OPT_STEP_MODE, mode)
        ctx.decode_step(shape, qs, ks, vs, masks, None, outs, idx_final, lens, ws)
        torch.cuda.synchronize()
        check_outputs(outs, what)
        check_final(idx_final.cpu().numpy(), what)
    del ws
    # (b) layer calls that leave their select pending: every layer's sets are visible
    ws2 = lb.alloc_workspace(shape, n_layers=2)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    sets = [torch.full((w.batch, w.n_kv_heads, w.k), -9, dtype=torch.int32, device="cuda") for _ in layers]
    for l, ly in enumerate(layers):
        ctx.decode_attn_deferred(shape, ly.q, ly.k_cache, ly.v_cache, ly.mask, sets[l - 1] if l else None,
                                 outs[l], sets[l], lens, ws2)
    ctx.select_flush()
    torch.cuda.synchronize()
    check_outputs(outs, "layer calls")
    n_diff_total = 0
    for l, ly in enumerate(layers):
        got = sets[l].cpu().numpy()
        for g in range(w.n_kv_heads):
            if g in refs[l][2]:
                ok, n_diff, msg = H.index_sets_match(got[0, g], refs[l][1][0, g], refs[l][2][g], w.k, H.TIE_REL)
                assert ok, "layer %d, KV head %d: %s" % (l, g, msg)
                assert (np.diff(got[0, g]) > 0).all()
                n_diff_total += n_diff
            else:
                assert (got[0, g] == refs[l][1][0, g]).all(), "layer %d, KV head %d: inherited set not handed on" % (l, g)
    assert n_diff_total == 0, "%d positions differ from the oracle's sets (inside its ties)" % n_diff_total
    assert ctx.wait_timeouts() == 0, "a bounded wait inside a layer launch gave up"


# ------------------------------------------------------------------ configuration 5: sweep
@pytest.mark.parametrize("n_retrieval", [1, 4, 32])
@pytest.mark.parametrize("k", [64, 1024, 8192, 131072])
def test_c5_budget_and_retrieval_fraction_sweep_with_ties(ctx, k, n_retrieval):
    w = wl.scaled(wl.WORKLOADS["c5"], k=k, n_retrieval=n_retrieval)
    rng = np.random.default_rng(k + n_retrieval)
    if n_retrieval == 32:
        mask = np.ones(32, np.uint8)
    elif n_retrieval == 4:
        mask = wl.head_type_mask(w, 0)
    else:
        mask = np.zeros(32, np.uint8)
        mask[int(rng.integers(0, 32))] = 1
    inp = wl.make_layer(w, device="cuda", mask=mask)
    # mass ties: 4096 key rows per KV head become copies of a few source rows (planted rows
    # and rows spread over the score range), V untouched
    src = np.stack([np.concatenate([inp.planted_pos[0, g, :8],
                                    rng.choice(w.max_len, size=24, replace=False)])
                    for g in range(w.n_kv_heads)])[None]
    wl.plant_ties(inp, 4096, src)
    if k >= w.max_len:
        idx_in = np.tile(np.arange(w.max_len, dtype=np.int32), (1, w.n_kv_heads, 1))
    else:
        idx_in = H.previous_layer_sets(inp, k)
    if n_retrieval == 32:
        idx_in = None
    _say("c5 k=%d retrieval heads %s" % (k, np.flatnonzero(mask).tolist()))
    dl, out_gpu, idx_gpu, out_ref, idx_ref, _ = H.check_layer(ctx, inp, mask, k, idx_in, "c5 k=%d r=%d" % (k, n_retrieval))
    if k >= w.max_len:
        # the full set: sparse heads must equal the dense kernel's result for those heads
        dense = H.run_dense(ctx, dl)
        assert np.abs(dense - out_gpu).max() <= 2 ** -6
        for g in range(w.n_kv_heads):
            if mask[g * 4:(g + 1) * 4].any():
                assert (idx_gpu[0, g] == np.arange(w.max_len)).all()


@pytest.mark.parametrize("mode", ["phased", "layerwise"])
def test_dense_decode_step(ctx, mode):
    lb = H.binding()
    n_layers = 3
    w = wl.scaled(wl.WORKLOADS["c4"], batch=2, max_len=2500, k=16, n_layers=n_layers, planted=16,
                  len_lo=900, len_hi=2500)
    lens_h = wl.lengths(w)
    layers = [wl.make_layer(w, layer=l, device="cuda", lens=lens_h, l_cap=2500) for l in range(n_layers)]
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 2500, w.k, kv=layers[0].k_cache)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED if mode == "phased" else lb.STEP_LAYERWISE)
    try:
        ctx.dense_decode_step(shape, [ly.q for ly in layers], [ly.k_cache for ly in layers],
                              [ly.v_cache for ly in layers], outs, torch.from_numpy(lens_h).cuda(), ws)
        torch.cuda.synchronize()
    finally:
        ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED)
    for l, ly in enumerate(layers):
        ref = lo.dense_attn(wl.bf16_bits(ly.q), wl.bf16_bits(ly.k_cache), wl.bf16_bits(ly.v_cache), lens_h)
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), ref, "dense step layer %d" % l)


# ------------------------------------------------------------------ every route of the select
@pytest.mark.parametrize("margin,route", [(60, "candidates in registers"),
                                          (1250, "candidates read from memory"),
                                          (-1000, "too few candidates: whole row ranked"),
                                          (100000, "list overflow: whole row ranked")])
def test_select_routes_give_the_same_sets(ctx, margin, route):
    """The sampled threshold only decides how the exact top-k is computed, never its result:
    the margin option drives the select through each of its routes."""
    lb = H.binding()
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=40000, k=500, planted=16)
    inp = wl.make_layer(w, l_cap=40000)
    _, _, sel0 = H.oracle_layer(inp, np.ones(w.n_q_heads, np.uint8), w.k, None)
    src = np.zeros((1, w.n_kv_heads, 8), np.int64)
    for g in range(w.n_kv_heads):
        order = np.argsort(-sel0[0, g, :40000], kind="stable")
        src[0, g] = order[w.k - 4:w.k + 4]     # duplicates of rows around the k-th score
    wl.plant_ties(inp, 3000, src)
    _say("select route: %s (margin %d)" % (route, margin))
    few0, many0 = ctx.select_stats()
    ctx.set_option(lb.OPT_SELECT_MARGIN, margin)
    try:
        H.check_layer(ctx, inp, np.ones(w.n_q_heads, np.uint8), w.k, None, route, exact_sets=True)
        H.check_layer(ctx, inp, inp.mask, w.k, H.previous_layer_sets(inp, w.k), route, exact_sets=True)
    finally:
        ctx.set_option(lb.OPT_SELECT_MARGIN, 60)
    few, many = ctx.select_stats()
    # 2 score rows in the all-retrieval call, those of the masked call on top
    n_rows = 2 + sum(1 for g in range(w.n_kv_heads) if inp.mask[g * w.group:(g + 1) * w.group].any())
    assert (few - few0, many - many0) == {60: (0, 0), 1250: (0, 0), -1000: (n_rows, 0), 100000: (0, n_rows)}[margin]


@pytest.mark.parametrize("L,k,copies", [
    (4096, 1, 0), (4096, 64, 63), (4096, 65, 70),   # every row a candidate; 64 and more equal keys at the cut
    (8191, 4096, 0), (8192, 4096, 500),             # the last list that is held in registers
    (8193, 4097, 500),                              # the first one that is read from memory
    (16500, 8250, 100),                             # more positions than are staged at a time
    (40000, 4096, 300), (65537, 2048, 0),           # sampled rows: the smaller and the larger sample
    (131072, 96, 0), (131073, 96, 70),              # the last row of a bitmap window, the first of the next
])
def test_select_at_the_edges_of_its_routes(ctx, L, k, copies):
    """The same sets from a plain call (which selects in its one launch) and from a deferred one (a later
    launch selects), against the oracle, with no position allowed to differ."""
    lb = H.binding()
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=L, k=k, planted=16)
    inp = wl.make_layer(w, l_cap=L)
    ones = np.ones(w.n_q_heads, np.uint8)
    if copies:
        _, _, sel0 = H.oracle_layer(inp, ones, k, None)
        src = np.zeros((1, w.n_kv_heads, 1), np.int64)
        for g in range(w.n_kv_heads):
            src[0, g, 0] = np.argsort(-sel0[0, g, :L], kind="stable")[k - 1]  # rows equal to the last one in
        wl.plant_ties(inp, copies, src)
    _say("select edge: L=%d k=%d copies=%d" % (L, k, copies))
    dl, _, idx, _, _, _ = H.check_layer(ctx, inp, ones, k, None, "L=%d k=%d" % (L, k), exact_sets=True)
    ws = lb.alloc_workspace(dl.shape, "cuda", n_layers=2)
    ws.fill_(0xFF)
    dl.idx_out.fill_(-7)
    ctx.decode_attn_deferred(dl.shape, dl.q, dl.k_cache, dl.v_cache, ones, None, dl.out, dl.idx_out, dl.lengths, ws)
    ctx.select_flush()
    torch.cuda.synchronize()
    assert (dl.idx_out.cpu().numpy() == idx).all()


@pytest.mark.parametrize("n_wg,L,k", [
    (0, 4097, 2048), (0, 20000, 1), (0, 32768, 3900), (0, 32768, 4100),  # thresholds by one unit and by four
    (0, 65, 3), (0, 129, 40),                       # pieces of one block and of a part of one
    (18, 8193, 100), (18, 16384, 700),              # pieces around 1024 and 2048 rows: one or two wavefronts filter
    (12, 16700, 900), (10, 33000, 300),             # around 4096: the last window of keys full, short, the second one
])
def test_pieces_filter_their_keys_at_the_edges_of_a_wavefronts_share(ctx, n_wg, L, k):
    """Plain and deferred calls of one sequence whose pieces end at the edges of what a wavefront filters, on grids
    that make them so long: the oracle's sets, with no position allowed to differ."""
    lb = H.binding()
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=L, k=k, planted=1)
    mask = np.zeros(w.n_q_heads, np.uint8)
    mask[[0, 5]] = 1
    inp = wl.make_layer(w, mask=mask, l_cap=L)
    idx_in = H.previous_layer_sets(inp, k)
    _say("filter edge: n_wg=%d L=%d k=%d" % (n_wg, L, k))
    ctx.set_option(lb.OPT_N_WG, n_wg)
    dl, _, idx, _, _, _ = H.check_layer(ctx, inp, mask, k, idx_in, "L=%d k=%d" % (L, k), exact_sets=True)
    ws = lb.alloc_workspace(dl.shape, "cuda", n_layers=2)
    ws.fill_(0xFF)
    dl.idx_out.fill_(-7)
    ctx.decode_attn_deferred(dl.shape, dl.q, dl.k_cache, dl.v_cache, mask, dl.idx_in, dl.out, dl.idx_out, dl.lengths, ws)
    ctx.select_flush()
    torch.cuda.synchronize()
    assert (dl.idx_out.cpu().numpy() == idx).all()
    assert ctx.wait_timeouts() == 0


@pytest.mark.parametrize("lens,Hkv,k,block,n_wg,tail", [
    # four and five rows on 64 workgroups, four on 63
    ([4099], 4, 300, 1, 64, 4), ([4099], 5, 300, 1, 64, 0), ([4099], 4, 300, 1, 63, 0),
    # 32 and 33 rows; segments of one piece
    ([700, 65, 1, 64], 8, 40, 1, 0, 32), ([700, 65, 1] * 11, 1, 40, 1, 0, 0),
    # too many rows; one row, at any length
    ([40000] * 2, 4, 900, 1, 64, 0), ([40000], 1, 900, 1, 64, 1),
    # four rows whose streaming is short enough for that, and one block too long
    ([65536], 4, 900, 1, 64, 4), ([65537], 4, 900, 1, 64, 0),
    # the set is everything; blocks
    ([65], 8, 200, 1, 0, 8), ([9000, 63, 130], 2, 9, 64, 0, 6),
])
def test_layer_calls_whose_rows_are_selected_at_the_end_of_the_grid(ctx, plan, lens, Hkv, k, block, n_wg, tail):
    """On both sides of the rule that gives a launch's score rows workgroups of their own: the oracle's sets, twice
    in a row (the second call finds the counters as the first left them)."""
    lb = H.binding()
    w = wl.scaled(wl.WORKLOADS["c1"], batch=len(lens), n_q_heads=2 * Hkv, n_kv_heads=Hkv, max_len=max(lens), k=k, planted=1)
    inp = wl.make_layer(w, mask=np.tile(np.array([1, 0], np.uint8), Hkv), lens=np.asarray(lens, np.int32), l_cap=max(lens))
    idx_in = H.previous_layer_sets(inp, k, block=block)
    _say("selects at the end: B%d rows=%d k=%d block=%d n_wg=%d" % (len(lens), len(lens) * Hkv, k, block, n_wg))
    rows = len(lens) * Hkv   # (the default grid is two workgroups per compute unit)
    grid = n_wg or 2 * torch.cuda.get_device_properties(0).multi_processor_count
    assert plan.tail_selects(rows, rows * -(-max(lens) // 64), grid) == tail
    ctx.set_option(lb.OPT_N_WG, n_wg)
    dl, out, idx, _, _, _ = H.check_layer(ctx, inp, inp.mask, k, idx_in, exact_sets=True, block=block)
    dl.out.fill_(float("nan"))
    dl.idx_out.fill_(-7)
    out2, idx2 = H.run_hybrid(ctx, dl, inp.mask)
    assert (out2 == out).all() and (idx2 == idx).all()
    assert ctx.wait_timeouts() == 0


@pytest.mark.parametrize("call", ["plain", "deferred"])
def test_a_list_that_a_piece_gave_up_on_is_not_selected_from(own_ctx, call):
    """One of a row's pieces gives up on the row's threshold, the others do not: what they list is more than the
    budget, but the best rows are the ones that are missing.  Nine workgroups take runs of 64 blocks of two segments of
    257 and 309 (and five each for a piece's fixed cost); the first segment's last block is a run's first piece,
    over long before the threshold is out, and the 40 rows in it are the highest-scoring ones."""
    lb, ctx = H.binding(), own_ctx
    lens, k = [256 * 64 + 40, 309 * 64], 300
    w = wl.scaled(wl.WORKLOADS["c1"], batch=2, n_q_heads=2, n_kv_heads=1, max_len=max(lens), k=k, planted=1)
    mask = np.ones(2, np.uint8)
    inp = wl.make_layer(w, mask=mask, lens=np.asarray(lens, np.int32), l_cap=max(lens))
    best = slice(256 * 64, lens[0])
    inp.k_cache[0, 0, best] = inp.q[0].float().sum(0).to(inp.k_cache.dtype)
    ref = H.oracle_layer(inp, mask, k, None)
    assert np.isin(np.arange(best.start, best.stop), ref[1][0, 0]).all()
    dl = H.DeviceLayer(inp, k, None)
    ws = lb.alloc_workspace(dl.shape, "cuda", n_layers=2)
    ctx.set_option(lb.OPT_N_WG, 12)
    for polls in (1, 1 << 20):
        _say("a piece without its threshold: %s polls=%d" % (call, polls))
        ctx.set_option(lb.OPT_WAIT_POLLS, polls)
        ws.fill_(0xFF)
        dl.out.fill_(float("nan"))
        dl.idx_out.fill_(-7)
        fallbacks = sum(ctx.select_stats())
        f = ctx.decode_attn_deferred if call == "deferred" else ctx.decode_attn
        f(dl.shape, dl.q, dl.k_cache, dl.v_cache, mask, None, dl.out, dl.idx_out, dl.lengths, ws)
        ctx.select_flush()
        torch.cuda.synchronize()
        H.assert_outputs_close(H.bf16_tensor_to_f64(dl.out), ref[0], "polls=%d" % polls)
        assert (dl.idx_out.cpu().numpy() == ref[1]).all(), "polls=%d" % polls
        if polls == 1:
            gave_up = ctx.wait_timeouts()
            assert gave_up > 0 and sum(ctx.select_stats()) > fallbacks
        else:  # (the counter is back at zero, whatever was left in it)
            assert ctx.wait_timeouts() == gave_up and sum(ctx.select_stats()) == fallbacks


@pytest.mark.parametrize("lens,k,block,rule,param", [
    ([4096, 3000, 4000, 2500], 200, 1, 0, 0.0),      # rows whose threshold is known
    ([20000, 9000], 500, 1, 0, 0.0),                 # and rows whose pieces give up on it too
    ([4096, 3000, 4000, 2500], 200, 1, 1, 1e-3), ([20000, 9000], 500, 1, 2, 0.8),
    ([20000, 9000, 131, 4096], 30, 64, 0, 0.0),
])
def test_rows_that_the_end_of_the_grid_gives_up_on(own_ctx, lens, k, block, rule, param):
    """The workgroups at the end of the grid give up on their rows at once, and the pieces that complete the rows select
    them: the oracle's sets, and the same from the next call, whose waits last, with nothing ranked whole in it."""
    lb, ctx = H.binding(), own_ctx
    w = wl.scaled(wl.WORKLOADS["c1"], batch=len(lens), n_q_heads=2, n_kv_heads=1, max_len=max(lens), k=k, planted=1)
    mask = np.array([1, 0], np.uint8)
    inp = wl.make_layer(w, mask=mask, lens=np.asarray(lens, np.int32), l_cap=max(lens))
    idx_in = H.previous_layer_sets(inp, k, block=block)
    ctx.set_option(lb.OPT_N_WG, 64)
    for polls in (0, 1 << 20):
        _say("rows given up on: B%d k=%d block=%d rule=%d polls=%d" % (len(lens), k, block, rule, polls))
        ctx.set_option(lb.OPT_WAIT_POLLS, polls)
        fallbacks = sum(ctx.select_stats())
        if rule:
            H.check_prob_rule_layer(ctx, inp, mask, k, rule, param, "polls=%d" % polls, idx_in)
        else:
            H.check_layer(ctx, inp, mask, k, idx_in, "polls=%d" % polls, exact_sets=True, block=block)
        if polls == 0:
            gave_up = ctx.wait_timeouts()
            assert gave_up > 0
    assert ctx.wait_timeouts() == gave_up and sum(ctx.select_stats()) == fallbacks


@pytest.mark.parametrize("lens,k,block", [
    ([61, 3001, 200, 1] * 20, 300, 1),       # runs that cross many short segments; set copies by every workgroup
    ([61, 3001, 200, 1] * 20, 5, 64),
    ([9000, 4097, 20000, 64] * 6, 1024, 1),  # front units in turn on few workgroups beside a long stream
])
def test_layer_calls_of_batches_whose_runs_cross_segments(ctx, lens, k, block):
    """Ragged batches in one launch each, sets included: heads that keep theirs, single-piece segments that
    write their output directly, and rows whose set is selected by the workgroup that completes them."""
    w = wl.scaled(wl.WORKLOADS["c1"], batch=len(lens), max_len=max(lens), k=k, planted=1)
    mask = np.zeros(w.n_q_heads, np.uint8)
    mask[1] = 1                                   # the second KV head keeps its sets
    inp = wl.make_layer(w, mask=mask, lens=np.array(lens, np.int32), l_cap=max(lens) + 3)
    idx_in = H.previous_layer_sets(inp, k, block=block)
    _say("batch of %d, longest %d, k=%d, block %d" % (len(lens), max(lens), k, block))
    H.check_layer(ctx, inp, mask, k, idx_in, "batch", exact_sets=True, block=block)


def test_a_layer_call_in_a_cache_far_larger_than_its_sequences(ctx):
    """Which workgroups run the front units follows from the lengths on the device: the same batch, in a cache
    with room for ten times its rows, gives the same sets, and outputs that another split may round otherwise."""
    lens = [5000, 9000, 4097, 300] * 10
    w = wl.scaled(wl.WORKLOADS["c1"], batch=len(lens), n_q_heads=8, n_kv_heads=4, max_len=max(lens), k=700, planted=4,
                  retrieval_heads=(0, 2, 4))
    inp = wl.make_layer(w, lens=np.array(lens, np.int32), l_cap=max(lens), device="cuda")
    idx_in = H.previous_layer_sets(inp, w.k)
    _say("batch of %d in caches of %d and %d rows" % (len(lens), max(lens), 10 * max(lens)))
    _, out, idx, _, _, _ = H.check_layer(ctx, inp, inp.mask, w.k, idx_in, "snug", exact_sets=True)
    for name in ("k_cache", "v_cache"):
        rows = getattr(inp, name)
        roomy = torch.full((w.batch, w.n_kv_heads, 10 * max(lens), 128), 50.0, dtype=torch.bfloat16, device="cuda")
        roomy[:, :, :max(lens)] = rows
        setattr(inp, name, roomy)
    dl = H.DeviceLayer(inp, w.k, idx_in)
    out2, idx2 = H.run_hybrid(ctx, dl, inp.mask)
    assert (idx2 == idx).all()
    H.assert_outputs_close(out2, out, "roomy")


def test_sequence_longer_than_one_bitmap_window(ctx):
    """The ordered write marks positions in windows of 131072: a longer sequence needs two."""
    w = wl.scaled(wl.WORKLOADS["c1"], n_q_heads=2, n_kv_heads=1, max_len=150000, k=700, planted=32)
    inp = wl.make_layer(w, l_cap=150000, mask=np.ones(2, np.uint8))
    _say("two bitmap windows: L 150000")
    _, _, idx_gpu, _, _, _ = H.check_layer(ctx, inp, np.ones(2, np.uint8), w.k, None, "two windows")
    assert (idx_gpu[0, 0] >= 131072).any() and (idx_gpu[0, 0][:10] < 131072).all()


# ------------------------------------------------------------------ the Ratio rule (Sec. 4.4.1)
@pytest.mark.parametrize("keep_ppm", [300000, 100000, 1000, 1000000])
def test_ratio_rule_layer_with_ragged_batch(ctx, keep_ppm):
    """A budget proportional to each sequence's length, in sets of capacity k."""
    w = wl.scaled(wl.WORKLOADS["c4"], batch=3, max_len=9000, k=3000, planted=16, len_lo=300, len_hi=9000)
    lens_h = wl.lengths(w)
    inp = wl.make_layer(w, lens=lens_h, l_cap=9000)
    _say("ratio rule: keep %d ppm of lengths %s" % (keep_ppm, lens_h.tolist()))
    mask = np.ones(w.n_q_heads, np.uint8)
    _, _, idx_gpu, _, _, _ = H.check_layer(ctx, inp, mask, w.k, None, "ratio all-retrieval", keep_ppm=keep_ppm)
    for b in range(w.batch):
        want = min(w.k, int(lens_h[b]), max(1, -(-int(lens_h[b]) * keep_ppm // 1000000)))
        assert ((idx_gpu[b] >= 0).sum(axis=1) == want).all()
    # a hybrid layer whose sparse heads inherit sets of the same rule
    _, idx_prev, _ = H.oracle_layer(inp, mask, w.k, None, keep_ppm)
    H.check_layer(ctx, inp, inp.mask, w.k, idx_prev, "ratio hybrid", keep_ppm=keep_ppm)


def test_ratio_rule_decode_step(ctx):
    lb = H.binding()
    n_layers, keep_ppm = 4, 200000
    w = wl.scaled(wl.WORKLOADS["c3"], max_len=20000, k=4096, n_layers=n_layers, planted=64)
    layers = [wl.make_layer(w, layer=l, device="cuda", l_cap=20000) for l in range(n_layers)]
    masks = np.stack([ly.mask for ly in layers])
    idx = None
    refs = []
    for ly in layers:
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, w.k, idx, keep_ppm)
        refs.append((out_ref, idx, sel_ref))
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 20000, w.k, kv=layers[0].k_cache,
                          keep_ppm=keep_ppm)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    idx_final = torch.full((w.batch, w.n_kv_heads, w.k), -9, dtype=torch.int32, device="cuda")
    lens = torch.from_numpy(layers[0].lengths).cuda()
    _say("ratio rule: 4-layer phased step, 20 % of 20000 rows")
    ctx.decode_step(shape, [ly.q for ly in layers], [ly.k_cache for ly in layers],
                    [ly.v_cache for ly in layers], masks, None, outs, idx_final, lens, ws)
    torch.cuda.synchronize()
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "ratio step layer %d" % l)
    got = idx_final.cpu().numpy()
    assert ((got[0] >= 0).sum(axis=1) == 4000).all()
    G = w.group
    for g in range(w.n_kv_heads):
        if layers[-1].mask[g * G:(g + 1) * G].any():
            ok, _, msg = H.index_sets_match(got[0, g], refs[-1][1][0, g], refs[-1][2][0, g, :20000], 4000, H.TIE_REL)
            assert ok, msg
        else:
            assert (got[0, g] == refs[-1][1][0, g]).all()


# ------------------------------------------------------------------ block-granular sets (App. C)
BLOCK_CASES = [
    # B, Hq, Hkv, L_cap, lens, k (blocks), mask kind
    (1, 8, 2, 4096, [4096], 8, "c1"),
    (1, 8, 2, 4096, [4096], 64, "all_r"),        # k = every block
    (2, 8, 2, 3000, [3000, 1111], 10, "mixed"),  # ragged last blocks
    (3, 12, 4, 900, [900, 64, 65], 3, "mixed"),  # one block exactly, one row into the second block
    (1, 4, 1, 20000, [19999], 100, "one_r"),
]


@pytest.mark.parametrize("case", BLOCK_CASES, ids=lambda c: "B%d_Hq%d_Hkv%d_L%d_k%d_%s" % (c[0], c[1], c[2], c[3], c[5], c[6]))
def test_block_granular_layers(ctx, case):
    B, Hq, Hkv, L_cap, lens, k, kind = case
    rng = np.random.default_rng(5)
    w = wl.scaled(wl.WORKLOADS["c1"], batch=B, n_q_heads=Hq, n_kv_heads=Hkv, max_len=L_cap, k=k, planted=8)
    mask = {"c1": None, "all_r": np.ones(Hq, np.uint8), "one_r": np.eye(1, Hq, 0, dtype=np.uint8)[0]}.get(kind)
    if kind == "mixed":
        mask = (rng.random(Hq) < 0.4).astype(np.uint8)
        mask[0] = 1
    if mask is None:
        mask = wl.head_type_mask(w)
    inp = wl.make_layer(w, mask=mask, lens=np.array(lens, np.int32), l_cap=L_cap)
    _say("block-granular layer %s" % (case,))
    idx_in = H.previous_layer_sets(inp, k, block=64)
    H.check_layer(ctx, inp, mask, k, idx_in, "block %s" % kind, block=64)
    H.check_layer(ctx, inp, np.ones(Hq, np.uint8), k, None, "block all-retrieval", block=64)


def test_block_granular_sets_with_ties_and_scattered_entries(ctx):
    """Tied best tokens in different blocks go to the lower block; inherited sets may come
    in any order, with -1 anywhere and with blocks that lie past the sequence."""
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=8192, k=16, planted=0)
    inp = wl.make_layer(w, l_cap=8192)
    _, _, sel0 = H.oracle_layer(inp, np.ones(8, np.uint8), 16, None, block=64)
    for g in range(2):
        best = np.argsort(-sel0[0, g, :8192], kind="stable")[:40]
        for t in best[:20]:                          # copies of strong rows into other blocks
            inp.k_cache[0, g, (int(t) + 64 * 31) % 8192] = inp.k_cache[0, g, int(t)]
    H.check_layer(ctx, inp, np.ones(8, np.uint8), 16, None, "block ties", exact_sets=True, block=64)
    idx_in = H.previous_layer_sets(inp, 16, block=64)
    rng = np.random.default_rng(3)
    for g in range(2):
        row = idx_in[0, g].copy()
        gone = rng.choice(16, 5, replace=False)
        row[gone] = -1
        row[gone[0]] = 1000                          # a block past the 128 blocks of the sequence
        row[gone[1]] = 2 ** 25 + 3 + g               # times 64 this wraps around 32 bits: still ignored
        row[gone[2]] = 2 ** 31 - 1
        rng.shuffle(row)
        idx_in[0, g] = row
    dl = H.DeviceLayer(inp, 16, idx_in, block=64)
    out_gpu, idx_gpu = H.run_hybrid(ctx, dl, inp.mask)
    # the oracle wants valid entries first: same sets, compacted
    idx_ref_in = np.full_like(idx_in, -1)
    for g in range(2):
        v = idx_in[0, g][(idx_in[0, g] >= 0) & (idx_in[0, g] < 128)]
        idx_ref_in[0, g, :v.size] = v
    out_ref, _, _ = H.oracle_layer(inp, inp.mask, 16, idx_ref_in, block=64)
    H.assert_outputs_close(out_gpu, out_ref, "block scattered sets")


@pytest.mark.parametrize("mode", ["phased", "layerwise"])
def test_block_granular_decode_step(ctx, mode):
    lb = H.binding()
    n_layers, k = 5, 12
    w = wl.scaled(wl.WORKLOADS["c3"], max_len=6000, k=k, n_layers=n_layers, planted=32)
    layers = [wl.make_layer(w, layer=l, device="cuda", l_cap=6000) for l in range(n_layers)]
    masks = np.stack([ly.mask for ly in layers])
    idx = None
    refs = []
    for ly in layers:
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, k, idx, block=64)
        refs.append((out_ref, idx, sel_ref))
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 6000, k, kv=layers[0].k_cache, block_size=64)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    idx_final = torch.full((w.batch, w.n_kv_heads, k), -9, dtype=torch.int32, device="cuda")
    lens = torch.from_numpy(layers[0].lengths).cuda()
    _say("block-granular %s step" % mode)
    ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED if mode == "phased" else lb.STEP_LAYERWISE)
    try:
        ctx.decode_step(shape, [ly.q for ly in layers], [ly.k_cache for ly in layers],
                        [ly.v_cache for ly in layers], masks, None, outs, idx_final, lens, ws)
        torch.cuda.synchronize()
    finally:
        ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED)
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "block step layer %d" % l)
    got = idx_final.cpu().numpy()
    G = w.group
    for g in range(w.n_kv_heads):
        if layers[-1].mask[g * G:(g + 1) * G].any():
            ok, _, msg = H.index_sets_match(got[0, g], refs[-1][1][0, g],
                                            H.unit_scores(refs[-1][2][0, g], 6000, 64), k, H.TIE_REL)
            assert ok, msg
        else:
            assert (got[0, g] == refs[-1][1][0, g]).all()


# ------------------------------------------------------------------ the cache append of Alg. 1
def test_block_granular_set_of_a_row_with_a_partial_last_block(ctx):
    """More blocks than the list of a smaller row holds, and the last of them a single position."""
    L, k = 2000001, 204
    w = wl.scaled(wl.WORKLOADS["c1"], n_q_heads=1, n_kv_heads=1, max_len=L, k=k, planted=8, retrieval_heads=(0,))
    inp = wl.make_layer(w, mask=np.ones(1, np.uint8), l_cap=L, device="cuda")
    inp.k_cache[0, 0, L - 1] = inp.k_cache[0, 0, int(inp.planted_pos[0, 0, 0])]
    _say("block-granular sets: %d positions in %d blocks" % (L, -(-L // 64)))
    _, _, idx_gpu, _, _, _ = H.check_layer(ctx, inp, inp.mask, k, None, "L=%d" % L, exact_sets=True, block=64)
    assert idx_gpu[0, 0].max() == (L - 1) // 64


@pytest.mark.parametrize("token_major", [False, True])
def test_append_kv_writes_exactly_the_new_rows(ctx, token_major):
    lb = H.binding()
    B, Hkv, L_cap = 3, 4, 500
    lens_h = np.array([500, 1, 263], np.int32)
    g = torch.Generator().manual_seed(77)
    def cache():
        t = torch.randn((B, L_cap, Hkv, 128) if token_major else (B, Hkv, L_cap, 128), generator=g).to(torch.bfloat16)
        return t.cuda().permute(0, 2, 1, 3) if token_major else t.cuda()
    K, V = cache(), cache()
    kn = torch.randn((B, Hkv, 128), generator=g).to(torch.bfloat16).cuda()
    vn = torch.randn((B, Hkv, 128), generator=g).to(torch.bfloat16).cuda()
    K_ref, V_ref = wl.bf16_bits(K).copy(), wl.bf16_bits(V).copy()
    lo_mod = H.lo
    lo_mod.append_kv(wl.bf16_bits(kn), wl.bf16_bits(vn), K_ref, V_ref, lens_h)
    shape = lb.make_shape(B, 4 * Hkv, Hkv, L_cap, 16, kv=K)
    _say("append_kv, token_major=%s" % token_major)
    ctx.append_kv(shape, kn, vn, K, V, torch.from_numpy(lens_h).cuda())
    torch.cuda.synchronize()
    assert (wl.bf16_bits(K) == K_ref).all() and (wl.bf16_bits(V) == V_ref).all()


@pytest.mark.parametrize("mode,block", [("phased", 1), ("layerwise", 1), ("phased", 64), ("layerwise", 64)])
def test_decode_step_with_the_append_inside(ctx, mode, block):
    lb = H.binding()
    n_layers = 4
    k = 8 if block == 64 else 300
    w = wl.scaled(wl.WORKLOADS["c3"], batch=2, max_len=5000, k=k, n_layers=n_layers, planted=32,
                  len_lo=4200, len_hi=5000)
    lens_h = wl.lengths(w)
    layers = [wl.make_layer(w, layer=l, device="cuda", lens=lens_h, l_cap=5000) for l in range(n_layers)]
    masks = np.stack([ly.mask for ly in layers])
    # the new token's rows are taken out of the generated caches; the caches get stale rows there
    k_new, v_new = [], []
    for ly in layers:
        kn = torch.stack([ly.k_cache[b, :, int(lens_h[b]) - 1] for b in range(w.batch)]).contiguous()
        vn = torch.stack([ly.v_cache[b, :, int(lens_h[b]) - 1] for b in range(w.batch)]).contiguous()
        k_new.append(kn)
        v_new.append(vn)
    idx = None
    refs = []
    for ly in layers:                       # the oracle sees the caches with the rows in place
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, k, idx, block=block)
        refs.append((out_ref, idx, sel_ref))
    want_k = [wl.bf16_bits(ly.k_cache).copy() for ly in layers]
    for ly in layers:
        for b in range(w.batch):
            ly.k_cache[b, :, int(lens_h[b]) - 1] = 7.0       # what a missing append would leave behind
            ly.v_cache[b, :, int(lens_h[b]) - 1] = -7.0
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 5000, k, kv=layers[0].k_cache, block_size=block)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    lens = torch.from_numpy(lens_h).cuda()
    _say("decode step with append: %s, block %d" % (mode, block))
    ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED if mode == "phased" else lb.STEP_LAYERWISE)
    try:
        ctx.decode_step_append(shape, [ly.q for ly in layers], k_new, v_new, [ly.k_cache for ly in layers],
                               [ly.v_cache for ly in layers], masks, None, outs, None, lens, ws)
        torch.cuda.synchronize()
    finally:
        ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED)
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "append step layer %d" % l)
        assert (wl.bf16_bits(layers[l].k_cache) == want_k[l]).all()


# ------------------------------------------------------------------ HIP graph capture and replay
@pytest.mark.parametrize("mode,block", [("phased", 1), ("phased", 64), ("layerwise", 1)])
def test_a_captured_decode_step_replays_correctly(ctx, mode, block):
    """The step's launches (and, phased, its one table upload) are captured into a graph and
    replayed with new queries in the same buffers; every replay must equal the eager step."""
    lb = H.binding()
    ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED if mode == "phased" else lb.STEP_LAYERWISE)
    n_layers = 10
    k = 30 if block == 64 else 1500
    # many layers of a medium length: the pooled streaming launch then hands out dynamic chunks,
    # i.e. it uses a chunk counter, which a replay must find at zero again
    w = wl.scaled(wl.WORKLOADS["c3"], max_len=20000, k=k, n_layers=n_layers, planted=64)
    layers = [wl.make_layer(w, layer=l, device="cuda", l_cap=20000) for l in range(n_layers)]
    masks = np.stack([ly.mask for ly in layers])
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 20000, k, kv=layers[0].k_cache, block_size=block)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    qs = [ly.q.clone() for ly in layers]
    outs = [torch.zeros_like(ly.q) for ly in layers]
    idx_final = torch.full((w.batch, w.n_kv_heads, k), -9, dtype=torch.int32, device="cuda")
    lens = torch.from_numpy(layers[0].lengths).cuda()

    def step():
        ctx.decode_step(shape, qs, [ly.k_cache for ly in layers], [ly.v_cache for ly in layers], masks,
                        None, outs, idx_final, lens, ws)

    step()                                   # eager once: uploads the table, warms everything
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.synchronize()
    gen = torch.Generator(device="cuda").manual_seed(5)
    for rep in range(3):
        _say("graph replay %d, %s, block %d" % (rep, mode, block))
        for qt in qs:                        # new queries in the captured buffers
            qt.copy_(torch.randn(qt.shape, generator=gen, device="cuda").to(torch.bfloat16))
        for o in outs:
            o.zero_()
        idx_final.fill_(-9)
        graph.replay()
        torch.cuda.synchronize()
        got_out = [o.clone() for o in outs]
        got_idx = idx_final.clone()
        step()                               # the program's own eager work between replays
        torch.cuda.synchronize()
        for l in range(n_layers):
            assert torch.equal(got_out[l], outs[l]), "replay %d layer %d differs from the eager step" % (rep, l)
        assert torch.equal(got_idx, idx_final)
    # and the eager result is the oracle's (last queries)
    idx = None
    for l, ly in enumerate(layers):
        ly.q.copy_(qs[l])
        out_ref, idx, _ = H.oracle_layer(ly, ly.mask, k, idx, block=block)
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), out_ref, "graph step layer %d" % l)


def _arena_case(n_layers=48):
    lb = H.binding()
    w = wl.scaled(wl.WORKLOADS["c3"], max_len=1024, k=64, n_layers=n_layers, planted=16)
    layers = [wl.make_layer(w, layer=l, device="cuda", l_cap=1024) for l in range(n_layers)]
    masks = np.stack([ly.mask for ly in layers])
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 1024, w.k, kv=layers[0].k_cache)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    lens = torch.from_numpy(layers[0].lengths).cuda()
    idx_final = torch.full((w.batch, w.n_kv_heads, w.k), -9, dtype=torch.int32, device="cuda")
    return lb, w, layers, masks, shape, ws, lens, idx_final


def test_descriptor_arena_recycles_after_many_distinct_buffer_sets():
    """Phased steps keep their layer descriptors in a 4 MiB arena of the context.  Steps whose
    output buffers differ each need a table of their own: after a few hundred the arena starts
    over (the call waits for the stream once).  Every step, before and after that, must still
    give the first step's result."""
    lb, w, layers, masks, shape, ws, lens, idx_final = _arena_case()
    n_layers = len(layers)
    c = lb.Context(0)
    try:
        c.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED)
        n_sets = 300                        # tables of 49 descriptors, about 45 KB each: the arena holds some 90
        pool = torch.zeros((n_sets, n_layers) + tuple(layers[0].q.shape), dtype=torch.bfloat16, device="cuda")
        args = ([ly.q for ly in layers], [ly.k_cache for ly in layers], [ly.v_cache for ly in layers], masks, None)
        first_idx = None
        for i in range(n_sets):
            if i % 100 == 0:
                _say("arena: step %d" % i)
            c.decode_step(shape, *args, [pool[i, l] for l in range(n_layers)], idx_final, lens, ws)
            if i == 0:
                torch.cuda.synchronize()
                first_idx = idx_final.clone()
        torch.cuda.synchronize()
        assert torch.equal(idx_final, first_idx)
        same = (pool == pool[0:1]).flatten(1).all(1)
        assert bool(same.all()), "steps %s differ from the first" % torch.nonzero(~same).flatten().tolist()[:8]
        out_ref, _, _ = H.oracle_layer(layers[0], layers[0].mask, w.k, None)
        H.assert_outputs_close(H.bf16_tensor_to_f64(pool[n_sets - 1, 0]), out_ref, "layer 0 of the last step")
    finally:
        c.close()


def test_descriptor_arena_is_not_recycled_under_a_captured_graph():
    """A captured graph points into the arena for as long as it lives.  Once a capture has seen
    the arena, a call that would have to recycle it returns LYCHEE_EARENA instead, and the graph
    still replays correctly."""
    lb, w, layers, masks, shape, ws, lens, idx_final = _arena_case()
    n_layers = len(layers)
    c = lb.Context(0)
    try:
        c.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED)
        args = ([ly.q for ly in layers], [ly.k_cache for ly in layers], [ly.v_cache for ly in layers], masks, None)
        outs = [torch.zeros_like(ly.q) for ly in layers]
        c.decode_step(shape, *args, outs, idx_final, lens, ws)
        torch.cuda.synchronize()
        want = [o.clone() for o in outs]
        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            with torch.cuda.graph(graph, stream=side):
                c.decode_step(shape, *args, outs, idx_final, lens, ws)
        torch.cuda.synchronize()
        pool = torch.zeros((300, n_layers) + tuple(layers[0].q.shape), dtype=torch.bfloat16, device="cuda")
        refused = None
        for i in range(300):
            try:
                c.decode_step(shape, *args, [pool[i, l] for l in range(n_layers)], idx_final, lens, ws)
            except lb.LycheeError as e:
                refused = (i, e.code)
                break
        torch.cuda.synchronize()
        assert refused is not None and refused[1] == lb.EARENA and refused[0] > 50, refused
        _say("arena: refused at step %d" % refused[0])
        for o in outs:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for l in range(n_layers):
            assert torch.equal(outs[l], want[l]), "replay after the refusal differs at layer %d" % l
        # the tables already resident still serve their calls
        c.decode_step(shape, *args, [pool[0, l] for l in range(n_layers)], idx_final, lens, ws)
        torch.cuda.synchronize()
        assert torch.equal(pool[0, 3], want[3])
    finally:
        c.close()


def test_ratio_rule_counts_blocks_with_block_granular_sets(ctx):
    w = wl.scaled(wl.WORKLOADS["c4"], batch=2, max_len=12000, k=100, planted=16, len_lo=3000, len_hi=12000)
    lens_h = wl.lengths(w)
    inp = wl.make_layer(w, lens=lens_h, l_cap=12000)
    mask = np.ones(w.n_q_heads, np.uint8)
    _say("ratio rule on blocks: a quarter of the blocks of lengths %s" % lens_h.tolist())
    _, _, idx_gpu, _, _, _ = H.check_layer(ctx, inp, mask, w.k, None, "ratio blocks", keep_ppm=250000, block=64)
    for b in range(w.batch):
        units = -(-int(lens_h[b]) // 64)
        assert ((idx_gpu[b] >= 0).sum(axis=1) == min(w.k, -(-units * 250000 // 1000000))).all()
    _, idx_prev, _ = H.oracle_layer(inp, mask, w.k, None, 250000, 64)
    H.check_layer(ctx, inp, inp.mask, w.k, idx_prev, "ratio blocks hybrid", keep_ppm=250000, block=64)



def test_scores_that_come_in_runs_do_not_mislead_the_threshold(ctx):
    """Rows that matter are consecutive in real contexts.  All the best rows sit in a few runs of
    hundreds of rows here; the sets must be exact and no score row may need the whole-row ranking."""
    w = wl.scaled(wl.WORKLOADS["c5"], n_q_heads=8, n_kv_heads=2, n_retrieval=0, retrieval_heads=(0, 5), k=4096)
    inp = wl.make_layer(w, mask=np.ones(8, np.uint8))
    rng = np.random.default_rng(17)
    for g in range(2):
        src = inp.planted_pos[0, g]                       # 1024 strong rows, all different
        starts = rng.choice(np.arange(2048, 131072 - 1024, 1024), size=8, replace=False)
        for c, s0 in enumerate(starts):                   # 8 runs of 500 consecutive strong rows
            rows = src[(np.arange(500) + 125 * c) % src.size]
            inp.k_cache[0, g, int(s0) + 13:int(s0) + 513] = inp.k_cache[0, g, rows]
    few0, many0 = ctx.select_stats()
    _say("scores in runs: 8 runs of 500 strong rows per KV head at 128K, k 4096")
    H.check_layer(ctx, inp, np.ones(8, np.uint8), w.k, None, "runs", exact_sets=True)
    assert ctx.select_stats() == (few0, many0)


# ------------------------------------------------------------------ Threshold and Top-p (Sec. 4.4.1)
@pytest.mark.parametrize("rule,param", [(1, 1e-2), (1, 1e-4), (1, 1e-6), (1, 0.9), (2, 0.5), (2, 0.9), (2, 0.999), (2, 1.0)])
def test_probability_rules_on_a_long_sequence(ctx, rule, param):
    w = wl.scaled(wl.WORKLOADS["c5"], n_q_heads=8, n_kv_heads=2, n_retrieval=0, retrieval_heads=(0, 4, 5), k=3000,
                  max_len=50000, planted=64)
    inp = wl.make_layer(w, l_cap=50000)
    _say("probability rule %d, parameter %g, L 50000, k 3000" % (rule, param))
    idx_in = H.previous_layer_sets(inp, w.k)
    sizes = H.check_prob_rule_layer(ctx, inp, inp.mask, w.k, rule, param, "rule %d %g" % (rule, param), idx_in)
    assert (sizes >= 0).all()
    sizes_all = H.check_prob_rule_layer(ctx, inp, np.ones(8, np.uint8), w.k, rule, param, "rule %d %g all" % (rule, param))
    if (rule, param) in ((1, 0.9), ):
        assert (sizes_all <= 1).all()          # nothing holds 90 % of the mass here: only the best position is kept
    if (rule, param) == (2, 1.0):
        assert (sizes_all == 3000).all()       # all of the mass: capped at k


@pytest.mark.parametrize("rule,param", [(1, 1e-3), (2, 0.8)])
def test_probability_rules_on_short_and_ragged_sequences(ctx, rule, param):
    w = wl.scaled(wl.WORKLOADS["c4"], batch=3, max_len=6000, k=500, planted=8, len_lo=40, len_hi=6000)
    lens_h = np.array([6000, 40, 333], np.int32)
    inp = wl.make_layer(w, lens=lens_h, l_cap=6000)
    _say("probability rule %d on ragged lengths %s (k larger than two of them)" % (rule, lens_h.tolist()))
    H.check_prob_rule_layer(ctx, inp, np.ones(w.n_q_heads, np.uint8), w.k, rule, param, "ragged rule %d" % rule)


@pytest.mark.parametrize("rule,param", [(1, 1e-3), (2, 0.8)])
@pytest.mark.parametrize("lens,n_wg", [([300, 65, 1, 64, 129, 1000], 24), ([300, 65, 1, 64, 129, 1000], 25), ([2000, 4100], 64)])
def test_probability_rules_beside_the_lines_between_their_routes(ctx, lens, n_wg, rule, param):
    """Twelve rows select in a second launch on 24 and 25 workgroups, as their segments complete on 48 and 50; four
    rows on 64 and 128 workgroups are selected at the end of the grid."""
    w = wl.scaled(wl.WORKLOADS["c1"], batch=len(lens), max_len=max(lens), k=100, planted=1)
    mask = np.tile(np.array([1, 0, 1, 0], np.uint8), w.n_q_heads // 4)
    inp = wl.make_layer(w, mask=mask, lens=np.asarray(lens, np.int32), l_cap=max(lens))
    idx_in = H.previous_layer_sets(inp, w.k)
    for n in (n_wg, 2 * n_wg):
        _say("rule routes: %d rows, rule=%d n_wg=%d" % (len(lens) * w.n_kv_heads, rule, n))
        ctx.set_option(H.binding().OPT_N_WG, n)
        H.check_prob_rule_layer(ctx, inp, mask, w.k, rule, param, "n_wg=%d" % n, idx_in)


@pytest.mark.parametrize("lens,rule,param", [([1000, 1, 900, 1000, 64, 950], 2, 0.8), ([1000, 1, 900, 1000, 64, 950], 1, 1e-3),
                                             ([5000, 4097, 4700, 5000, 4999, 4160], 2, 0.8)])
def test_where_a_rules_rows_are_selected_in_a_cache_of_many_times_their_length(own_ctx, lens, rule, param):
    """Twelve rows on 24 workgroups in a cache whose capacity says nothing about them.  Of the first lengths a workgroup's
    run holds several segments, and the second launch selects; of the other ones the first does, and the second
    finds nothing to do.  The same launches, and the oracle's sets, twice with either."""
    lb, ctx = H.binding(), own_ctx
    ctx.set_option(lb.OPT_N_WG, 24)
    ctx.timing_enable(True)
    w = wl.scaled(wl.WORKLOADS["c1"], batch=len(lens), max_len=9000, k=100, planted=1)
    mask = np.tile(np.array([1, 0, 1, 0], np.uint8), w.n_q_heads // 4)
    inp = wl.make_layer(w, mask=mask, lens=np.asarray(lens, np.int32), l_cap=w.max_len)
    idx_in = H.previous_layer_sets(inp, w.k)
    for i in range(2):
        _say("rule %d, up to %d rows in a cache of %d" % (rule, max(lens), w.max_len))
        H.check_prob_rule_layer(ctx, inp, mask, w.k, rule, param, "call %d" % i, idx_in)
        n = ctx.timing_read()[1]
        assert (n[lb.KERNEL_STREAM], n[lb.KERNEL_SELECT], sum(n)) == (1, 1, 2), n
    assert ctx.wait_timeouts() == 0


def test_a_captured_rule_call_follows_the_lengths_it_is_replayed_with(own_ctx):
    """A captured pair of launches decides anew in every replay: lengths of which the second launch selects and lengths of
    which the first does, in turn, against the eager call."""
    lb, ctx = H.binding(), own_ctx
    ctx.set_option(lb.OPT_N_WG, 24)
    w = wl.scaled(wl.WORKLOADS["c1"], batch=6, max_len=9000, k=100, planted=1)
    mask = np.tile(np.array([1, 0, 1, 0], np.uint8), w.n_q_heads // 4)
    inp = wl.make_layer(w, mask=mask, lens=np.full(6, 9000, np.int32), l_cap=w.max_len)
    dl = H.DeviceLayer(inp, w.k, np.tile(np.arange(w.k, dtype=np.int32), (6, w.n_kv_heads, 1)))
    dl.shape = lb.make_shape(6, w.n_q_heads, w.n_kv_heads, w.max_len, w.k, kv=dl.k_cache, prob_rule=2, prob_param=0.8)

    def call():
        ctx.decode_attn(dl.shape, dl.q, dl.k_cache, dl.v_cache, mask, dl.idx_in, dl.out, dl.idx_out, dl.lengths, dl.workspace)

    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            call()
    torch.cuda.synchronize()
    for i, lens in enumerate(([1000, 1, 900, 1000, 64, 950], [5000, 4097, 4700, 5000, 4999, 4160]) * 2):
        _say("replay %d, up to %d rows" % (i, max(lens)))
        dl.lengths.copy_(torch.tensor(lens, dtype=torch.int32))
        got = []
        for run in (graph.replay, call):
            dl.out.fill_(float("nan"))
            dl.idx_out.fill_(-7)
            run()
            torch.cuda.synchronize()
            got.append((dl.out.clone(), dl.idx_out.clone()))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), "replay %d" % i
        assert (dl.idx_out != -7).all() and ctx.wait_timeouts() == 0


@pytest.mark.parametrize("L,k", [(3000, 2000), (9000, 5000), (50000, 2000)])
def test_top_p_crosses_its_mass_among_equal_keys(ctx, L, k):
    """More equal keys than are looked at one by one hold the position where the mass is reached: the rest of
    it is counted in whole positions.  Rows of 3000 and of 9000 candidates (the first list fits registers, the
    second does not), and a sampled row."""
    copies = 400
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=L, k=k, planted=4)
    inp = wl.make_layer(w, l_cap=L)
    ones = np.ones(w.n_q_heads, np.uint8)
    _, _, sel0 = H.oracle_layer(inp, ones, w.k, None)
    src = np.zeros((1, w.n_kv_heads, 1), np.int64)
    for g in range(w.n_kv_heads):
        src[0, g, 0] = np.argsort(-sel0[0, g, :L], kind="stable")[6]  # (below the planted rows)
    wl.plant_ties(inp, copies, src)
    _, _, sel = H.oracle_layer(inp, ones, w.k, None)
    s = sel[0, :, :L]
    s = s - s.max(axis=1, keepdims=True)
    prob = np.exp(s) / np.exp(s).sum(axis=1, keepdims=True)
    tied = [s[g] == s[g, src[0, g, 0]] for g in range(w.n_kv_heads)]
    assert all(t.sum() > copies for t in tied)
    # the middle of the tied rows' share of the first KV head's mass
    above = prob[0][s[0] > s[0, src[0, 0, 0]]].sum()
    param = float(np.float32(above + 0.5 * prob[0][tied[0]].sum()))
    _say("top-p %g: L=%d, %d equal keys where the mass is reached" % (param, L, int(tied[0].sum())))
    sizes = H.check_prob_rule_layer(ctx, inp, ones, w.k, 2, param, "ties L=%d" % L)
    # (the mass the smaller of two sets may lack, as in check_prob_rule_layer, in positions of this probability)
    slack = 1 + 1e-4 * param / prob[0][src[0, 0, 0]]
    assert abs(int(sizes[0, 0]) - int((s[0] > s[0, src[0, 0, 0]]).sum()) - copies // 2) <= slack


def test_probability_rule_step_feeds_variable_sets_to_the_next_layers(ctx):
    lb = H.binding()
    n_layers, k = 4, 1500
    w = wl.scaled(wl.WORKLOADS["c3"], max_len=30000, k=k, n_layers=n_layers, planted=64)
    layers = [wl.make_layer(w, layer=l, device="cuda", l_cap=30000) for l in range(n_layers)]
    masks = np.stack([ly.mask for ly in layers])
    idx = None
    refs = []
    for ly in layers:
        out_ref, idx, _ = H.lo.decode_attn(wl.bf16_bits(ly.q), wl.bf16_bits(ly.k_cache), wl.bf16_bits(ly.v_cache),
                                           ly.mask, k, idx, ly.lengths, rule=2, rule_param=0.95)
        refs.append(out_ref)
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 30000, k, kv=layers[0].k_cache, prob_rule=lb.RULE_TOP_P,
                          prob_param=0.95)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    idx_final = torch.full((w.batch, w.n_kv_heads, k), -9, dtype=torch.int32, device="cuda")
    lens = torch.from_numpy(layers[0].lengths).cuda()
    _say("Top-p 0.95: 4-layer phased step")
    ctx.decode_step(shape, [ly.q for ly in layers], [ly.k_cache for ly in layers], [ly.v_cache for ly in layers],
                    masks, None, outs, idx_final, lens, ws)
    torch.cuda.synchronize()
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l], "top-p step layer %d" % l)
    got = idx_final.cpu().numpy()
    sizes = (got >= 0).sum(axis=2)
    assert (sizes >= 1).all() and (sizes <= k).all()


# ------------------------------------------------------------------ layer calls with a pending select
@pytest.mark.parametrize("margin,block", [(60, 1), (-1000, 1), (60, 64)])
def test_layer_calls_that_leave_their_select_pending(ctx, margin, block):
    """Layer after layer through lychee_decode_attn_deferred, the way a model would call it: one
    query buffer, overwritten with the next layer's queries as soon as a call is enqueued.  Each
    layer's selection runs inside the next call (or the flush) and must still see its own layer's
    queries - also on the route that recomputes the whole score row (margin -1000).  Outputs and
    every layer's sets against the oracle chain."""
    lb = H.binding()
    n_layers = 5
    k = 24 if block == 64 else 700
    w = wl.scaled(wl.WORKLOADS["c3"], max_len=12000, k=k, n_layers=n_layers, planted=48)
    layers = [wl.make_layer(w, layer=l, device="cuda", l_cap=12000) for l in range(n_layers)]
    idx = None
    refs = []
    for ly in layers:
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, k, idx, block=block)
        refs.append((out_ref, idx, sel_ref))
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 12000, k, kv=layers[0].k_cache, block_size=block)
    ws = lb.alloc_workspace(shape, n_layers=2)
    ws.fill_(0xFF)
    q_buf = torch.empty_like(layers[0].q)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    sets = [torch.full((w.batch, w.n_kv_heads, k), -9, dtype=torch.int32, device="cuda") for _ in layers]
    lens = torch.from_numpy(layers[0].lengths).cuda()
    few0, many0 = ctx.select_stats()
    ctx.set_option(lb.OPT_SELECT_MARGIN, margin)
    try:
        for rep in range(2):        # the second pass finds both halves of the workspace used
            for l, ly in enumerate(layers):
                _say("deferred layer call %d (margin %d, block %d, pass %d)" % (l, margin, block, rep))
                q_buf.copy_(ly.q)   # stream order: after the previous call's work, before its select has run
                ctx.decode_attn_deferred(shape, q_buf, ly.k_cache, ly.v_cache, ly.mask,
                                         sets[l - 1] if l else None, outs[l], sets[l], lens, ws)
            q_buf.zero_()
            ctx.select_flush()
            ctx.select_flush()      # nothing pending any more: a no-op
            torch.cuda.synchronize()
    finally:
        ctx.set_option(lb.OPT_SELECT_MARGIN, 60)
    few, many = ctx.select_stats()
    if margin == -1000:
        assert few - few0 > 0, "the recomputing route did not run"
    G = w.group
    for l, ly in enumerate(layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "deferred layer %d" % l)
        got = sets[l].cpu().numpy()
        for g in range(w.n_kv_heads):
            if ly.mask[g * G:(g + 1) * G].any():
                sc = H.unit_scores(refs[l][2][0, g], int(ly.lengths[0]), block)
                ok, _, msg = H.index_sets_match(got[0, g], refs[l][1][0, g], sc, k, H.TIE_REL)
                assert ok, "layer %d head %d: %s" % (l, g, msg)
            else:
                assert (got[0, g] == refs[l][1][0, g]).all(), "layer %d head %d: inherited set not copied" % (l, g)
    # the same chain through two set buffers used in turn, as a model would hold them: layer l reads
    # the buffer that the select of layer l-1 fills in this very call, and writes the other one
    pair = [torch.full_like(sets[0], -9) for _ in range(2)]
    outs2 = [torch.zeros_like(o) for o in outs]
    for l, ly in enumerate(layers):
        q_buf.copy_(ly.q)
        ctx.decode_attn_deferred(shape, q_buf, ly.k_cache, ly.v_cache, ly.mask,
                                 pair[(l - 1) % 2] if l else None, outs2[l], pair[l % 2], lens, ws)
    ctx.select_flush()
    torch.cuda.synchronize()
    for l in range(n_layers):
        assert torch.equal(outs2[l], outs[l]), "two buffers in turn: layer %d differs" % l
    assert torch.equal(pair[(n_layers - 1) % 2], sets[-1])


@pytest.mark.parametrize("L", [5000, 16384, 40000])
def test_deferred_layer_calls_over_context_lengths(ctx, L):
    """The layer launch splits its workgroups between streaming and gathering from the lengths it
    finds on the device; contexts of a few thousand to tens of thousands of rows exercise the split
    where gathers outweigh the streaming, about even it, and are outweighed.  Five deferred calls
    with the c3 head layout against the oracle chain; no bounded wait may have given up."""
    lb = H.binding()
    n_layers = 5
    k = 1024
    w = wl.scaled(wl.WORKLOADS["c3"], max_len=L, k=k, n_layers=n_layers, planted=32)
    layers = [wl.make_layer(w, layer=l, device="cuda", l_cap=L) for l in range(n_layers)]
    idx = None
    refs = []
    for ly in layers:
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, k, idx)
        refs.append((out_ref, idx, sel_ref))
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, L, k, kv=layers[0].k_cache)
    ws = lb.alloc_workspace(shape, n_layers=2)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    pair = [torch.full((w.batch, w.n_kv_heads, k), -9, dtype=torch.int32, device="cuda") for _ in range(2)]
    lens = torch.from_numpy(layers[0].lengths).cuda()
    waits0 = ctx.wait_timeouts()
    for l, ly in enumerate(layers):
        _say("context %d: deferred layer call %d" % (L, l))
        ctx.decode_attn_deferred(shape, ly.q, ly.k_cache, ly.v_cache, ly.mask,
                                 pair[(l - 1) % 2] if l else None, outs[l], pair[l % 2], lens, ws)
    ctx.select_flush()
    torch.cuda.synchronize()
    assert ctx.wait_timeouts() == waits0
    G = w.group
    for l, ly in enumerate(layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "context %d layer %d" % (L, l))
    got = pair[(n_layers - 1) % 2].cpu().numpy()
    last = layers[-1]
    for g in range(w.n_kv_heads):
        if last.mask[g * G:(g + 1) * G].any():
            ok, _, msg = H.index_sets_match(got[0, g], refs[-1][1][0, g], refs[-1][2][0, g, :L], k, H.TIE_REL)
            assert ok, "context %d head %d: %s" % (L, g, msg)
        else:
            assert (got[0, g] == refs[-1][1][0, g]).all()


@pytest.mark.parametrize("n_wg", [1, 3, 7, 37])
def test_deferred_layer_calls_on_tiny_grids(ctx, n_wg):
    """A handful of workgroups for a whole layer launch: below 8 the front workgroups (the previous
    call's select, this call's thresholds) take pieces themselves afterwards, a single workgroup does
    everything in turn, and a piece is many thousand rows long, so it filters its key buffer several
    times on the way.  Four deferred calls against the oracle chain."""
    lb = H.binding()
    n_layers, k, L = 4, 900, 21000
    w = wl.scaled(wl.WORKLOADS["c3"], max_len=L, k=k, n_layers=n_layers, planted=32)
    layers = [wl.make_layer(w, layer=l, device="cuda", l_cap=L) for l in range(n_layers)]
    idx = None
    refs = []
    for ly in layers:
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, k, idx)
        refs.append((out_ref, idx, sel_ref))
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, L, k, kv=layers[0].k_cache)
    ws = lb.alloc_workspace(shape, n_layers=2)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    pair = [torch.full((w.batch, w.n_kv_heads, k), -9, dtype=torch.int32, device="cuda") for _ in range(2)]
    lens = torch.from_numpy(layers[0].lengths).cuda()
    waits0 = ctx.wait_timeouts()
    ctx.set_option(lb.OPT_N_WG, n_wg)
    try:
        for l, ly in enumerate(layers):
            _say("grid of %d: deferred layer call %d" % (n_wg, l))
            ctx.decode_attn_deferred(shape, ly.q, ly.k_cache, ly.v_cache, ly.mask,
                                     pair[(l - 1) % 2] if l else None, outs[l], pair[l % 2], lens, ws)
        ctx.select_flush()
        torch.cuda.synchronize()
    finally:
        ctx.set_option(lb.OPT_N_WG, 0)
    assert ctx.wait_timeouts() == waits0
    G = w.group
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "grid %d layer %d" % (n_wg, l))
    got = pair[(n_layers - 1) % 2].cpu().numpy()
    last = layers[-1]
    for g in range(w.n_kv_heads):
        if last.mask[g * G:(g + 1) * G].any():
            ok, _, msg = H.index_sets_match(got[0, g], refs[-1][1][0, g], refs[-1][2][0, g, :L], k, H.TIE_REL)
            assert ok, "grid %d head %d: %s" % (n_wg, g, msg)
        else:
            assert (got[0, g] == refs[-1][1][0, g]).all()


def test_deferred_calls_of_layers_without_a_retrieval_head(ctx):
    """Every piece is a gather and every gather waits for a set that the same launch copies: 300 copies,
    written by workgroups that take no pieces."""
    lb = H.binding()
    n_seq, k = 150, 12
    lens_h = np.array([64, 700, 3001] * 50, np.int32)
    w = wl.scaled(wl.WORKLOADS["c1"], batch=n_seq, max_len=3001, k=k, planted=1)
    mask = np.zeros(w.n_q_heads, np.uint8)
    inp = wl.make_layer(w, mask=mask, lens=lens_h, l_cap=3001)
    idx_in = H.previous_layer_sets(inp, k, block=64)
    out_ref, _, _ = H.oracle_layer(inp, mask, k, idx_in, block=64)
    dl = H.DeviceLayer(inp, k, idx_in, block=64)
    ws = lb.alloc_workspace(dl.shape, "cuda", n_layers=2)
    ws.fill_(0xFF)
    sets = [dl.idx_in] + [torch.full_like(dl.idx_in, -7) for _ in range(3)]
    outs = [torch.full_like(dl.out, float("nan")) for _ in range(3)]
    waits0 = ctx.wait_timeouts()
    _say("three all-sparse layers, %d sequences, block-granular sets" % n_seq)
    for l in range(3):
        ctx.decode_attn_deferred(dl.shape, dl.q, dl.k_cache, dl.v_cache, mask, sets[l], outs[l], sets[l + 1], dl.lengths, ws)
    ctx.select_flush()
    torch.cuda.synchronize()
    assert ctx.wait_timeouts() == waits0
    for l in range(3):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), out_ref, "all-sparse layer %d" % l)
        assert torch.equal(sets[l + 1], dl.idx_in)


def test_two_contexts_on_two_streams_run_layer_calls_side_by_side():
    """Two contexts, each on a stream of its own, run deferred layer chains at the same time (two
    model replicas on one GPU).  The launches share the GPU's workgroup slots; every wait inside a
    launch is for a front unit of the same launch, which is dispatched before its waiters, so the
    two must neither disturb nor stall each other.  Both chains against the oracle; no wait gave up."""
    lb = H.binding()
    n_layers = 4
    k = 512
    L = 20000
    chains = []
    for seed_shift in (0, 1):
        w = wl.scaled(wl.WORKLOADS["c3"], max_len=L, k=k, n_layers=n_layers + seed_shift, planted=32)
        layers = [wl.make_layer(w, layer=l + seed_shift, device="cuda", l_cap=L) for l in range(n_layers)]
        if seed_shift:   # (layer 0 of a chain passes no inherited sets: every head must be a retrieval head there)
            layers[0].mask[:] = 1
        idx = None
        refs = []
        for ly in layers:
            out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, k, idx)
            refs.append((out_ref, idx, sel_ref))
        shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, L, k, kv=layers[0].k_cache)
        chains.append(dict(w=w, layers=layers, refs=refs, shape=shape, ctx=lb.Context(0), stream=torch.cuda.Stream(),
                           ws=lb.alloc_workspace(shape, n_layers=2),
                           outs=[torch.zeros_like(ly.q) for ly in layers],
                           pair=[torch.full((w.batch, w.n_kv_heads, k), -9, dtype=torch.int32, device="cuda") for _ in range(2)],
                           lens=torch.from_numpy(layers[0].lengths).cuda()))
    torch.cuda.synchronize()
    try:
        for rep in range(3):
            for l in range(n_layers):
                for ch in chains:   # alternate between the two streams: the launches overlap on the GPU
                    ly = ch["layers"][l]
                    ch["ctx"].decode_attn_deferred(ch["shape"], ly.q, ly.k_cache, ly.v_cache, ly.mask,
                                                   ch["pair"][(l - 1) % 2] if l else None, ch["outs"][l], ch["pair"][l % 2],
                                                   ch["lens"], ch["ws"], stream=ch["stream"])
            for ch in chains:
                ch["ctx"].select_flush(stream=ch["stream"])
        torch.cuda.synchronize()
        for i, ch in enumerate(chains):
            assert ch["ctx"].wait_timeouts() == 0
            for l in range(n_layers):
                H.assert_outputs_close(H.bf16_tensor_to_f64(ch["outs"][l]), ch["refs"][l][0], "chain %d layer %d" % (i, l))
            w, last = ch["w"], ch["layers"][-1]
            got = ch["pair"][(n_layers - 1) % 2].cpu().numpy()
            for g in range(w.n_kv_heads):
                if last.mask[g * w.group:(g + 1) * w.group].any():
                    ok, _, msg = H.index_sets_match(got[0, g], ch["refs"][-1][1][0, g], ch["refs"][-1][2][0, g, :L], k, H.TIE_REL)
                    assert ok, "chain %d head %d: %s" % (i, g, msg)
                else:
                    assert (got[0, g] == ch["refs"][-1][1][0, g]).all()
    finally:
        torch.cuda.synchronize()
        for ch in chains:
            ch["ctx"].close()


def test_a_pending_select_pins_its_workspace_and_shape(ctx):
    lb = H.binding()
    w = wl.scaled(wl.WORKLOADS["c1"], max_len=6000, k=100)
    inp = wl.make_layer(w, device="cuda", l_cap=6000)
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 6000, w.k, kv=inp.k_cache)
    ws2 = lb.alloc_workspace(shape, n_layers=2)
    other = lb.alloc_workspace(shape, n_layers=2)
    out = torch.zeros_like(inp.q)
    idx_a = torch.zeros((w.batch, w.n_kv_heads, w.k), dtype=torch.int32, device="cuda")
    idx_b = torch.zeros_like(idx_a)
    lens = torch.from_numpy(inp.lengths).cuda()
    ones = np.ones(w.n_q_heads, np.uint8)
    with pytest.raises(lb.LycheeError) as e:      # a one-layer workspace is too small
        ctx.decode_attn_deferred(shape, inp.q, inp.k_cache, inp.v_cache, ones, None, out, idx_a, lens,
                                 lb.alloc_workspace(shape))
    assert e.value.code == lb.EWORKSPACE
    ctx.decode_attn_deferred(shape, inp.q, inp.k_cache, inp.v_cache, ones, None, out, idx_a, lens, ws2)
    with pytest.raises(lb.LycheeError) as e:      # another workspace while a select is pending
        ctx.decode_attn_deferred(shape, inp.q, inp.k_cache, inp.v_cache, ones, None, out, idx_b, lens, other)
    assert e.value.code == lb.EINVAL
    with pytest.raises(lb.LycheeError) as e:      # nor may another kind of call use the pinned workspace
        ctx.decode_attn(shape, inp.q, inp.k_cache, inp.v_cache, ones, None, out, idx_b, lens, ws2)
    assert e.value.code == lb.EINVAL
    ctx.select_flush()
    ctx.decode_attn_deferred(shape, inp.q, inp.k_cache, inp.v_cache, ones, None, out, idx_b, lens, other)
    ctx.select_flush()
    torch.cuda.synchronize()
    assert torch.equal(idx_a, idx_b)


@pytest.mark.parametrize("rule", ["ratio", "threshold", "top_p"])
def test_pending_selects_under_the_other_selection_rules(ctx, rule):
    """The rules of Sec. 4.4.1 decide inside the select, from what the streaming left in the
    layer's scratch (for the probability rules also the pooled log-sum-exp): a pending select must
    find all of it in its own half of the workspace.  The plain layer call, whose parity with the
    oracle the tests above establish, is the reference for the probability rules: the sets bit for
    bit (the select is exact, whoever streamed a row), the outputs to the bar of the parity tests
    (the two kinds of call cut a layer's rows into different pieces).  Under the Ratio rule the
    chain of pending selects is also checked against the oracle's chain directly."""
    lb = H.binding()
    n_layers = 4
    k = 600
    w = wl.scaled(wl.WORKLOADS["c4"], batch=2, max_len=9000, k=k, n_layers=n_layers, planted=32,
                  len_lo=2500, len_hi=9000)
    lens_h = wl.lengths(w)
    layers = [wl.make_layer(w, layer=l, device="cuda", lens=lens_h, l_cap=9000) for l in range(n_layers)]
    kw = {"ratio": dict(keep_ppm=40000), "threshold": dict(prob_rule=lb.RULE_THRESHOLD, prob_param=2e-4),
          "top_p": dict(prob_rule=lb.RULE_TOP_P, prob_param=0.6)}[rule]
    shape = lb.make_shape(w.batch, w.n_q_heads, w.n_kv_heads, 9000, k, kv=layers[0].k_cache, **kw)
    lens = torch.from_numpy(lens_h).cuda()
    first = torch.from_numpy(H.previous_layer_sets(layers[0], k)).cuda()

    def run(deferred):
        ws = lb.alloc_workspace(shape, n_layers=2 if deferred else 1)
        ws.fill_(0xFF)
        outs = [torch.zeros_like(ly.q) for ly in layers]
        sets = [torch.full((w.batch, w.n_kv_heads, k), -9, dtype=torch.int32, device="cuda") for _ in layers]
        for l, ly in enumerate(layers):
            call = ctx.decode_attn_deferred if deferred else ctx.decode_attn
            call(shape, ly.q, ly.k_cache, ly.v_cache, ly.mask, sets[l - 1] if l else first, outs[l], sets[l], lens, ws)
        if deferred:
            ctx.select_flush()
        torch.cuda.synchronize()
        return outs, sets

    _say("pending selects, rule %s" % rule)
    outs_a, sets_a = run(False)
    outs_b, sets_b = run(True)
    kept = 0
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs_b[l]), H.bf16_tensor_to_f64(outs_a[l]),
                               "layer %d, pending vs plain" % l)
        assert torch.equal(sets_a[l], sets_b[l]), "layer %d: sets differ" % l
        kept += int((sets_a[l] >= 0).sum())
    assert 0 < kept < n_layers * w.batch * w.n_kv_heads * k, "the rule kept everything or nothing"
    if rule == "ratio":
        idx = first.cpu().numpy()
        for l, ly in enumerate(layers):
            out_ref, idx_new, sel_ref = H.oracle_layer(ly, ly.mask, k, idx, keep_ppm=kw["keep_ppm"])
            H.assert_outputs_close(H.bf16_tensor_to_f64(outs_b[l]), out_ref, "layer %d, pending vs oracle" % l)
            H.assert_sets_match(sets_b[l].cpu().numpy(), idx_new, sel_ref, ly.mask, ly, k, idx,
                                "layer %d, pending vs oracle" % l, keep_ppm=kw["keep_ppm"])
            idx = idx_new


# ------------------------------------------------------------------ seeded sweep over odd shapes
def _sweep_cases(n=24, seed=20260204):
    rng = np.random.default_rng(seed)
    cases = []
    for i in range(n):
        Hkv = int(rng.choice([1, 2, 3, 4, 8]))
        G = int(rng.choice([1, 2, 3, 4]))
        B = int(rng.choice([1, 1, 2, 3, 5]))
        l_cap = int(rng.choice([97, 640, 1500, 4097, 9000, 20000]))
        lens = [int(x) for x in rng.integers(max(1, l_cap // 3), l_cap + 1, size=B)]
        block = int(rng.choice([1, 1, 1, 64]))
        units = (l_cap + 63) // 64 if block == 64 else l_cap
        k = int(max(1, min(units, rng.choice([1, 7, 64, 300, 1024, 5000]))))
        keep_ppm = int(rng.choice([0, 0, 0, 30000]))
        mask = (rng.random(Hkv * G) < rng.choice([0.15, 0.4, 0.8])).astype(np.uint8)
        cases.append((i, B, Hkv, G, l_cap, lens, k, block, keep_ppm, mask))
    return cases


@pytest.mark.parametrize("case", _sweep_cases(), ids=lambda c: "s%02d_B%d_kv%d_G%d_L%d_k%d_b%d_r%d" % (
    c[0], c[1], c[2], c[3], c[4], c[6], c[7], c[8]))
def test_seeded_sweep_of_shapes_masks_and_modes(ctx, case):
    """Layer calls on drawn shapes (KV heads 1-8, group sizes 1-4, batches of ragged lengths, budgets
    from 1 to more than the sequence, token- and block-granular sets, the Ratio rule, masks from
    mostly sparse to mostly retrieval): outputs and sets against the oracle.  The grid's padded and
    unpadded static splits, one or two workgroups per CU, all depend on these numbers."""
    i, B, Hkv, G, l_cap, lens, k, block, keep_ppm, mask = case
    w = wl.scaled(wl.WORKLOADS["c1"], batch=B, n_q_heads=Hkv * G, n_kv_heads=Hkv, max_len=l_cap, k=k,
                  planted=min(6, min(lens)), retrieval_heads=(), config_id=900 + i)
    inp = wl.make_layer(w, mask=mask, lens=np.asarray(lens, np.int32), l_cap=l_cap)
    idx_in = None if mask.all() else H.previous_layer_sets(inp, k, block=block)
    _say("sweep %s lens=%s mask=%s" % (case[:5] + case[6:9], lens, mask.tolist()))
    H.check_layer(ctx, inp, mask, k, idx_in, "sweep%d" % i, keep_ppm=keep_ppm, block=block)


@pytest.mark.parametrize("B,Hkv,G", [(256, 2, 1), (2, 64, 4), (256, 8, 4)])
def test_largest_batch_and_head_counts(ctx, B, Hkv, G):
    """The limits of a shape: 256 sequences (one per thread of the workgroup-wide scans over the batch), 64 KV
    heads (the per-head tables of a layer descriptor), groups of 4, and both at once with 2048 query heads.
    One further sequence or KV head is refused."""
    lb = H.binding()
    l_cap, k = 500, 24
    rng = np.random.default_rng(1000 * B + Hkv)
    lens = rng.integers(1, l_cap + 1, size=B).astype(np.int32)
    lens[0], lens[-1] = l_cap, 1
    mask = (rng.random(Hkv * G) < 0.3).astype(np.uint8)
    mask[0], mask[-1] = 1, 0     # both kinds of head present
    w = wl.scaled(wl.WORKLOADS["c1"], batch=B, n_q_heads=Hkv * G, n_kv_heads=Hkv, max_len=l_cap, k=k,
                  planted=1, retrieval_heads=(), config_id=970 + Hkv)
    inp = wl.make_layer(w, mask=mask, lens=lens, l_cap=l_cap)
    idx_in = H.previous_layer_sets(inp, k)
    _say("limits: batch %d, %d KV heads, group %d" % (B, Hkv, G))
    dl = H.check_layer(ctx, inp, mask, k, idx_in, "limits B%d kv%d" % (B, Hkv))[0]
    assert ctx.wait_timeouts() == 0
    too_many = lb.make_shape(B + 1 if B == 256 else B, (Hkv + 1 if Hkv == 64 else Hkv) * G, Hkv + 1 if Hkv == 64 else Hkv,
                             l_cap, k, kv=dl.k_cache)
    assert lb.check_shape(too_many) == lb.EUNSUPPORTED


@pytest.mark.parametrize("block", [1, 64])
def test_a_serving_batch_of_many_short_sequences(ctx, block):
    """64 sequences of 40 to 3000 rows in one call (a serving batch): hundreds of (sequence, KV head)
    segments, more than the grid has workgroups, so the runs are unpadded and most workgroups cross
    from one segment into the next.  A layer call, then a three-layer layer-after-layer step."""
    lb = H.binding()
    B, Hkv, G, l_cap = 64, 4, 2, 3000
    k = 10 if block == 64 else 200
    rng = np.random.default_rng(77)
    lens = rng.integers(40, l_cap + 1, size=B).astype(np.int32)
    lens[:3] = (1, l_cap, 64)
    mask = np.array([1, 0, 0, 0, 0, 1, 0, 0], np.uint8)   # KV heads 0 and 2 hold a retrieval head
    w = wl.scaled(wl.WORKLOADS["c1"], batch=B, n_q_heads=Hkv * G, n_kv_heads=Hkv, max_len=l_cap, k=k,
                  planted=1, retrieval_heads=(), config_id=950 + block)
    inp = wl.make_layer(w, mask=mask, lens=lens, l_cap=l_cap)
    idx_in = H.previous_layer_sets(inp, k, block=block)
    _say("serving batch, block %d: layer call" % block)
    H.check_layer(ctx, inp, mask, k, idx_in, "batch64", block=block)
    # the step: layer 0 all-retrieval, then two hybrid layers
    n_layers = 3
    masks = np.stack([np.ones(Hkv * G, np.uint8), mask, mask[::-1].copy()])
    layers = [wl.make_layer(wl.scaled(w, config_id=960 + 10 * block + l), mask=masks[l], lens=lens, l_cap=l_cap, device="cuda")
              for l in range(n_layers)]
    idx = None
    refs = []
    for ly in layers:
        out_ref, idx, sel_ref = H.oracle_layer(ly, ly.mask, k, idx, block=block)
        refs.append((out_ref, idx, sel_ref))
    shape = lb.make_shape(B, Hkv * G, Hkv, l_cap, k, kv=layers[0].k_cache, block_size=block)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    idx_final = torch.full((B, Hkv, k), -9, dtype=torch.int32, device="cuda")
    lens_d = torch.from_numpy(lens).cuda()
    ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_LAYERWISE)
    _say("serving batch, block %d: step" % block)
    ctx.decode_step(shape, [ly.q for ly in layers], [ly.k_cache for ly in layers], [ly.v_cache for ly in layers],
                    masks, None, outs, idx_final, lens_d, ws)
    torch.cuda.synchronize()
    assert ctx.wait_timeouts() == 0
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "batch64 step layer %d" % l)
    got = idx_final.cpu().numpy()
    last = layers[-1]
    for b in range(B):
        for g in range(Hkv):
            if last.mask[g * G:(g + 1) * G].any():
                sc = H.unit_scores(refs[-1][2][b, g], int(lens[b]), block)
                ok, _, msg = H.index_sets_match(got[b, g], refs[-1][1][b, g], sc, min(k, len(sc)), H.TIE_REL)
                assert ok, "sequence %d head %d: %s" % (b, g, msg)
            else:
                assert (got[b, g] == refs[-1][1][b, g]).all()


def _step_cases(n=10, seed=20260205):
    rng = np.random.default_rng(seed)
    cases = []
    for i in range(n):
        Hkv = int(rng.choice([2, 4, 8]))
        G = int(rng.choice([1, 2, 4]))
        B = int(rng.choice([1, 2, 4]))
        n_layers = int(rng.integers(2, 6))
        l_cap = int(rng.choice([700, 3000, 11000, 30000]))
        lens = [int(x) for x in rng.integers(max(1, l_cap // 4), l_cap + 1, size=B)]
        block = int(rng.choice([1, 1, 64]))
        units = (l_cap + 63) // 64 if block == 64 else l_cap
        k = int(max(1, min(units, rng.choice([5, 100, 900, 4000]))))
        masks = (rng.random((n_layers, Hkv * G)) < rng.choice([0.1, 0.3, 0.6])).astype(np.uint8)
        mode = str(rng.choice(["phased", "layerwise"]))
        cases.append((i, B, Hkv, G, n_layers, l_cap, lens, k, block, mode, masks))
    return cases


@pytest.mark.parametrize("case", _step_cases(), ids=lambda c: "t%02d_B%d_kv%d_G%d_n%d_L%d_k%d_b%d_%s" % (
    c[0], c[1], c[2], c[3], c[4], c[5], c[7], c[8], c[9]))
def test_seeded_sweep_of_decode_steps(ctx, case):
    """Whole steps on drawn shapes and per-layer masks (layers without any retrieval head included:
    their sets pass through), in both step modes, with caller-supplied sets for the first layer:
    every layer's output and the final sets against the oracle's chain."""
    lb = H.binding()
    i, B, Hkv, G, n_layers, l_cap, lens_l, k, block, mode, masks = case
    w = wl.scaled(wl.WORKLOADS["c4"], batch=B, n_q_heads=Hkv * G, n_kv_heads=Hkv, max_len=l_cap, k=k,
                  n_layers=n_layers, planted=min(6, min(lens_l)), config_id=950 + i)
    lens_h = np.asarray(lens_l, np.int32)
    layers = [wl.make_layer(w, layer=l, device="cuda", mask=masks[l], lens=lens_h, l_cap=l_cap) for l in range(n_layers)]
    idx0 = H.previous_layer_sets(layers[0], k, block=block)
    idx = idx0
    refs = []
    for l, ly in enumerate(layers):
        out_ref, idx, sel_ref = H.oracle_layer(ly, masks[l], k, idx, block=block)
        refs.append((out_ref, idx, sel_ref))
    shape = lb.make_shape(B, Hkv * G, Hkv, l_cap, k, kv=layers[0].k_cache, block_size=block)
    ws = lb.alloc_workspace(shape, n_layers=n_layers)
    ws.fill_(0xFF)
    outs = [torch.zeros_like(ly.q) for ly in layers]
    idx_final = torch.full((B, Hkv, k), -9, dtype=torch.int32, device="cuda")
    lens = torch.from_numpy(lens_h).cuda()
    _say("step sweep %s lens=%s" % (case[:6] + case[7:10], lens_l))
    ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED if mode == "phased" else lb.STEP_LAYERWISE)
    try:
        ctx.decode_step(shape, [ly.q for ly in layers], [ly.k_cache for ly in layers],
                        [ly.v_cache for ly in layers], masks, torch.from_numpy(idx0).cuda(), outs, idx_final, lens, ws)
        torch.cuda.synchronize()
    finally:
        ctx.set_option(lb.OPT_STEP_MODE, lb.STEP_PHASED)
    for l in range(n_layers):
        H.assert_outputs_close(H.bf16_tensor_to_f64(outs[l]), refs[l][0], "step sweep %d layer %d" % (i, l))
    # the final set of a KV head comes from the last layer that selected for it (or from idx0)
    got = idx_final.cpu().numpy()
    for g in range(Hkv):
        src = None
        for l in range(n_layers - 1, -1, -1):
            if masks[l][g * G:(g + 1) * G].any():
                src = l
                break
        for b in range(B):
            if src is None:
                assert (got[b, g] == idx0[b, g]).all(), "head %d: caller's set not handed on" % g
            else:
                sc = H.unit_scores(refs[src][2][b, g], int(lens_h[b]), block)
                ok, _, msg = H.index_sets_match(got[b, g], refs[src][1][b, g], sc, min(k, sc.size), H.TIE_REL)
                assert ok, "seq %d head %d (selected in layer %d): %s" % (b, g, src, msg)
