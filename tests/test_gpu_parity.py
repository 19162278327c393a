"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle on the same seeded inputs.

Bars (stated with the build's target): accept lengths, emitted tokens, kv_len and pending bit-exact; logits within
2e-2 max-abs of the float32 oracle; drafted ids equal wherever the oracle's top-1/top-2 margin exceeds 1e-2.
A tighter bound (LOGIT_TIGHT) guards the design itself: activations enter every product as hi+lo bf16 pairs
(relative error < 2^-16) and sums are float32, so the measured gap sits near 1e-4; a dropped lo term or a wrong
lane mapping would land between the two bounds.
"""
import itertools

import numpy as np
import pytest

from paper_2509_18362_amd import synth
from plan_cases import BODY_TILES, HEAD_TILES, LIST_GROUPS

pytestmark = pytest.mark.gpu

LOGIT_TOL = 2e-2
LOGIT_TIGHT = 2e-3
MARGIN = 1e-2


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available()
    from oracle.oracle import Oracle
    from oracle import oracle as orc_mod
    from paper_2509_18362_amd import binding
    return {"torch": torch, "Oracle": Oracle, "orc": orc_mod, "binding": binding}


def appended_entries_close(got_bits, ref_bits, recursive_from=None):
    """Appended cache entries [Hkv][slots][hd]: both sides round a float32 value to bf16, but they sum in different
    orders, so the float32 values differ by ~1e-6 of the vector's scale and the rounded ones by at most one bf16 step
    (2^-7 relative) plus that absolute slack (which matters only for entries that cancel to almost zero).
    Slots from `recursive_from` on were produced by recursive steps (Sec. 2.3: step k > 1 consumes the head's own
    output hidden state), where the two sides' INPUTS already differ by the hidden-state gap the same test bounds by
    2e-3: their keys and values may differ by a matrix row's worth of that (measured up to 6e-5 of the scale at the
    third step of a one-token context), so the absolute slack there is 2e-4 of the scale."""
    g = synth.bf16_bits_to_f32(got_bits).astype(np.float64)
    r = synth.bf16_bits_to_f32(ref_bits).astype(np.float64)
    scale = max(float(np.abs(r).max()), 1e-30)
    slack = np.full(r.shape[1], 1e-5)
    if recursive_from is not None:
        slack[recursive_from:] = 2e-4
    return bool((np.abs(g - r) <= 2.0 ** -7 * np.abs(r) + slack[None, :, None] * scale).all())


def run_both(gpu, shape, w_host, w_dev, act, subsets, subset_index, K, engine=None, forced="oracle", seqs=None,
             max_batch=None):
    """Runs the oracle (float32) and the library on the same inputs.  `forced="oracle"`: the library is fed the
    oracle's drafts at steps 2..K so both chains see identical inputs; `None`: free-running.
    `seqs`: oracle only on these sequences (library always runs the whole batch)."""
    torch, Oracle, binding = gpu["torch"], gpu["Oracle"], gpu["binding"]
    B = len(act["kv_len"])
    cap = act["kv_capacity"]
    ids = None if subset_index < 0 else subsets[subset_index]
    sel = list(range(B)) if seqs is None else list(seqs)
    orc = Oracle(shape, w_host, cap, "f32")
    okc, ovc = act["k_cache"][sel].copy(), act["v_cache"][sel].copy()
    ref = orc.chain(K, act["hidden_in"][sel], act["token_in"][sel], okc, ovc, act["kv_len"][sel], ids)
    own = engine is None
    if own:
        engine = binding.DraftEngine(shape, w_dev, subsets, max_batch or B, cap, K)
    dkc, dvc = engine.to_device_bits(act["k_cache"]), engine.to_device_bits(act["v_cache"])
    forced_dev = None
    if forced == "oracle" and K > 1:
        full = np.zeros((B, K - 1), dtype=np.int32)
        full[sel] = ref["draft"][:, :K - 1]
        forced_dev = engine.to_device_i32(full)
    out = engine.draft(K, subset_index, engine.to_device_bits(act["hidden_in"]), engine.to_device_i32(act["token_in"]),
                       dkc, dvc, engine.to_device_i32(act["kv_len"]), forced=forced_dev, want_logits=True,
                       want_hidden=True)
    torch.cuda.synchronize()
    assert engine.poll_error() == 0
    res = {"draft": out["draft"].cpu().numpy()[sel], "logits": out["logits"].cpu().numpy()[sel],
           "hidden": out["hidden"].cpu().numpy()[sel],
           "k_cache": dkc.cpu().numpy().view(np.uint16)[sel], "v_cache": dvc.cpu().numpy().view(np.uint16)[sel]}
    if own:
        engine.close()
    return ref, res, (okc, ovc)


def check_chain(ref, res, caches, kv_len, K, aligned=True, need_clear=True):
    okc, ovc = caches
    gap = float(np.abs(ref["logits"] - res["logits"]).max()) if aligned else None
    if aligned:
        assert gap <= LOGIT_TOL, gap
        assert gap <= LOGIT_TIGHT, gap
        assert np.abs(ref["hidden"] - res["hidden"]).max() <= 2e-3
        clear = ref["margin"] > MARGIN
        assert clear.any() or not need_clear
        np.testing.assert_array_equal(ref["draft"][clear], res["draft"][clear])
    else:  # free-running: compare every chain up to its first unclear step
        for b in range(ref["draft"].shape[0]):
            for k in range(K):
                if ref["margin"][b, k] <= MARGIN:
                    break
                assert ref["draft"][b, k] == res["draft"][b, k]
                assert np.abs(ref["logits"][b, k] - res["logits"][b, k]).max() <= LOGIT_TOL
    # cache: prior entries untouched, appended entries equal up to one bf16 step (the two sides sum in different orders)
    for i, L in enumerate(kv_len):
        L = int(L)
        assert np.array_equal(res["k_cache"][i][:, :L], okc[i][:, :L])
        assert np.array_equal(res["v_cache"][i][:, :L], ovc[i][:, :L])
        if aligned:
            assert appended_entries_close(res["k_cache"][i][:, L:L + K], okc[i][:, L:L + K], recursive_from=1)
            assert appended_entries_close(res["v_cache"][i][:, L:L + K], ovc[i][:, L:L + K], recursive_from=1)
        assert np.array_equal(res["k_cache"][i][:, L + K:], okc[i][:, L + K:])
    return gap


# ------------------------------------------------------------------------------------------ tiny head (config 1)
def test_tiny_chain_forced_and_free(gpu, tiny):
    act, ids = tiny["act"], tiny["ids"]
    for forced in ("oracle", None):
        ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [ids], 0, 3, forced=forced)
        check_chain(ref, res, caches, act["kv_len"], 3, aligned=(forced == "oracle"))


def test_tiny_ragged_batch_and_empty_context(gpu, tiny):
    """B = 5 with contexts 0 (no prior entries), 1, 63, 64 and 150: spans split boundaries and the degenerate case."""
    wl = tiny["wl"]
    act = synth.make_activations(wl, ctx=np.array([0, 1, 63, 64, 150], dtype=np.int32), capacity=192)
    ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, 3)
    check_chain(ref, res, caches, act["kv_len"], 3)


def test_tiny_long_capacity_matrix_core_attention(gpu, tiny):
    """A large cache capacity makes the split plan long enough for the matrix-core attention kernel (448 tokens per
    split here) and, with seven sequences, for the batched matrix phases.  Contexts cover: nothing cached, fewer
    tokens than one 16-row tile, exactly one 32-token iteration, one more, several iterations per wave, and several
    splits (merged by the workgroup that finishes last)."""
    wl = tiny["wl"]
    ctx = np.array([0, 1, 31, 32, 33, 300, 1000], dtype=np.int32)
    act = synth.make_activations(wl, ctx=ctx, capacity=32768)
    ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, 3)
    check_chain(ref, res, caches, act["kv_len"], 3)


def test_tiny_many_long_contexts_items_handed_out(gpu, tiny):
    """Forty sequences with a capacity of 32768: splits are capped at 4096 tokens, which leaves up to 640 attention
    items for one workgroup per compute unit, so the matrix-core attention numbers the splits that exist longest
    first and hands them out through the counter.  Contexts sit on and around the split boundaries (a length that is
    a whole number of splits has no ragged final split, at each of the three steps once), at zero, and at the last
    slot that still fits K drafts; the call is made twice on one engine (the counter must be back at zero after the
    first)."""
    wl = tiny["wl"]
    K, cap = 3, 32768
    edge = [0, 1, 4092, 4093, 4094, 4095, 4096, 4097, 8191, 8192, 12000, 20000, 28671, 28672, 30000, cap - K]
    rng = np.random.default_rng(77)
    ctx = np.array(edge + list(rng.integers(0, cap - K, size=40 - len(edge))), dtype=np.int32)
    act = synth.make_activations(wl, ctx=ctx, capacity=cap)
    engine = gpu["binding"].DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], len(ctx), cap, K)
    for _ in range(2):
        ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, K, engine=engine)
        check_chain(ref, res, caches, act["kv_len"], K)
    engine.close()


@pytest.mark.parametrize("B", [17, 20, 40, 70, 130, 300])
def test_tiny_wide_batches(gpu, tiny, B):
    """Batches above 16 take tiled matrix products over all sequences, except for the down projection: the tiny head's
    reduction length there (d_ffn = 688) is no multiple of 32, which keeps it on the core whose waves split the tiles (two
    or four sequence tiles, the last one ragged; 70 sequences are two weight passes, 64 + 6, 130 three, 64 + 64 + 2), with
    row counts that leave most tile slots of a block empty."""
    wl = tiny["wl"]
    rng = np.random.default_rng(100 + B)
    ctx = rng.integers(0, 120, size=B).astype(np.int32)
    act = synth.make_activations(wl, ctx=ctx, capacity=192)
    ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, 3)
    check_chain(ref, res, caches, act["kv_len"], 3)


@pytest.mark.parametrize("B", [2, 3, 4])
def test_tiny_row_kernels_on_request(gpu, tiny, B):
    """Two to four sequences take the batched kernels by default; launch mode 3 keeps them on the row-streaming
    kernels (the form the library falls back to for matrices of 2 GiB or more): a K = 3 chain with ragged contexts,
    and a block of new positions whose rows (two per sequence where they fit) are row-streamed."""
    binding = gpu["binding"]
    wl = tiny["wl"]
    ctx = np.array([0, 63, 150, 7][:B], dtype=np.int32)
    act = synth.make_activations(wl, ctx=ctx, capacity=192)
    engine = binding.DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], B, 192, 3)
    assert binding.mtp_set_launch_mode(engine.handle, binding.LAUNCH_ROWS) == 0
    ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, 3, engine=engine)
    check_chain(ref, res, caches, act["kv_len"], 3)
    engine.close()
    if B == 2:
        engine = binding.DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], 4, 192, 1)
        assert binding.mtp_set_launch_mode(engine.handle, binding.LAUNCH_ROWS) == 0
        ext_len = np.array([2, 1], dtype=np.int32)
        hid, tok = extend_inputs(tiny["shape"], act, 2, 215)
        ref, res, caches = run_extend(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, hid, tok, ext_len,
                                      engine=engine)
        assert res["err"] == 0
        check_extend(ref, res, caches, act, ext_len)
        engine.close()


# head geometries that together instantiate every (query-group size, head dimension) variant of the attention kernels
GEOMETRIES = [(4, 4, 64), (8, 2, 64), (8, 1, 64), (2, 2, 128), (2, 1, 128), (4, 1, 128), (8, 1, 128)]


@pytest.mark.parametrize("hq,hkv,hd", GEOMETRIES)
@pytest.mark.parametrize("long_splits", [False, True])
def test_small_heads_every_attention_variant(gpu, hq, hkv, hd, long_splits):
    """Group sizes 1, 2, 4, 8 at head dimensions 64 and 128, each through the short-split vector attention (small
    cache capacity) and through the matrix-core attention with merged splits (large capacity), three sequences
    (row-streaming matrix phases) with ragged contexts, K = 2."""
    shape = synth.HeadShape(256, hq, hkv, hd, 512, 2048)
    wl = synth.Workload(f"sweep_{hq}_{hkv}_{hd}", 40 + hq + 3 * hkv + hd, shape, 3, 0, 0, (512,), 2, 0.5,
                        zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    ctx = np.array([0, 45, 700 if long_splits else 130], dtype=np.int32)
    # three sequences and hkv KV heads: a split holds capacity * 3 * hkv / 256 tokens (at least 128)
    cap = 768 if not long_splits else 256 * 256 // (3 * hkv) + 64
    act = synth.make_activations(wl, ctx=ctx, capacity=cap)
    ref, res, caches = run_both(gpu, shape, w, w, act, [ids], 0, 2)
    check_chain(ref, res, caches, act["kv_len"], 2)


@pytest.mark.parametrize("hq,hkv,hd", GEOMETRIES)
def test_small_heads_block_of_positions_shared_reads(gpu, hq, hkv, hd):
    """Blocks of new positions on every (group size, head dimension) variant of the matrix-core attention that serves
    16 / G positions of a sequence per item (sixteen, eight, four or two): 19 positions per sequence (a ragged last
    group everywhere), ragged counts including zero, a block that crosses a split boundary, an empty cache."""
    shape = synth.HeadShape(256, hq, hkv, hd, 512, 2048)
    wl = synth.Workload(f"block_{hq}_{hkv}_{hd}", 60 + hq + 3 * hkv + hd, shape, 4, 0, 0, (512,), 1, 0.5,
                        zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    cap, m = 16384, 19
    # 4 x 19 rows and hkv KV heads: splits of capacity * 76 * hkv / 256 tokens, capped at 4096
    ctx = np.array([4090, 0, 9000, 300], dtype=np.int32)
    ext_len = np.array([19, 19, 7, 0], dtype=np.int32)
    act = synth.make_activations(wl, ctx=ctx, capacity=cap)
    hid, tok = extend_inputs(shape, act, m, 77 + hq + hkv + hd)
    ref, res, caches = run_extend(gpu, shape, w, w, act, [ids], 0, hid, tok, ext_len)
    assert res["err"] == 0
    check_extend(ref, res, caches, act, ext_len)


@pytest.mark.parametrize("hq,hkv,hd", GEOMETRIES)
@pytest.mark.parametrize("d,ctx,ext,m", [
    (256, [0, 13, 96, 500], [19, 19, 7, 0], 19),   # row-major activations; rounds of 32 tokens per wave: several, one
    (256, [31, 109, 255, 125], [1, 19, 1, 4], 19), # or none; lengths on their edges, groups without a position
    (512, [127, 30], [3, 2], 3),                   # six rows in operand order
])
def test_small_heads_block_of_positions_in_small_workgroups(gpu, hq, hkv, hd, d, ctx, ext, m):
    """Blocks in caches of a few hundred slots: the attention whose small workgroups serve 16 / G positions each over all
    their tokens, on every (group size, head dimension); here with eight waves."""
    block_in_small_workgroups(gpu, hq, hkv, hd, d, ctx, ext, m)


@pytest.mark.parametrize("hq,hkv,hd", GEOMETRIES)
@pytest.mark.parametrize("ctx,ext,m", [([0, 13, 96, 500], [19, 19, 7, 0], 19), ([31, 109, 255, 125], [1, 19, 1, 4], 19)])
def test_blocks_of_positions_in_small_workgroups(gpu, hq, hkv, hd, ctx, ext, m):
    """The same blocks in caches of 2048 slots: with fewer, splits are short and the vector attention serves most of them (splits of
    capacity * rows * hkv / 256 tokens: the matrix cores from 449 on, up to the next 64)."""
    block_in_small_workgroups(gpu, hq, hkv, hd, 256, ctx, ext, m, cap=2048)


@pytest.mark.parametrize("hq,hkv,hd,ctx,ext,m", [
    (8, 8, 64, [127, 30], [4, 3], 4), (16, 8, 128, [127, 0], [4, 1], 4), (32, 8, 64, [700], [8], 8),     # up to eight rows, packed
    (4, 4, 64, [127, 30, 0, 900], [4, 4, 2, 0], 4), (16, 4, 128, [500, 64], [8, 5], 8),                  # up to sixteen
])
def test_blocks_of_few_rows_in_small_workgroups(gpu, hq, hkv, hd, ctx, ext, m):
    """The same attention, its results in the operand order of the kernel of up to sixteen rows."""
    block_in_small_workgroups(gpu, hq, hkv, hd, 512, ctx, ext, m, cap=2048)


@pytest.mark.parametrize("hq,hkv,hd,ctx,m,cap", [
    (8, 2, 64, [100], 4, 2112), (8, 1, 128, [2000], 6, 2112), (32, 8, 128, [511], 4, 2112), (4, 4, 64, [60, 0, 130], 2, 192)])
def test_a_later_position_that_is_not_finite_leaves_the_earlier_ones_alone(gpu, hq, hkv, hd, ctx, m, cap):
    """Blocks with short splits: the earlier positions' outputs are the same bits whatever stands at the last one."""
    last_position_not_finite(gpu, hq, hkv, hd, ctx, m, cap, m - 1)


@pytest.mark.parametrize("hq,hkv,hd", [(8, 8, 64), (8, 8, 128)])
def test_a_position_that_is_not_finite_stays_in_its_round(gpu, hq, hkv, hd):
    """On the matrix cores sixteen positions share the rounds of 32 tokens they read: what is not finite reaches those with tokens
    in the same round (0 x infinity), and no other.  The sixteenth position is the fourth token of the second round."""
    last_position_not_finite(gpu, hq, hkv, hd, [20], 16, 2048, 12)


def last_position_not_finite(gpu, hq, hkv, hd, ctx, m, cap, same):
    binding = gpu["binding"]
    shape = synth.HeadShape(512, hq, hkv, hd, 512, 2048)
    wl = synth.Workload(f"finite_{hq}_{hkv}_{hd}", 90 + hq + hd, shape, len(ctx), 0, 0, (512,), 1, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    act = synth.make_activations(wl, ctx=np.array(ctx, dtype=np.int32), capacity=cap)
    hid, tok = extend_inputs(shape, act, m, 91)
    eng = binding.DraftEngine(shape, w, [ids], len(ctx) * m, cap, 1)
    got = []
    for last in (None, 0x7fc0, 0x7f80):  # as drawn, NaN, infinity
        if last is not None:
            hid[m - 1] = last
        out = eng.extend(0, eng.to_device_bits(hid), eng.to_device_i32(tok), eng.to_device_i32(np.full(len(ctx), m, np.int32)),
                         eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"]), eng.to_device_i32(act["kv_len"]),
                         want_logits=True, want_hidden=True)
        got.append({k: out[k].cpu().numpy()[:same] for k in ("logits", "hidden", "draft")})
    eng.close()
    assert np.isfinite(got[0]["logits"]).all()
    for other in got[1:]:
        for k in got[0]:
            np.testing.assert_array_equal(got[0][k], other[k])


@pytest.mark.parametrize("hkv,hd", [(2, 64), (4, 64), (8, 64), (16, 64), (2, 128), (4, 128), (8, 128), (16, 128)])
def test_small_heads_long_blocks_in_smaller_workgroups(gpu, hkv, hd):
    """More (sequence, KV head, 16 / G positions) than compute units: four waves each."""
    groups = 7 * hkv * -(-73 * (16 // hkv) // 16)
    assert groups > 256
    block_in_small_workgroups(gpu, 16, hkv, hd, 256, [0, 55, 127, 1, 30, 64, 90], [73, 73, 1, 0, 40, 64, 73], 73)


@pytest.mark.parametrize("hkv,hd", [(2, 64), (4, 64), (8, 64), (16, 64), (2, 128), (4, 128), (8, 128), (16, 128)])
def test_long_blocks_in_smaller_workgroups(gpu, hkv, hd):
    """The same in caches of 2048 slots."""
    block_in_small_workgroups(gpu, 16, hkv, hd, 256, [0, 55, 127, 1, 30, 64, 90], [73, 73, 1, 0, 40, 64, 73], 73, cap=2048)


@pytest.mark.parametrize("hq,hkv,hd", GEOMETRIES + [(16, 8, 64), (16, 16, 128)])
def test_small_workgroups_give_the_bits_of_the_splits(gpu, hq, hkv, hd):
    """A cache of 1024 slots (small workgroups: of eight waves, in the last two cases of four) and one of 16448 (splits of 4096
    tokens, each of these contexts is one): the same tokens in eight sums, so the same bits."""
    torch, binding = gpu["torch"], gpu["binding"]
    m, short, long = 73, 1024, 16448
    ctx = np.array([0, 55, 127, 1, 950, 300][:6 if hkv >= 8 else 3] + [900], dtype=np.int32)
    groups = len(ctx) * hkv * -(-m * (hq // hkv) // 16)
    assert len(ctx) * m > 128 and (groups > 256) == (hkv >= 8)  # splits not sized by the lengths; waves of a workgroup
    shape = synth.HeadShape(256, hq, hkv, hd, 512, 2048)
    wl = synth.Workload(f"bits_{hq}_{hkv}_{hd}", 170 + hq + 3 * hkv + hd, shape, len(ctx), 0, 0, (512,), 1, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    act = synth.make_activations(wl, ctx=ctx, capacity=short)
    hid, tok = extend_inputs(shape, act, m, 171)
    ext_len = np.array([m, 60, m, 0, m, 19][:len(ctx) - 1] + [40], dtype=np.int32)
    got = []
    for cap in (short, long):
        eng = binding.DraftEngine(shape, w, [ids], len(ctx) * m, cap, 1)
        caches = []
        for name in ("k_cache", "v_cache"):
            c = torch.zeros((len(ctx), hkv, cap, hd), dtype=torch.int16, device="cuda:0")
            c[:, :, :short] = eng.to_device_bits(act[name])
            caches.append(c)
        out = eng.extend(0, eng.to_device_bits(hid), eng.to_device_i32(tok), eng.to_device_i32(ext_len), *caches,
                         eng.to_device_i32(act["kv_len"]), want_logits=True, want_hidden=True)
        live = np.arange(m)[:, None] < ext_len[None, :]
        got.append([out[k].cpu().numpy()[live] for k in ("logits", "hidden", "draft")])
        eng.close()
    assert np.isfinite(got[0][0]).all()
    for small, split in zip(*got):
        np.testing.assert_array_equal(small, split)


def test_more_rounds_in_small_workgroups(gpu):
    """Up to 40 rounds of 128 tokens where the splits are not sized by the lengths found: one context fills the cache."""
    block_in_small_workgroups(gpu, 8, 8, 64, 256, [5102, 0, 127, 3000] * 5, [18, 19, 1, 4] * 5, 19, cap=5120)


def block_in_small_workgroups(gpu, hq, hkv, hd, d, ctx, ext, m, cap=576):
    shape = synth.HeadShape(d, hq, hkv, hd, 512, 2048)
    wl = synth.Workload(f"small_{hq}_{hkv}_{hd}", 70 + hq + 3 * hkv + hd, shape, len(ctx), 0, 0, (512,), 1, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    ext_len = np.array(ext, dtype=np.int32)
    act = synth.make_activations(wl, ctx=np.array(ctx, dtype=np.int32), capacity=cap)
    hid, tok = extend_inputs(shape, act, m, 79 + hq + hkv + hd)
    ref, res, caches = run_extend(gpu, shape, w, w, act, [ids], 0, hid, tok, ext_len)
    assert res["err"] == 0
    check_extend(ref, res, caches, act, ext_len)


@pytest.mark.parametrize("B", [1, 3, 12, 40])
def test_activations_are_split_after_they_are_rounded(gpu, B):
    """A normalised input x = g * (h * inv) goes through the products as bf16(x) + bf16(x - bf16(x)) of the float x.  The projection picks its
    elements one by one and all else is zero, so that the step's output is that sum times one number; inputs are multiples of 1/16,
    whose squares add up exactly in any order, so inv is known to the bit.  The output's scale and two roundings stay within 2^-22;
    a lo half that rounds the other way is off by up to 2^-16."""
    binding = gpu["binding"]
    d = 1024
    shape = synth.HeadShape(d, 8, 8, 128, 512, 2048)
    rng = np.random.default_rng(600 + B)
    w = {k: np.zeros(s, np.float32) for k, s in synth.weight_shapes(shape).items()}
    for k in w:
        if k.startswith("g_"):
            w[k][:] = 1.0
    w["g_hnorm"] = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(rng.uniform(0.5, 2.0, d).astype(np.float32)))
    w["w_proj"][np.arange(d), np.arange(d)] = 1.0
    w["embed"][:] = 1.0
    eng = binding.DraftEngine(shape, {k: synth.f32_to_bf16_bits(v) for k, v in w.items()}, [np.arange(512, dtype=np.int32)], B, 64, 1)
    zero = eng.to_device_bits(np.zeros((B, 8, 64, 128), np.uint16))
    for _ in range(1 + 40 // B):
        h = (rng.integers(1, 64, (B, d)) * rng.choice([-1, 1], (B, d)) / 16).astype(np.float32)
        mean = ((h.astype(np.float64) ** 2).sum(-1) / d).astype(np.float32)
        inv = np.float32(1) / np.sqrt(mean + np.float32(shape.rms_eps))
        x = w["g_hnorm"] * (h * inv[:, None])
        hi = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x))
        want = (hi + synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(x - hi))).astype(np.float64)
        out = eng.draft(1, 0, eng.to_device_bits(synth.f32_to_bf16_bits(h)), eng.to_device_i32(np.zeros(B)), zero.clone(), zero.clone(),
                        eng.to_device_i32(np.zeros(B)), want_hidden=True)
        ratio = out["hidden"].cpu().numpy()[:, 0].astype(np.float64) / want
        assert np.abs(ratio / np.median(ratio, axis=-1, keepdims=True) - 1).max() <= 2.0 ** -22
    eng.close()


def test_tiny_full_vocab_equals_identity_subset(gpu, tiny):
    """Eq. (3) with the identity list is the full head: same logits bit for bit on the device as well."""
    act = tiny["act"]
    V = tiny["shape"].vocab_size
    ident = np.arange(V, dtype=np.int32)
    ref, res_full, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [ident], -1, 2)
    check_chain(ref, res_full, caches, act["kv_len"], 2)
    _, res_id, _ = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [ident], 0, 2)
    np.testing.assert_array_equal(res_full["logits"], res_id["logits"])
    np.testing.assert_array_equal(res_full["draft"], res_id["draft"])


def test_tiny_without_bias_and_single_step(gpu, tiny):
    w = {k: v for k, v in tiny["w"].items() if not k.startswith("b_")}
    act = tiny["act"]
    ref, res, caches = run_both(gpu, tiny["shape"], w, w, act, [tiny["ids"]], 0, 1)
    check_chain(ref, res, caches, act["kv_len"], 1)


def test_tiny_ragged_subset_sizes(gpu, tiny):
    """Subset sizes that are not multiples of the 16-row tile, down to a single id."""
    act = tiny["act"]
    rng = np.random.default_rng(5)
    V = tiny["shape"].vocab_size
    subsets = [np.sort(rng.choice(V, size=n, replace=False)).astype(np.int32) for n in (1, 17, 1000, 4095)]
    torch, binding = gpu["torch"], gpu["binding"]
    eng = binding.DraftEngine(tiny["shape"], tiny["w"], subsets, 1, act["kv_capacity"], 2)
    for si in range(len(subsets)):
        ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, subsets, si, 2, engine=eng)
        if subsets[si].size > 1:
            check_chain(ref, res, caches, act["kv_len"], 2)
        else:
            assert (res["draft"] == subsets[si][0]).all()
    eng.close()


def test_tiny_determinism(gpu, tiny):
    """Same inputs, repeated calls: identical ids and logits (the cross-workgroup argmax and the split merge are
    order-independent)."""
    torch, binding = gpu["torch"], gpu["binding"]
    act = synth.make_activations(tiny["wl"], ctx=np.array([150, 20, 77], dtype=np.int32), capacity=192)
    eng = binding.DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], 3, 192, 3)
    outs = []
    for _ in range(5):
        o = eng.draft(3, 0, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"]),
                      eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"]),
                      eng.to_device_i32(act["kv_len"]), want_logits=True)
        torch.cuda.synchronize()
        outs.append((o["draft"].cpu().numpy(), o["logits"].cpu().numpy()))
    for d, l in outs[1:]:
        np.testing.assert_array_equal(d, outs[0][0])
        np.testing.assert_array_equal(l, outs[0][1])
    eng.close()


def test_device_detected_errors(gpu, tiny):
    torch, binding = gpu["torch"], gpu["binding"]
    cap = 192
    act = synth.make_activations(tiny["wl"], ctx=np.array([100, 190], dtype=np.int32), capacity=cap)
    eng = binding.DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], 2, cap, 3)
    kc, vc = eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"])
    o = eng.draft(3, 0, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"]), kc, vc,
                  eng.to_device_i32(act["kv_len"]))
    torch.cuda.synchronize()
    assert eng.poll_error() == -9  # sequence 1: 190 + 3 > 192
    assert eng.poll_error() == 0   # the error word is cleared by the poll
    d = o["draft"].cpu().numpy()
    assert (d[1] == -1).all() and (d[0] >= 0).all()
    np.testing.assert_array_equal(kc.cpu().numpy().view(np.uint16)[1], act["k_cache"][1])  # cache untouched
    tok = act["token_in"].copy()
    tok[0] = tiny["shape"].vocab_size
    bad_tok = eng.draft(1, 0, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(tok), kc, vc,
                        eng.to_device_i32(np.array([100, 100])), want_logits=True)
    torch.cuda.synchronize()
    assert eng.poll_error() == -10
    # the id outside the vocabulary is reported and replaced by id 0: the call equals one that was given id 0
    bad_draft, bad_logits = bad_tok["draft"].cpu().numpy().copy(), bad_tok["logits"].cpu().numpy().copy()
    tok[0] = 0
    zero_tok = eng.draft(1, 0, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(tok), kc, vc,
                         eng.to_device_i32(np.array([100, 100])), want_logits=True)
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    np.testing.assert_array_equal(bad_draft, zero_tok["draft"].cpu().numpy())
    np.testing.assert_array_equal(bad_logits, zero_tok["logits"].cpu().numpy())
    # host-detected
    assert binding.mtp_draft_steps(eng.handle, 3, 1, 0, kc, kc, kc, vc, kc, None, kc, None, None) == -4
    assert binding.mtp_draft_steps(eng.handle, 1, 4, 0, kc, kc, kc, vc, kc, None, kc, None, None) == -5
    assert binding.mtp_draft_steps(eng.handle, 1, 1, 1, kc, kc, kc, vc, kc, None, kc, None, None) == -6
    assert binding.mtp_draft_steps(eng.handle, 1, 1, 0, None, kc, kc, vc, kc, None, kc, None, None) == -1
    assert binding.mtp_draft_steps(eng.handle, 1, 1, 0, kc.data_ptr() + 2, kc, kc, vc, kc, None, kc, None, None) == -2
    assert binding.mtp_accept(eng.handle, 1, 1, kc, kc, 2, kc, kc, kc, kc) == -11
    eng.close()
    # an invalid id list is refused at init
    bad = np.array([5, 5, 9], dtype=np.int32)
    with pytest.raises(binding.MTPError) as e:
        binding.DraftEngine(tiny["shape"], tiny["w"], [bad], 1, cap, 1)
    assert e.value.status == -6


def test_single_launch_mode_matches_oracle(gpu, tiny):
    """Launch mode 1 with several sequences against the oracle, ragged batch, two calls per engine.  (Mode 1 is the
    single cooperative launch for ONE sequence; a kernel that ran several sequences in one launch behind grid barriers
    was retired, so several sequences take the kernels of mode 0 whatever the mode says.)"""
    torch, binding = gpu["torch"], gpu["binding"]
    act = synth.make_activations(tiny["wl"], ctx=np.array([0, 130, 64], dtype=np.int32), capacity=192)
    eng = binding.DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], 3, 192, 3)
    assert binding.mtp_set_launch_mode(eng.handle, binding.LAUNCH_SINGLE) == 0
    for _ in range(2):  # twice: the barrier counters carry over from call to call
        ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, 3, engine=eng)
        check_chain(ref, res, caches, act["kv_len"], 3)
    assert binding.mtp_set_launch_mode(eng.handle, 7) == -11
    assert binding.mtp_set_launch_mode(eng.handle, -1) == -11
    eng.close()


ROW_GEOMETRIES = [(8, 8, 64), (8, 4, 64), (8, 2, 64), (8, 1, 64), (4, 4, 128), (4, 2, 128), (4, 1, 128), (8, 1, 128)]


@pytest.mark.parametrize("hq,hkv,hd", ROW_GEOMETRIES)
def test_single_launch_one_sequence_row_streaming(gpu, hq, hkv, hd):
    """One sequence with every reduction at least 512 long takes the single-launch kernel on the row-streaming core.
    Group sizes 1, 2, 4, 8 at both head dimensions; d_ffn = 688 is not a multiple of the 512-element row block; an
    empty cache, a context inside one split (capacity 192) and several merged splits (capacity 768); every engine is
    called twice, so the barrier counters carry over.  With one sequence and three steps a case may have no step
    whose winner is clear of the runner-up; the ids are then only compared where it is."""
    binding = gpu["binding"]
    shape = synth.HeadShape(512, hq, hkv, hd, 688, 2048)
    wl = synth.Workload(f"rows_{hq}_{hkv}_{hd}", 70 + hq + 3 * hkv + hd, shape, 1, 0, 0, (512,), 3, 0.5,
                        zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    for ctx, cap, K in ((0, 192, 2), (150, 192, 3), (700, 768, 3)):
        act = synth.make_activations(wl, ctx=np.array([ctx], dtype=np.int32), capacity=cap)
        eng = binding.DraftEngine(shape, w, [ids], 1, cap, K)
        assert binding.mtp_set_launch_mode(eng.handle, binding.LAUNCH_SINGLE) == 0
        for _ in range(2):
            ref, res, caches = run_both(gpu, shape, w, w, act, [ids], 0, K, engine=eng)
            check_chain(ref, res, caches, act["kv_len"], K, need_clear=False)
        eng.close()


@pytest.mark.parametrize("hq,hkv,hd", [(8, 1, 64), (8, 1, 128), (4, 2, 128), (8, 8, 64)])
@pytest.mark.parametrize("splits", [1, 2, 16, 33, 63])
def test_single_launch_merges_of_many_splits(gpu, hq, hkv, hd, splits):
    """The first step's context fills its splits of 128 tokens, the second one's last split is the new token alone; an
    output's partials then lie in one row of lanes (up to 16 splits), in a wave, or beyond one."""
    binding = gpu["binding"]
    cap = 128 * 64 // hkv
    ctx = min(128 * splits, cap - 128) - 1
    shape = synth.HeadShape(512, hq, hkv, hd, 688, 2048)
    wl = synth.Workload(f"splits_{hq}_{hkv}_{hd}", 170 + hq + hd + splits, shape, 1, 0, 0, (512,), 3, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    act = synth.make_activations(wl, ctx=np.array([ctx], dtype=np.int32), capacity=cap)
    eng = binding.DraftEngine(shape, w, [ids], 1, cap, 3)
    assert binding.mtp_set_launch_mode(eng.handle, binding.LAUNCH_SINGLE) == 0
    for _ in range(2):
        ref, res, caches = run_both(gpu, shape, w, w, act, [ids], 0, 3, engine=eng)
        check_chain(ref, res, caches, act["kv_len"], 3, need_clear=False)
    eng.close()


@pytest.mark.parametrize("d_ffn", [1288, 3400])
def test_single_launch_gate_and_up_rows_left_over(gpu, d_ffn):
    """The gate and up rows beyond whole rounds of the grid's 2048 waves are dealt singly; where more than 1024 of each
    are left over (1288 without a round of pairs, 1352 behind one) they take two rounds of the waves."""
    binding = gpu["binding"]
    shape = synth.HeadShape(512, 4, 2, 128, d_ffn, 2048)
    wl = synth.Workload(f"ffn_{d_ffn}", 90 + d_ffn % 7, shape, 1, 0, 0, (512,), 3, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    act = synth.make_activations(wl, ctx=np.array([70], dtype=np.int32), capacity=192)
    eng = binding.DraftEngine(shape, w, [synth.make_subsets(wl)[0]], 1, 192, 3)
    for _ in range(2):
        ref, res, caches = run_both(gpu, shape, w, w, act, [synth.make_subsets(wl)[0]], 0, 3, engine=eng)
        check_chain(ref, res, caches, act["kv_len"], 3, need_clear=False)
    eng.close()


@pytest.mark.parametrize("d,hq,hkv,hd,d_ffn", [(1024, 8, 4, 128, 3072), (1024, 8, 8, 64, 2600), (2048, 16, 8, 128, 6144), (2080, 16, 4, 128, 11008),
                                               (1536, 4, 1, 64, 256)])
def test_single_launch_phases_of_three_chunks(gpu, d, hq, hkv, hd, d_ffn):
    """Waves with three rows of one chunk (gate and up of 1024 wide heads; the narrow head's every 1536-row phase) or one row of three
    (their down projections, in chunks of two, four and eight blocks): the third chunk, in the LDS slot, has nothing requested behind it."""
    binding = gpu["binding"]
    shape = synth.HeadShape(d, hq, hkv, hd, d_ffn, 2048)
    wl = synth.Workload(f"three_{d}", 130 + d % 89, shape, 1, 0, 0, (512,), 3, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    act = synth.make_activations(wl, ctx=np.array([70], dtype=np.int32), capacity=192)
    eng = binding.DraftEngine(shape, w, [ids], 1, 192, 3)
    assert binding.mtp_set_launch_mode(eng.handle, binding.LAUNCH_SINGLE) == 0
    for _ in range(2):
        ref, res, caches = run_both(gpu, shape, w, w, act, [ids], 0, 3, engine=eng)
        check_chain(ref, res, caches, act["kv_len"], 3, need_clear=False)
    eng.close()


@pytest.mark.parametrize("d,hq,hkv,hd,d_ffn", [(256, 4, 4, 64, 256), (288, 2, 1, 128, 1000), (480, 8, 2, 64, 2048),
                                               (1024, 8, 4, 128, 520), (1056, 10, 5, 128, 4104), (2048, 16, 8, 128, 2600)])
@pytest.mark.parametrize("ctx,cap", [(0, 64), (250, 256), (300, 320), (317, 352), (700, 768)])
def test_single_launch_short_rows(gpu, d, hq, hkv, hd, d_ffn, ctx, cap):
    """Rows of one 512-element block or less, chunks of two, four and eight blocks, reductions that end inside a block;
    capacities of one split (two rounds of the attention) and of several."""
    binding = gpu["binding"]
    shape = synth.HeadShape(d, hq, hkv, hd, d_ffn, 2048)
    wl = synth.Workload(f"short_{d}", 110 + d % 97, shape, 1, 0, 0, (520,), 3, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    act = synth.make_activations(wl, ctx=np.array([ctx], dtype=np.int32), capacity=cap)
    eng = binding.DraftEngine(shape, w, [ids], 1, cap, 3)
    for _ in range(2):
        ref, res, caches = run_both(gpu, shape, w, w, act, [ids], 0, 3, engine=eng)
        check_chain(ref, res, caches, act["kv_len"], 3, need_clear=False)
    eng.close()


def narrow_engine(gpu, d, hq, hkv, hd, d_ffn, ctx, cap, seed):
    """A one-sequence engine of a head with a reduction below 512, and its call on a stream (outputs on the device)."""
    torch, binding = gpu["torch"], gpu["binding"]
    shape = synth.HeadShape(d, hq, hkv, hd, d_ffn, 2048)
    wl = synth.Workload(f"narrow_{d}_{seed}", 130 + seed, shape, 1, 0, 0, (520,), 3, 0.5, zipf_subset=False)
    act = synth.make_activations(wl, ctx=np.array([ctx], dtype=np.int32), capacity=cap)
    eng = binding.DraftEngine(shape, synth.make_weights(wl), [synth.make_subsets(wl)[0]], 1, cap, 3)
    hid, tok, kv = eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"]), eng.to_device_i32(act["kv_len"])
    k0, v0 = eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"])
    torch.cuda.synchronize()

    def call(stream=0, steps=3):
        kc, vc = k0.clone(), v0.clone()
        out = eng.draft(steps, 0, hid, tok, kc, vc, kv, want_logits=True, want_hidden=True, stream=stream)
        return [out["draft"], out["logits"], out["hidden"], kc, vc]

    return eng, call


@pytest.mark.parametrize("d,hq,hkv,hd,d_ffn", [(256, 4, 2, 64, 688), (480, 4, 1, 64, 776), (256, 16, 4, 128, 256),
                                               (256, 40, 10, 64, 256)])  # (chunks of 2, 2, 4 and 8 KiB)
@pytest.mark.parametrize("ctx,cap", [(0, 64), (700, 768)])
def test_narrow_single_launch_gives_the_same_bits_alone(gpu, d, hq, hkv, hd, d_ffn, ctx, cap):
    """A narrow head's single launch whose workgroups are not all there in time is done by one of them: the same rows, splits
    and sums, so the same bits; before and after calls of all workgroups (the two admission words take turns)."""
    torch, binding = gpu["torch"], gpu["binding"]
    eng, call = narrow_engine(gpu, d, hq, hkv, hd, d_ffn, ctx, cap, 1)
    want = call()
    for ticks in (30000, 0, 0, 0, 30000, 1, 1, 30000, 0, 30000):
        assert binding.mtp_set_admission_ticks(eng.handle, ticks) == 0
        got = call()
        torch.cuda.synchronize()
        assert eng.poll_error() == 0
        assert all(torch.equal(a, b) for a, b in zip(want, got)), ticks
    assert binding.mtp_set_admission_ticks(eng.handle, -1) == -3
    eng.close()


@pytest.mark.parametrize("d,hq,hkv,hd,d_ffn", [(256, 4, 2, 64, 688), (1024, 8, 8, 128, 1024), (2048, 16, 8, 128, 8200)])
def test_single_launches_of_handles_that_share_a_workspace(gpu, d, hq, hkv, hd, d_ffn):
    """Handles that do not run concurrently may share a workspace: what one call of the single launch leaves in it (tags, arrivals)
    is not taken for another handle's."""
    torch, binding = gpu["torch"], gpu["binding"]
    engines = [narrow_engine(gpu, d, hq, hkv, hd, d_ffn, 300, 768, seed) for seed in (20, 21)]
    want = [[call(steps=k) for k in (1, 3)] for _, call in engines]
    torch.cuda.synchronize()
    shared = engines[0][0].workspace
    for eng, _ in engines:
        binding.mtp_draft_destroy(eng.handle)
        st, eng.handle = binding.mtp_draft_init(eng.cfg, eng.w, eng.subsets, [s.numel() for s in eng.subsets], shared,
                                                shared.numel())
        assert st == 0
    for k, turn in [(k, turn) for k in (0, 1) for turn in (0, 1, 0, 1, 1, 0)]:
        eng, call = engines[turn]  # (one step first: every vector keeps the tags of the call's only step)
        got = call(steps=(1, 3)[k])
        torch.cuda.synchronize()
        assert eng.poll_error() == 0
        assert all(torch.equal(a, b) for a, b in zip(want[turn][k], got)), (turn, k)
    for eng, _ in engines:
        eng.close()


def test_phase_trace_of_a_launch_on_a_quarter_of_the_units(gpu):
    """Stamps lie [step][section][point][compute units], also where the launch has fewer workgroups."""
    torch, binding = gpu["torch"], gpu["binding"]
    eng, call = narrow_engine(gpu, 256, 4, 2, 64, 688, 100, 192, 9)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    buf = torch.zeros(binding.mtp_phase_trace_bytes(eng.cfg) // 8, dtype=torch.int64, device="cuda:0")
    assert binding.mtp_set_phase_trace(eng.handle, buf) == 0
    call()
    torch.cuda.synchronize()
    n = 3 * len(binding.TRACE_SECTIONS) * len(binding.TRACE_POINTS)
    t = buf[:n * cus].view(n, cus).cpu()
    assert (t[:, :cus // 4] > 0).all() and (t[:, cus // 4:] == 0).all() and (buf[n * cus:] == 0).all().item()
    eng.close()


def test_narrow_single_launches_overlap_each_other_and_a_wide_one(gpu):
    """More calls in flight than the device has room for at a time, and one that wants every compute unit: nobody's wait
    depends on another call's, and everybody's result is that of a call by itself."""
    torch, binding = gpu["torch"], gpu["binding"]
    shapes = [(256, 4, 2, 64, 688), (480, 4, 1, 64, 776), (256, 16, 4, 128, 256), (256, 4, 2, 64, 688), (320, 4, 4, 128, 1024),
              (256, 2, 1, 128, 512), (1024, 8, 8, 128, 1024)]  # (the last: no reduction below 512)
    engines = [narrow_engine(gpu, *s, 300, 768, 2 + i) for i, s in enumerate(shapes)]
    want = [call() for _, call in engines]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in engines]
    got = []
    for turn in range(4):
        for (eng, call), st in zip(engines, streams):
            with torch.cuda.stream(st):
                got.append(call(st.cuda_stream))
    torch.cuda.synchronize()
    for i, g in enumerate(got):
        assert all(torch.equal(a, b) for a, b in zip(want[i % len(engines)], g)), i
    for eng, _ in engines:
        assert eng.poll_error() == 0
        eng.close()


# ------------------------------------------------------------------------------------------ block of new positions
def extend_inputs(shape, act, m_max, seed):
    """Position-major inputs of the multi-position first step: hidden states with the workload's spread, tokens."""
    rng = np.random.default_rng(seed)
    B = len(act["kv_len"])
    std = float(synth.bf16_bits_to_f32(act["hidden_in"]).std())
    hid = synth.f32_to_bf16_bits((rng.standard_normal((m_max, B, shape.d_model)) * std).astype(np.float32))
    tok = rng.integers(0, shape.vocab_size, size=(m_max, B)).astype(np.int32)
    return hid, tok


def run_extend(gpu, shape, w_host, w_dev, act, subsets, subset_index, hid, tok, ext_len, engine=None, seqs=None):
    """Oracle and library on the same block; returns (ref, res, (oracle caches), engine-side kv_len)."""
    torch, Oracle, binding = gpu["torch"], gpu["Oracle"], gpu["binding"]
    m_max, B = tok.shape
    cap = act["kv_capacity"]
    ids = None if subset_index < 0 else subsets[subset_index]
    sel = list(range(B)) if seqs is None else list(seqs)
    orc = Oracle(shape, w_host, cap, "f32")
    okc, ovc = act["k_cache"][sel].copy(), act["v_cache"][sel].copy()
    ref = orc.extend(np.ascontiguousarray(hid[:, sel]), np.ascontiguousarray(tok[:, sel]), ext_len[sel], okc, ovc,
                     act["kv_len"][sel], ids)
    own = engine is None
    if own:
        engine = binding.DraftEngine(shape, w_dev, subsets, B * m_max, cap, 1)
    dkc, dvc = engine.to_device_bits(act["k_cache"]), engine.to_device_bits(act["v_cache"])
    dkv = engine.to_device_i32(act["kv_len"])
    out = engine.extend(subset_index, engine.to_device_bits(hid), engine.to_device_i32(tok),
                        engine.to_device_i32(ext_len), dkc, dvc, dkv, want_logits=True, want_hidden=True)
    torch.cuda.synchronize()
    err = engine.poll_error()
    res = {"draft": out["draft"].cpu().numpy()[:, sel], "logits": out["logits"].cpu().numpy()[:, sel],
           "hidden": out["hidden"].cpu().numpy()[:, sel], "kv_len": dkv.cpu().numpy()[sel],
           "k_cache": dkc.cpu().numpy().view(np.uint16)[sel], "v_cache": dvc.cpu().numpy().view(np.uint16)[sel],
           "err": err}
    if own:
        engine.close()
    return ref, res, (okc, ovc)


def check_extend(ref, res, caches, act, ext_len, sel=None):
    okc, ovc = caches
    sel = list(range(len(ext_len))) if sel is None else list(sel)
    np.testing.assert_array_equal(res["kv_len"], ref["kv_len"])
    worst = 0.0
    for i, b in enumerate(sel):
        m, L = int(ext_len[b]), int(act["kv_len"][b])
        fits = L + m <= act["kv_capacity"]
        live = m if fits else 0
        assert (res["draft"][live:, i] == -1).all() and (ref["draft"][live:, i] == -1).all()
        if live:
            gap = float(np.abs(ref["logits"][:live, i] - res["logits"][:live, i]).max())
            worst = max(worst, gap)
            assert gap <= LOGIT_TIGHT, (b, gap)
            assert np.abs(ref["hidden"][:live, i] - res["hidden"][:live, i]).max() <= 2e-3
            clear = ref["margin"][:live, i] > MARGIN
            np.testing.assert_array_equal(ref["draft"][:live, i][clear], res["draft"][:live, i][clear])
        # cache: only the new slots change, and they match the oracle's up to one bf16 step
        assert np.array_equal(res["k_cache"][i][:, :L], okc[i][:, :L])
        assert np.array_equal(res["v_cache"][i][:, :L], ovc[i][:, :L])
        if live:
            assert appended_entries_close(res["k_cache"][i][:, L:L + live], okc[i][:, L:L + live])
            assert appended_entries_close(res["v_cache"][i][:, L:L + live], ovc[i][:, L:L + live])
        assert np.array_equal(res["k_cache"][i][:, L + live:], okc[i][:, L + live:])
        assert np.array_equal(res["v_cache"][i][:, L + live:], ovc[i][:, L + live:])
    return worst


@pytest.mark.parametrize("ctx,ext,m_max", [
    ([100], [3], 3),                         # three rows
    ([0, 60], [2, 1], 2),                    # four rows, one sequence starting from an empty cache
    ([0, 130, 64], [4, 0, 2], 4),            # twelve rows (batched matrix phases), ragged, one sequence idle
    ([5, 150, 64, 1, 99, 127], [5, 5, 1, 3, 0, 5], 5),   # thirty rows: two sequence tiles per weight tile
    ([0, 40, 7, 90], [70, 65, 0, 33], 70),   # 280 rows (a prompt's worth): the body's phases as tiled matrix products
])
def test_tiny_extend_block_of_positions(gpu, tiny, ctx, ext, m_max):
    """The first draft step over several new positions per sequence against the oracle's position-by-position
    result: logits, hidden states and drafts of every live position, the appended cache slots, the new kv_len."""
    act = synth.make_activations(tiny["wl"], ctx=np.array(ctx, dtype=np.int32), capacity=192)
    ext_len = np.array(ext, dtype=np.int32)
    hid, tok = extend_inputs(tiny["shape"], act, m_max, 200 + len(ctx))
    ref, res, caches = run_extend(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, hid, tok, ext_len)
    assert res["err"] == 0
    check_extend(ref, res, caches, act, ext_len)


@pytest.mark.parametrize("d_ffn,subset", [(1056, 0), (1064, -1)])
@pytest.mark.parametrize("rows", [5, 9, 16, 17, 33, 64, 65, 129, 257, 400])
def test_many_rows_tiled_matrix_products(gpu, d_ffn, subset, rows):
    """Every phase as a tiled matrix product (small reductions take it from nine rows on; five: few_rows.h), here in the tiles of 16
    rows and, from 257 rows on, of 32 (gate/up and the head): one block to twenty-five, full and ragged last ones.  The down
    projection of 1056 ends in half a step, that of 1064 in less than that (few_rows.h or the batched core then); gate/up rows and a
    vocabulary that end inside a tile of sixteen; the list and the full head; the candidates of a row from several
    blocks of weight rows.  The other tiles: the two tests below."""
    shape = synth.HeadShape(512, 4, 2, 128, d_ffn, 2111)
    wl = synth.Workload(f"rows_{d_ffn}", 95, shape, 1, 0, 0, (517,), 1, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    act = synth.make_activations(wl, ctx=np.array([40], dtype=np.int32), capacity=448)
    hid, tok = extend_inputs(shape, act, rows, 230 + rows)
    ext_len = np.array([rows], dtype=np.int32)
    ref, res, caches = run_extend(gpu, shape, w, w, act, [ids], subset, hid, tok, ext_len)
    assert res["err"] == 0
    check_extend(ref, res, caches, act, ext_len)


@pytest.mark.parametrize("d,rows,n", [(1024, 5, 3584), (1024, 12, 3584), (2048, 16, 8192), (1024, 20, 8192), (1024, 64, 3584), (2048, 20, 8192),
                                      (2048, 100, 8192), (2048, 192, 8192), (4096, 5, 3584), (4096, 20, 8192),
                                      (4096, 40, 8192), (4096, 100, 8192), (4096, 192, 3584)])
def test_tiled_products_add_up_as_exactly_as_the_batched_core(gpu, d, rows, n):
    """The output head on activations that the bf16 pairs hold exactly (x = +-w of a diagonal projection, no attention, no
    MLP: eight bits of mantissa, times a gain of eight), so that its logits are off by the rounding of the sums alone,
    up to the row's norm scale, which is fitted away.  Every kernel adds d products of each half in single precision; how
    often a large partial sum is rounded is up to the order.  The batched core, whose waves and parts add up short
    chains, is 1.0 to 1.9e-7 off at these sizes (rms, of the logits' rms); one chain of matrix instructions over a whole
    reduction, lo halves and all, 2.0 to 3.8e-7."""
    binding = gpu["binding"]
    rng = np.random.default_rng(31)
    shape = synth.HeadShape(d, 4, 2, 64, 256, n, rms_eps=0.0)
    w = {k: np.zeros(s, np.float32) for k, s in synth.weight_shapes(shape).items()}
    for k in w:
        if k.startswith("g_") or k == "embed":
            w[k][:] = 1.0
    w["w_proj"][np.arange(d), np.arange(d)] = 1.0 + 0.3 * rng.standard_normal(d)
    w["lm_head"] = rng.standard_normal((n, d)).astype(np.float32) * 0.02
    w["g_final_norm"] = (1.0 + 0.3 * rng.standard_normal(d)).astype(np.float32)
    w = {k: synth.f32_to_bf16_bits(v) for k, v in w.items()}
    f64 = {k: synth.bf16_bits_to_f32(w[k]).astype(np.float64) for k in ("w_proj", "lm_head", "g_final_norm")}
    h = np.where(rng.random((rows, d)) < 0.5, -1.0, 1.0).astype(np.float32)
    ref = (h * np.diag(f64["w_proj"]) * f64["g_final_norm"]) @ f64["lm_head"].T
    eng = binding.DraftEngine(shape, w, [], rows, 64, 1)

    def error(B):
        cache = [gpu["torch"].zeros((rows, 2, 64, 64), dtype=gpu["torch"].bfloat16, device="cuda") for _ in range(2)]
        out = eng.draft(1, -1, eng.to_device_bits(synth.f32_to_bf16_bits(h[:B])), eng.to_device_i32(np.zeros(B, np.int32)),
                        *cache, eng.to_device_i32(np.zeros(B, np.int32)), want_logits=True)
        assert eng.poll_error() == 0
        z = out["logits"][:, 0].cpu().numpy().astype(np.float64)
        z /= (z * ref[:B]).sum(1, keepdims=True) / (ref[:B] ** 2).sum(1, keepdims=True)
        return np.sqrt(((z - ref[:B]) ** 2).mean() / (ref[:B] ** 2).mean())

    err = error(rows)
    eng.close()
    print(f"rms error {err:.2e}")
    assert err <= 1.9e-7, err


@pytest.mark.parametrize("rows", [5, 12, 17, 33, 64, 100, 200])
def test_widths_that_end_inside_a_reduction_step(gpu, rows):
    """d = 544 and d_ffn = 1056: every reduction but the output projection's is 32 modulo 64, the tiles for few rows (from nine on
    here) walk it in steps of 64 (the weights behind a row's end are the next row's, the activations the next phase's)."""
    shape = synth.HeadShape(544, 4, 2, 128, 1056, 2111)
    wl = synth.Workload("width_544", 96, shape, 1, 0, 0, (517,), 1, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    act = synth.make_activations(wl, ctx=np.array([40], dtype=np.int32), capacity=256)
    hid, tok = extend_inputs(shape, act, rows, 330 + rows)
    ext_len = np.array([rows], dtype=np.int32)
    for subset in (0, -1):
        ref, res, caches = run_extend(gpu, shape, w, w, act, [ids], subset, hid, tok, ext_len)
        assert res["err"] == 0
        check_extend(ref, res, caches, act, ext_len)


def run_block_of_one_sequence(gpu, shape, rows, seed):
    """A block of `rows` positions of one sequence with a short context, full vocabulary, against the oracle."""
    wl = synth.Workload(f"block_{shape.d_model}_{rows}", 97, shape, 1, 0, 0, (min(517, shape.vocab_size),), 1, 0.5,
                        zipf_subset=False)
    w = synth.make_weights(wl)
    act = synth.make_activations(wl, ctx=np.array([40], dtype=np.int32), capacity=-(-(rows + 40) // 64) * 64)
    hid, tok = extend_inputs(shape, act, rows, seed)
    ext_len = np.array([rows], dtype=np.int32)
    ref, res, caches = run_extend(gpu, shape, w, w, act, [synth.make_subsets(wl)[0]], -1, hid, tok, ext_len)
    assert res["err"] == 0
    check_extend(ref, res, caches, act, ext_len)


@pytest.mark.parametrize("d,vocab,rows", [c[:3] for c in HEAD_TILES])
def test_drafts_from_every_tile_of_the_output_head(gpu, d, vocab, rows):
    """The head's candidates from each of the tiles, in one part (one candidate per block of weight rows) and in several (one
    per group of the launch that adds the parts): drafts and logits.  test_rows_plan.py holds the tile of each case."""
    run_block_of_one_sequence(gpu, synth.HeadShape(d, 4, 2, 64, 256, vocab), rows, 400 + rows)


@pytest.mark.parametrize("d,d_ffn,rows", [c[:3] for c in BODY_TILES])
def test_body_phases_in_the_larger_tiles(gpu, d, d_ffn, rows):
    """The projections, gate/up and down in tiles of 16 to 256 rows, whole and split (their tiles: test_rows_plan.py)."""
    run_block_of_one_sequence(gpu, synth.HeadShape(d, d // 128, d // 256, 128, d_ffn, 2111), rows, 500 + rows)


# d_model, query / KV heads of 128, d_ffn, vocabulary: weight tiles per workgroup of the phases (256 workgroups at most)
FEW_ROWS_SHAPES = [
    (384, 2, 1, 264, 2111),      # two chunks of the reduction (264 = 256 + 8) to three, idle waves, one tile
    (416, 2, 2, 1000, 8000),     # reductions that end inside a chunk; head: two tiles
    (384, 4, 4, 8200, 24000),    # gate/up: three pairs (six tiles); head: six
    (384, 2, 2, 16400, 70000),   # gate/up: five pairs (two groups); head: eighteen tiles, three groups, the last ragged
    # narrower: the down projection (reductions that are no multiple of 32) with row-major activations, the rest in tiles
    (256, 2, 1, 264, 2111),
    (288, 4, 1, 1000, 8000),
    (544, 4, 2, 4104, 16000),    # gate/up: two pairs in one workgroup, one in the others; head: four tiles
    (256, 4, 4, 8200, 24000),
    (256, 2, 2, 16400, 70000),
    (2304, 4, 1, 1032, 33000),   # 9..16 rows in operand order; head: nine tiles
    (4128, 33, 33, 264, 2111),   # projections: two tiles; q/k/v: four
]


@pytest.mark.parametrize("d,hq,hkv,d_ffn,vocab", FEW_ROWS_SHAPES)
@pytest.mark.parametrize("rows", [2, 8, 9, 16])
def test_few_rows_every_tile_count(gpu, d, hq, hkv, d_ffn, vocab, rows):
    """2 to 16 rows, full vocabulary and a list of odd size: hi and lo halves in one operand (up to 8 rows) and in two."""
    shape = synth.HeadShape(d, hq, hkv, 128, d_ffn, vocab)
    wl = synth.Workload(f"few_{d}_{d_ffn}", 99, shape, 1, 0, 0, (vocab // 2 + 1,), 1, 0.5, zipf_subset=False)
    w = synth.make_weights(wl)
    ids = synth.make_subsets(wl)[0]
    act = synth.make_activations(wl, ctx=np.array([40], dtype=np.int32), capacity=64)
    hid, tok = extend_inputs(shape, act, rows, 600 + rows)
    ext_len = np.array([rows], dtype=np.int32)
    for subset in (0, -1):
        ref, res, caches = run_extend(gpu, shape, w, w, act, [ids], subset, hid, tok, ext_len)
        assert res["err"] == 0
        check_extend(ref, res, caches, act, ext_len)


@pytest.fixture(scope="module")
def huge_vocab():
    """More output-head rows than the tiled products have room for candidates (1024 blocks of 512), a ragged last tile."""
    shape = synth.HeadShape(256, 4, 2, 64, 256, 524309)
    wl = synth.Workload("huge_vocab", 98, shape, 1, 0, 0, (517,), 1, 0.5, zipf_subset=False)
    return wl, synth.make_weights(wl)


@pytest.mark.parametrize("rows", [3, 16, 20, 40])
def test_heads_beyond_the_tiles_candidates_stay_on_the_batched_core(gpu, huge_vocab, rows):
    """Two and four sequence tiles of the core whose waves split the weight tiles; up to sixteen rows few_rows.h, with row-major
    activations."""
    wl, w = huge_vocab
    act = synth.make_activations(wl, ctx=np.array([9], dtype=np.int32), capacity=64)
    hid, tok = extend_inputs(wl.shape, act, rows, 600 + rows)
    ext_len = np.array([rows], dtype=np.int32)
    ref, res, caches = run_extend(gpu, wl.shape, w, w, act, [synth.make_subsets(wl)[0]], -1, hid, tok, ext_len)
    assert res["err"] == 0
    check_extend(ref, res, caches, act, ext_len)


def test_tiny_extend_long_capacity_matrix_core_attention(gpu, tiny):
    """A large capacity makes the splits long enough for the matrix-core attention (which merges its own splits)."""
    act = synth.make_activations(tiny["wl"], ctx=np.array([0, 31, 300, 1000], dtype=np.int32), capacity=32768)
    ext_len = np.array([3, 2, 3, 1], dtype=np.int32)
    hid, tok = extend_inputs(tiny["shape"], act, 3, 210)
    ref, res, caches = run_extend(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, hid, tok, ext_len)
    assert res["err"] == 0
    check_extend(ref, res, caches, act, ext_len)


def length_sized_splits(cap, rows, kv_heads, lens, groups=1, units=256):
    """Tokens per split where the attention sizes its splits by the lengths it finds (restated from the plan: splits for the
    capacity, from 1024 tokens on; at most four times as many, in 64 candidate lengths, the first that gives no more
    items than there are compute units), and which candidate that is; (0, 0) where splits stay as planned."""
    def up64(x):
        return (x + 63) // 64 * 64
    planned = min(up64(max(-(-cap * rows * kv_heads // 256), 128)), 4096)
    if planned < 1024:
        return 0, 0
    first = max(256, up64(-(-cap // max(4 * -(-cap // planned), 16))))
    step = max(64, up64((cap - first + 62) // 63))
    for lane in range(64):
        t = first + lane * step
        if sum(-(-n // t) for n in lens) * kv_heads * groups <= units:
            return t, lane
    raise AssertionError("the last candidate covers the capacity")


@pytest.mark.parametrize("ctx,ext,tokens,lane", [
    # nine sequences, the shortest splits: steps that end on, before and behind a split's last token
    ([573, 574, 575, 576, 0, 31, 1150, 1151, 5000], None, 576, 0),
    # too many items for the shortest: a longer candidate; caches that the last step fills, ends at its multiples
    ([32765, 32765, 32765, 1085, 1086, 1087, 2174, 3262, 20670], None, 1088, 1),
    # four: the shortest splits there are
    ([253, 254, 255, 256], None, 256, 0),
    ([32765, 32765, 830, 2495], None, 832, 1),
    # one and two sequences: as planned
    ([32700, 1], None, 0, 0),
    ([0], None, 0, 0),
    # blocks of positions that cross a split's end, an idle sequence
    ([1015, 0, 2041, 1023, 40], [12, 12, 7, 0, 1], 1024, 0),
    # the same with a longer candidate, and blocks that fill their cache
    ([32756, 32756, 32000, 2043, 40], [12, 12, 12, 12, 1], 2048, 2),
])
def test_tiny_attention_splits_sized_by_the_lengths(gpu, tiny, ctx, ext, tokens, lane):
    """Few sequences in a large cache: the matrix-core attention sizes its splits by the lengths it finds, one item per
    workgroup.  Two sequences at least, so that the draft steps take the batched path; a single one in the
    launch-per-phase mode."""
    cap, kv_heads, K = 32768, tiny["shape"].n_kv_heads, 3
    for step in range(1 if ext else K):
        lens = [c + (e if ext else step + 1) for c, e in zip(ctx, ext or ctx) if not ext or e]
        rows, groups = (len(ctx) * 12, 2) if ext else (len(ctx), 1)  # (8 of a block's 12 positions beside 2 query heads)
        assert length_sized_splits(cap, rows, kv_heads, lens, groups) == (tokens, lane)
    act = synth.make_activations(tiny["wl"], ctx=np.array(ctx, dtype=np.int32), capacity=cap)
    if ext is not None:
        ext_len = np.array(ext, dtype=np.int32)
        hid, tok = extend_inputs(tiny["shape"], act, 12, 214)
        ref, res, caches = run_extend(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, hid, tok, ext_len)
        assert res["err"] == 0
        check_extend(ref, res, caches, act, ext_len)
        return
    eng = gpu["binding"].DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], len(ctx), cap, K)
    assert gpu["binding"].mtp_set_launch_mode(eng.handle, 0) == 0
    ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, K, engine=eng)
    check_chain(ref, res, caches, act["kv_len"], K, need_clear=False)
    eng.close()


def test_tiny_extend_long_block_positions_share_the_cache_reads(gpu, tiny):
    """Twenty positions per sequence with splits of 4096 tokens: the matrix-core attention serves eight positions of
    a sequence per item (three groups, the last ragged), each position seeing the cache up to its own slot.  One block
    crosses a split boundary (positions 4090 .. 4109: the later ones have a second split, the earlier ones not), one
    sequence starts empty, one sits deep in its cache, one is idle, one has a block shorter than a group."""
    act = synth.make_activations(tiny["wl"], ctx=np.array([4090, 0, 12000, 77, 8191], dtype=np.int32), capacity=32768)
    ext_len = np.array([20, 20, 13, 0, 3], dtype=np.int32)
    hid, tok = extend_inputs(tiny["shape"], act, 20, 212)
    ref, res, caches = run_extend(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, hid, tok, ext_len)
    assert res["err"] == 0
    check_extend(ref, res, caches, act, ext_len)


def test_tiny_extend_overflow_and_then_draft(gpu, tiny):
    """A block that does not fit leaves its sequence alone and is reported; the other sequence is extended, and the
    recursive draft steps that follow start from the extended cache on both sides."""
    torch, binding = gpu["torch"], gpu["binding"]
    cap = 192
    act = synth.make_activations(tiny["wl"], ctx=np.array([cap - 2, 80], dtype=np.int32), capacity=cap)
    ext_len = np.array([3, 3], dtype=np.int32)
    hid, tok = extend_inputs(tiny["shape"], act, 3, 220)
    eng = binding.DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], 6, cap, 3)
    ref, res, caches = run_extend(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, hid, tok, ext_len,
                                  engine=eng)
    assert res["err"] == -9 and ref["overflow"]
    check_extend(ref, res, caches, act, ext_len)
    # K = 3 recursive steps of sequence 1 from the extended caches (the oracle's own on its side)
    act2 = {"hidden_in": act["hidden_in"][1:], "token_in": act["token_in"][1:], "kv_len": ref["kv_len"][1:],
            "k_cache": caches[0][1:].copy(), "v_cache": caches[1][1:].copy(), "kv_capacity": cap}
    ref2, res2, caches2 = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act2, [tiny["ids"]], 0, 3, engine=eng)
    check_chain(ref2, res2, caches2, act2["kv_len"], 3, need_clear=False)
    eng.close()


def check_extend_then_continue(gpu, shape, w_host, w_dev, act, subsets, ext_len, m_max, K, seed, launch_mode=0,
                               seqs=None):
    """A block of new positions, then K recursive steps from the hidden state and draft of each sequence's last new
    position: the oracle by single steps fed back by hand, the library by mtp_draft_extend + mtp_draft_continue
    (fed its own hidden state, the oracle's tokens)."""
    torch, Oracle, binding = gpu["torch"], gpu["Oracle"], gpu["binding"]
    B = len(ext_len)
    cap = act["kv_capacity"]
    ids = subsets[0]
    sel = list(range(B)) if seqs is None else list(seqs)
    hid, tok = extend_inputs(shape, act, m_max, seed)
    eng = binding.DraftEngine(shape, w_dev, subsets, B * m_max, cap, K)
    ref, res, (okc, ovc) = run_extend(gpu, shape, w_host, w_dev, act, subsets, 0, hid, tok, ext_len, engine=eng,
                                      seqs=seqs)
    assert res["err"] == 0
    check_extend(ref, res, (okc, ovc), act, ext_len, sel=seqs)
    # the oracle's continuation, sequence by sequence, on its own extended caches
    orc = Oracle(shape, w_host, cap, "f32")
    cont = []
    for i, b in enumerate(sel):
        last = int(ext_len[b]) - 1
        cont.append(orc.chain_from_own_hidden(K, ref["hidden"][last, i], int(ref["draft"][last, i]), okc[i], ovc[i],
                                              int(ref["kv_len"][i]), ids))
    # the library's: engine state after the same extend
    dkc, dvc = eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"])
    dkv = eng.to_device_i32(act["kv_len"])
    ex = eng.extend(0, eng.to_device_bits(hid), eng.to_device_i32(tok), eng.to_device_i32(ext_len), dkc, dvc, dkv,
                    want_hidden=True)
    rows = torch.tensor([int(ext_len[b]) - 1 for b in range(B)], device="cuda:0")
    own = ex["hidden"][rows, torch.arange(B, device="cuda:0")].contiguous()          # [B][d], the library's own
    tok1 = np.zeros(B, np.int32)
    forced = np.zeros((B, max(K - 1, 1)), np.int32)
    for i, b in enumerate(sel):
        tok1[b] = ref["draft"][int(ext_len[b]) - 1, i]
        forced[b, :K - 1] = cont[i]["draft"][:K - 1]
    assert binding.mtp_set_launch_mode(eng.handle, launch_mode) == 0
    out = eng.draft_continue(K, 0, own, eng.to_device_i32(tok1), dkc, dvc, dkv,
                             forced=eng.to_device_i32(forced) if K > 1 else None, want_logits=True, want_hidden=True)
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    lg, hd, dr = out["logits"].cpu().numpy(), out["hidden"].cpu().numpy(), out["draft"].cpu().numpy()
    kc_after = dkc.cpu().numpy().view(np.uint16)
    worst = 0.0
    for i, b in enumerate(sel):
        gap = float(np.abs(lg[b] - cont[i]["logits"]).max())
        worst = max(worst, gap)
        assert gap <= LOGIT_TIGHT, (b, gap)
        assert np.abs(hd[b] - cont[i]["hidden"]).max() <= 2e-3
        clear = cont[i]["margin"] > MARGIN
        np.testing.assert_array_equal(dr[b][clear], cont[i]["draft"][clear])
        L = int(ref["kv_len"][i])
        assert appended_entries_close(kc_after[b][:, L:L + K], okc[i][:, L:L + K], recursive_from=0)
        assert np.array_equal(kc_after[b][:, L + K:], okc[i][:, L + K:])
    eng.close()
    return worst


def test_tiny_extend_then_continue(gpu, tiny):
    act = synth.make_activations(tiny["wl"], ctx=np.array([40, 0, 120], dtype=np.int32), capacity=192)
    check_extend_then_continue(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]],
                               np.array([3, 1, 2], dtype=np.int32), 3, 2, 240)
    # the same through the single-launch kernel of the recursive steps (tile core, three sequences)
    check_extend_then_continue(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]],
                               np.array([3, 1, 2], dtype=np.int32), 3, 2, 241, launch_mode=1)
    # seven sequences: batched kernels on both calls
    act = synth.make_activations(tiny["wl"], ctx=np.array([40, 0, 120, 7, 99, 64, 3], dtype=np.int32), capacity=192)
    check_extend_then_continue(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]],
                               np.array([2, 1, 2, 2, 1, 2, 1], dtype=np.int32), 2, 3, 242)


# ------------------------------------------------------------------------------------------ one id list per sequence
def check_lists(gpu, shape, w, lists, act, seq_subset, K):
    """A call with one list per sequence against the oracle run sequence by sequence, with its drafts forced.  Returns the engine."""
    torch, Oracle, binding = gpu["torch"], gpu["Oracle"], gpu["binding"]
    B, cap = len(seq_subset), act["kv_capacity"]
    orc = Oracle(shape, w, cap, "f32")
    refs, okc, ovc = [], act["k_cache"].copy(), act["v_cache"].copy()
    forced = np.zeros((B, K - 1), np.int32)
    for b in range(B):
        ids = None if seq_subset[b] < 0 else lists[seq_subset[b]]
        r = orc.chain(K, act["hidden_in"][b:b + 1], act["token_in"][b:b + 1], okc[b:b + 1], ovc[b:b + 1],
                      act["kv_len"][b:b + 1], ids)
        refs.append(r)
        forced[b] = r["draft"][0, :K - 1]
    eng = binding.DraftEngine(shape, w, lists, B, cap, K)
    dkc, dvc = eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"])
    out = eng.draft_lists(K, seq_subset, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"]),
                          dkc, dvc, eng.to_device_i32(act["kv_len"]), forced=eng.to_device_i32(forced),
                          want_logits=True, want_hidden=True)
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    lg, hd, dr = out["logits"].cpu().numpy(), out["hidden"].cpu().numpy(), out["draft"].cpu().numpy()
    kc = dkc.cpu().numpy().view(np.uint16)
    some_clear = False
    for b in range(B):
        r = refs[b]
        n = r["logits"].shape[-1]
        assert np.abs(lg[b, :, :n] - r["logits"][0]).max() <= LOGIT_TIGHT
        assert np.abs(hd[b] - r["hidden"][0]).max() <= 2e-3
        clear = r["margin"][0] > MARGIN
        some_clear |= bool(clear.any())
        np.testing.assert_array_equal(dr[b][clear], r["draft"][0][clear])
        L = int(act["kv_len"][b])
        assert appended_entries_close(kc[b][:, L:L + K], okc[b][:, L:L + K], recursive_from=1)
        assert np.array_equal(kc[b][:, :L], okc[b][:, :L])
    assert some_clear
    return eng


@pytest.mark.parametrize("ctx,seq_subset", [
    ([100, 0, 64], [0, 1, -1]),                                   # row-streaming phases, three lists
    ([10, 20, 150, 64], [1, 1, 0, 0]),
    ([0, 1, 63, 64, 150, 7, 99], [0, 0, 0, 1, 1, -1, -1]),        # batched phases
    (list(range(3, 123, 6)), [2] * 9 + [0] * 6 + [1] * 5),        # twenty sequences, two sequence tiles
    ([(7 * i) % 150 for i in range(270)], [1] * 100 + [-1] * 90 + [0] * 80),  # 270: tiled body phases, passes per list
])
def test_tiny_one_list_per_sequence(gpu, tiny, ctx, seq_subset):
    """Several id lists in one batch (several languages): every sequence against the oracle run with its own list
    - logits over its own rows, drafts mapped through its own list, caches - K = 3 with the oracle's drafts forced."""
    torch, binding = gpu["torch"], gpu["binding"]
    shape, K = tiny["shape"], 3
    rng = np.random.default_rng(11)
    lists = [tiny["ids"], np.sort(rng.choice(shape.vocab_size, 300, replace=False)).astype(np.int32),
             np.sort(rng.choice(shape.vocab_size, 37, replace=False)).astype(np.int32)]
    act = synth.make_activations(tiny["wl"], ctx=np.array(ctx, dtype=np.int32), capacity=192)
    B = len(ctx)
    eng = check_lists(gpu, shape, tiny["w"], lists, act, seq_subset, K)
    dkc, dvc = eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"])
    # one list for everybody through the same entry point equals the plain call bit for bit
    same = eng.draft_lists(K, [0] * B, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"]),
                           eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"]),
                           eng.to_device_i32(act["kv_len"]), want_logits=True)
    plain = eng.draft(K, 0, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"]),
                      eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"]),
                      eng.to_device_i32(act["kv_len"]), want_logits=True)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(same["draft"].cpu().numpy(), plain["draft"].cpu().numpy())
    np.testing.assert_array_equal(same["logits"].cpu().numpy(), plain["logits"].cpu().numpy())
    # lists that are not adjacent are refused before anything is enqueued
    if B >= 3:
        bad = [0, 1, 0] + [0] * (B - 3)
        st = binding.mtp_draft_steps_lists(eng.handle, B, K, bad, dkc, dkc, dkc, dvc, dkc, None, dkc)
        assert st == -6
    eng.close()


@pytest.mark.parametrize("d,groups", LIST_GROUPS)
def test_lists_of_a_larger_batch_read_row_major_activations(gpu, d, groups):
    """Few sequences per list in a batch of many, lists that the tiles do not serve as fast: few_rows.h on activations that the tiles
    of the other phases left row by row, up to eight rows with the lo halves in the second half of the operand, from an offset of
    rows on (test_rows_plan.py holds the route)."""
    shape = synth.HeadShape(d, 4, 2, 128, 1032, max(n for _, n in groups))
    B = sum(r for r, _ in groups)
    wl = synth.Workload(f"lists_{d}", 120, shape, B, 0, 0, (64,), 2, 0.5, zipf_subset=False)
    rng = np.random.default_rng(12)
    lists = [np.sort(rng.choice(shape.vocab_size, n, replace=False)).astype(np.int32) for _, n in groups]
    seq_subset = [-1 if n == shape.vocab_size else g for g, (r, n) in enumerate(groups) for _ in range(r)]
    act = synth.make_activations(wl, ctx=rng.integers(0, 60, B).astype(np.int32), capacity=64)
    check_lists(gpu, shape, synth.make_weights(wl), lists, act, seq_subset, 2).close()


# ------------------------------------------------------------------------------------------ teacher-forced loss
@pytest.mark.parametrize("n_pos,K", [(3, 2), (40, 3), (70, 3), (300, 2)])
def test_tiny_teacher_forced_loss(gpu, tiny, n_pos, K):
    """Eq. (1)-(2): the K per-step cross-entropies and their weighted sum against the oracle (3 positions: one
    sequence tile; 40: three; 70: two weight passes, and the output head as a tiled matrix product; 300: every
    matrix phase tiled except the down projection, whose reduction length 688 is not a multiple of the
    tiling's step).  The logits agree to ~1e-4, a mean of log-probabilities to better than 1e-3."""
    torch, Oracle, binding, orc_mod = gpu["torch"], gpu["Oracle"], gpu["binding"], gpu["orc"]
    shape = tiny["shape"]
    rng = np.random.default_rng(300 + n_pos)
    std = float(synth.bf16_bits_to_f32(tiny["act"]["hidden_in"]).std())
    hid = synth.f32_to_bf16_bits((rng.standard_normal((n_pos, shape.d_model)) * std).astype(np.float32))
    tok = rng.integers(0, shape.vocab_size, size=n_pos + K + 1).astype(np.int32)
    cap = max(128, (n_pos + 63) // 64 * 64)
    want = orc_mod.train_loss(Oracle(shape, tiny["w"], cap, "f32"), hid, tok, K, 0.6)
    eng = binding.DraftEngine(shape, tiny["w"], [], n_pos, cap, 1)
    got, logits = eng.train_loss(eng.to_device_bits(hid), eng.to_device_i32(tok), K, 0.6, want_logits=True)
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    got = got.cpu().numpy()
    np.testing.assert_allclose(got[:K], want["ce"], atol=1e-3)
    assert abs(got[K] - want["loss"]) <= 1e-3
    # the last step's logits, every position and every vocabulary row
    assert np.abs(logits.cpu().numpy() - want["logits"][K - 1]).max() <= LOGIT_TIGHT
    assert abs(got[K] - float((want["alpha"] * got[:K]).sum())) <= 1e-5       # Eq. (2) on its own numbers
    # twice in a row gives the same bits (fixed summation order), and a label out of range is reported
    again = eng.train_loss(eng.to_device_bits(hid), eng.to_device_i32(tok), K, 0.6).cpu().numpy()
    np.testing.assert_array_equal(again, got)
    bad = tok.copy()
    bad[-1] = shape.vocab_size
    eng.train_loss(eng.to_device_bits(hid), eng.to_device_i32(bad), K, 0.6)
    torch.cuda.synchronize()
    assert eng.poll_error() == -10
    eng.close()


# ------------------------------------------------------------------------------------------ accept / rollback
# ------------------------------------------------------------------------------------------ randomized cases
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_tiny_randomized_cases(gpu, tiny, seed):
    """Fifty seeded random cases per seed on the tiny head, each against the oracle: draft chains (1 to 257 sequences,
    K = 1..5, capacities from 192 to 32768, random contexts including empty ones), blocks of new positions (up to 40
    positions per sequence, ragged counts) and the teacher-forced loss (1 to 300 positions, K = 1..3).  The draws
    walk through every dispatch boundary of the host side: row-streaming / batched / tiled phases, one to four
    sequence tiles, one to five weight passes, vector / matrix-core / shared-read attention, static and handed-out
    attention items."""
    torch, Oracle, binding, orc_mod = gpu["torch"], gpu["Oracle"], gpu["binding"], gpu["orc"]
    wl, shape = tiny["wl"], tiny["shape"]
    rng = np.random.default_rng(seed)
    for case in range(50):
        kind = int(rng.integers(0, 3))
        cap = int(rng.choice([192, 512, 4096, 32768]))
        K = int(rng.integers(1, 6))
        if kind == 0:
            B = int(rng.choice([1, 2, 3, 4, 5, 9, 16, 17, 33, 64, 65, 100, 257]))
            if cap >= 4096:
                B = min(B, 40)
            ctx = rng.integers(0, cap - K, size=B).astype(np.int32)
            if rng.random() < 0.3:
                ctx[rng.integers(0, B)] = 0
            print(f"seed {seed} case {case}: chain B={B} capacity={cap} K={K}", flush=True)
            act = synth.make_activations(wl, ctx=ctx, capacity=cap)
            ref, res, caches = run_both(gpu, shape, tiny["w"], tiny["w"], act, [tiny["ids"]], 0, K)
            check_chain(ref, res, caches, act["kv_len"], K, need_clear=False)
        elif kind == 1:
            B = int(rng.choice([1, 2, 3, 5, 8, 16, 30]))
            m = int(rng.choice([1, 2, 3, 4, 5, 9, 17, 40]))
            if cap >= 4096:
                B = min(B, 8)
            while B * m > 320:
                m = max(1, m // 2)
            ctx = rng.integers(0, max(1, cap - m), size=B).astype(np.int32)
            ext = rng.integers(0, m + 1, size=B).astype(np.int32)
            ext[rng.integers(0, B)] = m
            print(f"seed {seed} case {case}: block B={B} positions={m} capacity={cap}", flush=True)
            act = synth.make_activations(wl, ctx=ctx, capacity=cap)
            hid, tok = extend_inputs(shape, act, m, 1000 * seed + case)
            ref, res, caches = run_extend(gpu, shape, tiny["w"], tiny["w"], act, [tiny["ids"]], 0, hid, tok, ext)
            assert res["err"] == 0
            check_extend(ref, res, caches, act, ext)
        else:
            n_pos = int(rng.choice([1, 2, 5, 33, 64, 65, 129, 256, 300]))
            Kt = int(rng.integers(1, 4))
            print(f"seed {seed} case {case}: loss positions={n_pos} K={Kt}", flush=True)
            hid = synth.f32_to_bf16_bits(rng.standard_normal((n_pos, shape.d_model)).astype(np.float32))
            tok = rng.integers(0, shape.vocab_size, size=n_pos + Kt + 1).astype(np.int32)
            capt = max(128, (n_pos + 63) // 64 * 64)
            want = orc_mod.train_loss(Oracle(shape, tiny["w"], capt, "f32"), hid, tok, Kt, 0.6)
            eng = binding.DraftEngine(shape, tiny["w"], [], n_pos, capt, 1)
            got, logits = eng.train_loss(eng.to_device_bits(hid), eng.to_device_i32(tok), Kt, 0.6, want_logits=True)
            torch.cuda.synchronize()
            assert eng.poll_error() == 0
            np.testing.assert_allclose(got.cpu().numpy()[:Kt], want["ce"], atol=1e-3)
            assert np.abs(logits.cpu().numpy() - want["logits"][Kt - 1]).max() <= LOGIT_TIGHT
            eng.close()


@pytest.mark.parametrize("K", [1, 3, 5])
@pytest.mark.parametrize("mode", [0, 1])
def test_accept_bit_exact(gpu, tiny, K, mode):
    torch, binding, orc = gpu["torch"], gpu["binding"], gpu["orc"]
    pats = list(itertools.product([0, 1], repeat=K))
    B = len(pats)
    rng = np.random.default_rng(K * 7 + mode)
    draft = rng.integers(0, 4096, size=(B, K)).astype(np.int32)
    target = rng.integers(0, 4096, size=(B, K + 1)).astype(np.int32)
    for bi, pt in enumerate(pats):
        for j in range(K):
            target[bi, j] = draft[bi, j] if pt[j] else (draft[bi, j] + 1 + j) % 4096
    L = rng.integers(0, 100, size=B).astype(np.int32)
    want = orc.accept(draft, target, L, mode)
    eng = binding.DraftEngine(tiny["shape"], tiny["w"], [], B, 192, K)
    kv = eng.to_device_i32(L)
    got = eng.accept(eng.to_device_i32(draft), eng.to_device_i32(target), kv, mode)
    torch.cuda.synchronize()
    for k in ("accept_len", "out_tokens", "pending", "kv_len"):
        np.testing.assert_array_equal(got[k].cpu().numpy(), want[k])
    eng.close()


def test_draft_then_accept_rollback(gpu, tiny):
    """Whole cycle on a ragged batch: draft, accept against a synthetic target chain, and check that the cache
    below the new kv_len still equals what drafting left there."""
    torch, binding, orc = gpu["torch"], gpu["binding"], gpu["orc"]
    wl = tiny["wl"]
    ctx = np.array([10, 64, 100, 129, 31, 5, 77, 150], dtype=np.int32)
    act = synth.make_activations(wl, ctx=ctx, capacity=192)
    K = 3
    eng = binding.DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], len(ctx), 192, K)
    kc, vc = eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"])
    kv = eng.to_device_i32(act["kv_len"])
    o = eng.draft(K, 0, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"]), kc, vc, kv)
    torch.cuda.synchronize()
    drafts = o["draft"].cpu().numpy()
    before = kc.cpu().numpy().copy()
    tgt = synth.make_targets(wl, drafts, accept_prob=0.7)
    want = orc.accept(drafts, tgt, act["kv_len"], 0)
    got = eng.accept(o["draft"], eng.to_device_i32(tgt), kv, 0)
    torch.cuda.synchronize()
    for k in ("accept_len", "out_tokens", "pending", "kv_len"):
        np.testing.assert_array_equal(got[k].cpu().numpy(), want[k])
    assert len(set(want["accept_len"].tolist())) > 1
    np.testing.assert_array_equal(kc.cpu().numpy(), before)  # rollback moves no bytes
    assert (want["kv_len"] - act["kv_len"] == np.minimum(want["accept_len"] + 1, K)).all()
    eng.close()


# ------------------------------------------------------------------------------------------ 7B-shaped head
@pytest.fixture(scope="module")
def big(gpu):
    """7B-shaped weights (shared by configs 2-5), on the host for the oracle and on the device for the library."""
    torch = gpu["torch"]
    wl = synth.WORKLOADS["c2_7b_b1"]
    w = synth.make_weights(wl, threads=16)
    dev = {k: torch.from_numpy(v.view(np.int16)).to("cuda:0") for k, v in w.items()}
    return {"w": w, "dev": dev, "shape": wl.shape}


def test_7b_batch1_ctx2048(gpu, big):
    wl = synth.WORKLOADS["c2_7b_b1"]
    act = synth.make_activations(wl)
    subsets = synth.make_subsets(wl)
    binding = gpu["binding"]
    eng = binding.DraftEngine(big["shape"], big["dev"], subsets, 1, act["kv_capacity"], wl.draft_steps)
    assert binding.mtp_set_launch_mode(eng.handle, binding.LAUNCH_PER_PHASE) == 0   # one launch per phase
    ref, res, caches = run_both(gpu, big["shape"], big["w"], big["dev"], act, subsets, 0, wl.draft_steps, engine=eng)
    gap = check_chain(ref, res, caches, act["kv_len"], wl.draft_steps)
    print("c2 max |dlogit| =", gap)
    ref, res, caches = run_both(gpu, big["shape"], big["w"], big["dev"], act, subsets, 0, wl.draft_steps, forced=None,
                                engine=eng)
    check_chain(ref, res, caches, act["kv_len"], wl.draft_steps, aligned=False)
    # the library's default (automatic: the single launch for this shape), free-running
    assert binding.mtp_set_launch_mode(eng.handle, binding.LAUNCH_AUTO) == 0
    ref, res, caches = run_both(gpu, big["shape"], big["w"], big["dev"], act, subsets, 0, wl.draft_steps, forced=None,
                                engine=eng)
    check_chain(ref, res, caches, act["kv_len"], wl.draft_steps, aligned=False)
    # the same through the single-launch path, asked for explicitly
    assert binding.mtp_set_launch_mode(eng.handle, binding.LAUNCH_SINGLE) == 0
    ref, res, caches = run_both(gpu, big["shape"], big["w"], big["dev"], act, subsets, 0, wl.draft_steps, engine=eng)
    check_chain(ref, res, caches, act["kv_len"], wl.draft_steps)
    eng.close()


def test_7b_extend_four_positions(gpu, big):
    """Config 2's head and context with a block of four new positions (an accepted run of three plus the bonus
    token), one sequence, and config 3's ragged batch of sixteen with up to four positions each (64 rows)."""
    for name, seed in (("c2_7b_b1", 230), ("c3_7b_b16", 231)):
        wl = synth.WORKLOADS[name]
        act = synth.make_activations(wl)
        subsets = synth.make_subsets(wl)
        B = wl.batch
        ext_len = np.array([max(0, 4 - (b % 4 == 3) * 3 - (b % 5 == 2) * 2) for b in range(B)], dtype=np.int32)
        hid, tok = extend_inputs(big["shape"], act, 4, seed)
        seqs = None if B == 1 else [0, 3, 7]   # the oracle on three of the sixteen sequences
        ref, res, caches = run_extend(gpu, big["shape"], big["w"], big["dev"], act, subsets, 0, hid, tok, ext_len,
                                      seqs=seqs)
        assert res["err"] == 0
        gap = check_extend(ref, res, caches, act, ext_len, sel=seqs)
        print(name, "extend max |dlogit| =", gap)


@pytest.mark.parametrize("n_pos,K", [(24, 2), (80, 2), (260, 1)])
def test_7b_teacher_forced_loss(gpu, big, n_pos, K):
    """The 7B-shaped head, full 151680-id vocabulary: the cross-entropies and the loss.  Every phase is a tiled matrix
    product over all positions (tiles of 32 to 128 rows at 24 and 80 positions, split reductions in the body), the
    head's without candidates, with a ragged block of positions and a ragged last block of vocabulary rows."""
    torch, Oracle, binding, orc_mod = gpu["torch"], gpu["Oracle"], gpu["binding"], gpu["orc"]
    shape = big["shape"]
    rng = np.random.default_rng(330)
    hid = synth.f32_to_bf16_bits(rng.standard_normal((n_pos, shape.d_model)).astype(np.float32))
    tok = rng.integers(0, shape.vocab_size, size=n_pos + K + 1).astype(np.int32)
    cap = (n_pos + 63) // 64 * 64
    want = orc_mod.train_loss(Oracle(shape, big["w"], cap, "f32"), hid, tok, K, 0.6)
    eng = binding.DraftEngine(shape, big["dev"], [], n_pos, cap, 1)
    got, logits = eng.train_loss(eng.to_device_bits(hid), eng.to_device_i32(tok), K, 0.6, want_logits=True)
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    got = got.cpu().numpy()
    print("7B teacher-forced CE", got[:K], "oracle", want["ce"], "loss", got[K], want["loss"])
    np.testing.assert_allclose(got[:K], want["ce"], atol=1e-3)
    assert abs(got[K] - want["loss"]) <= 1e-3
    gap = float(np.abs(logits.cpu().numpy() - want["logits"][K - 1]).max())
    print("last step's logits: largest gap", gap)
    # 3.6 to 12 million logits of the second step, each side recurring on its own float32 hidden state: the stated
    # bar; the largest gap seen is 3e-3
    assert gap <= LOGIT_TOL
    eng.close()


def test_7b_batch16_two_lists(gpu, big):
    """Config 3's ragged batch of sixteen with two id lists (nine sequences on the 32768-id list, seven on a 16384-id
    one built like config 4's): sampled sequences of both groups against the oracle."""
    torch, Oracle, binding = gpu["torch"], gpu["Oracle"], gpu["binding"]
    wl = synth.WORKLOADS["c3_7b_b16"]
    act = synth.make_activations(wl)
    lists = [synth.make_subsets(wl)[0], synth.make_subsets(synth.WORKLOADS["c4_7b_vocab"])[0]]
    B, K = wl.batch, wl.draft_steps
    seq_subset = [0] * 9 + [1] * 7
    eng = binding.DraftEngine(big["shape"], big["dev"], lists, B, act["kv_capacity"], K)
    dkc, dvc = eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"])
    out = eng.draft_lists(K, seq_subset, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"]),
                          dkc, dvc, eng.to_device_i32(act["kv_len"]), want_logits=True)
    torch.cuda.synchronize()
    assert eng.poll_error() == 0
    lg, dr = out["logits"].cpu().numpy(), out["draft"].cpu().numpy()
    orc = Oracle(big["shape"], big["w"], act["kv_capacity"], "f32")
    for b in (0, 8, 9, 15):
        ids = lists[seq_subset[b]]
        r = orc.chain(1, act["hidden_in"][b:b + 1], act["token_in"][b:b + 1], act["k_cache"][b:b + 1].copy(),
                      act["v_cache"][b:b + 1].copy(), act["kv_len"][b:b + 1], ids)
        gap = float(np.abs(lg[b, 0, :len(ids)] - r["logits"][0, 0]).max())
        assert gap <= LOGIT_TIGHT, (b, gap)
        if r["margin"][0, 0] > MARGIN:
            assert dr[b, 0] == r["draft"][0, 0]
    eng.close()


@pytest.mark.parametrize("launch_mode", [0, 1])
def test_7b_extend_then_continue(gpu, big, launch_mode):
    """Config 2: four new positions, then two recursive steps from the head's own hidden state, with a launch per
    phase and through the single-launch kernel for one sequence."""
    wl = synth.WORKLOADS["c2_7b_b1"]
    act = synth.make_activations(wl)
    gap = check_extend_then_continue(gpu, big["shape"], big["w"], big["dev"], act, synth.make_subsets(wl),
                                     np.array([4], dtype=np.int32), 4, 2, 250 + launch_mode, launch_mode=launch_mode)
    print("c2 extend + continue max |dlogit| =", gap)


@pytest.mark.parametrize("launch_mode", [0, 1])
def test_7b_vocab_sweep_ctx8192(gpu, big, launch_mode):
    """Full 151680-row head against nested compressed heads; the compressed logits are rows of the full ones.
    Once with a launch per phase and once through the single-launch kernel (the mode the bench times here)."""
    wl = synth.WORKLOADS["c4_7b_vocab"]
    act = synth.make_activations(wl)
    subsets = synth.make_subsets(wl)
    binding = gpu["binding"]
    eng = binding.DraftEngine(big["shape"], big["dev"], subsets, 1, act["kv_capacity"], wl.draft_steps)
    assert binding.mtp_set_launch_mode(eng.handle, launch_mode) == 0
    K = wl.draft_steps
    ref_full, res_full, caches = run_both(gpu, big["shape"], big["w"], big["dev"], act, subsets, -1, K, engine=eng)
    check_chain(ref_full, res_full, caches, act["kv_len"], K)
    for si in range(len(subsets)):
        ref, res, caches = run_both(gpu, big["shape"], big["w"], big["dev"], act, subsets, si, K, engine=eng)
        check_chain(ref, res, caches, act["kv_len"], K)
        # step 1 sees the same inputs whatever the head: compressed logits are a row gather of the full logits
        np.testing.assert_array_equal(res["logits"][0, 0], res_full["logits"][0, 0][subsets[si]])
    assert set(subsets[0]).issubset(set(subsets[1])) and set(subsets[1]).issubset(set(subsets[2]))
    eng.close()


def test_7b_batch16_ragged_with_accept(gpu, big):
    torch, binding, orc = gpu["torch"], gpu["binding"], gpu["orc"]
    wl = synth.WORKLOADS["c3_7b_b16"]
    act = synth.make_activations(wl, threads=16)
    subsets = synth.make_subsets(wl)
    K = wl.draft_steps
    eng = binding.DraftEngine(big["shape"], big["dev"], subsets, wl.batch, act["kv_capacity"], K)
    ref, res, caches = run_both(gpu, big["shape"], big["w"], big["dev"], act, subsets, 0, K, engine=eng)  # all 16
    check_chain(ref, res, caches, act["kv_len"], K)
    # accept + rollback on the whole batch, per-position acceptance 0.8
    kv = eng.to_device_i32(act["kv_len"])
    o = eng.draft(K, 0, eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"]),
                  eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"]), kv)
    torch.cuda.synchronize()
    drafts = o["draft"].cpu().numpy()
    tgt = synth.make_targets(wl, drafts)
    want = orc.accept(drafts, tgt, act["kv_len"], 0)
    got = eng.accept(o["draft"], eng.to_device_i32(tgt), kv, 0)
    torch.cuda.synchronize()
    for k in ("accept_len", "out_tokens", "pending", "kv_len"):
        np.testing.assert_array_equal(got[k].cpu().numpy(), want[k])
    eng.close()


def test_7b_batch64_long_context_sampled(gpu, big):
    """Throughput regime (B = 64, contexts in [8192, 32768], K = 5): the library runs the whole batch, the oracle
    sixteen of its sequences: the shortest, the longest, the four whose contexts end closest below and the four closest
    above a multiple of the 4096-token attention split, and six more spread over the lengths."""
    wl = synth.WORKLOADS["c5_7b_b64"]
    act = synth.make_activations(wl, threads=16)
    subsets = synth.make_subsets(wl)
    K = wl.draft_steps
    L = act["kv_len"]
    by_len = np.argsort(L)
    edge = np.argsort(L % 4096)
    pick = {int(by_len[0]), int(by_len[-1])} | {int(b) for b in edge[:4]} | {int(b) for b in edge[-4:]}
    for b in by_len[3::9]:
        if len(pick) < 16:
            pick.add(int(b))
    for b in by_len:
        if len(pick) < 16:
            pick.add(int(b))
    seqs = sorted(pick)
    assert len(seqs) == 16
    ref, res, caches = run_both(gpu, big["shape"], big["w"], big["dev"], act, subsets, 0, K, seqs=seqs,
                                max_batch=wl.batch)
    check_chain(ref, res, caches, L[seqs], K)


def test_7b_seven_draft_steps(gpu, big):
    """Config 2 with K = 7, the longest chain of the draft-length sweep (Sec. 3.5), through the single-launch kernel and
    with a launch per phase; the oracle's drafts forced, so that every step sees the same inputs on both sides."""
    wl = synth.WORKLOADS["c2_7b_b1"]
    act = synth.make_activations(wl, capacity=2112)
    subsets = synth.make_subsets(wl)
    binding = gpu["binding"]
    eng = binding.DraftEngine(big["shape"], big["dev"], subsets, 1, act["kv_capacity"], 7)
    for mode in (binding.LAUNCH_AUTO, binding.LAUNCH_PER_PHASE):
        assert binding.mtp_set_launch_mode(eng.handle, mode) == 0
        ref, res, caches = run_both(gpu, big["shape"], big["w"], big["dev"], act, subsets, 0, 7, engine=eng)
        gap = check_chain(ref, res, caches, act["kv_len"], 7)
        print("c2 K=7 mode", mode, "max |dlogit| =", gap)
    eng.close()


@pytest.mark.parametrize("B", [1, 3])
def test_tiny_seven_draft_steps(gpu, tiny, B):
    act = synth.make_activations(tiny["wl"], ctx=np.array([100, 0, 150][:B], dtype=np.int32), capacity=192)
    ref, res, caches = run_both(gpu, tiny["shape"], tiny["w"], tiny["w"], act, [tiny["ids"]], 0, 7)
    check_chain(ref, res, caches, act["kv_len"], 7)


NAN_BITS = np.uint16(0x7FC0)


def drafting_loop(gpu, wl, w_host, w_dev, act, subsets, K, cycles, seed, accept_prob=0.6):
    """The loop of Sec. 2.3 over several cycles, library against oracle.  One cycle: the first draft step over the new
    confirmed positions with the target model's hidden states (mtp_draft_extend: one position, or two where the cycle
    before accepted all K drafts and the entry of the last one is still missing), K - 1 recursive steps from the head's
    own output (mtp_draft_continue), acceptance with rollback mode 0 (mtp_accept).  Every cache slot at or beyond the
    live length holds NaN on both sides, at the start and again after every rollback: a read past the live length
    would poison the logits.  The library is fed the oracle's tokens, so both sides see the same inputs in every cycle;
    integer results (accept lengths, emitted tokens, pending flags, lengths) must agree bit for bit."""
    torch, Oracle, binding, orc_mod = gpu["torch"], gpu["Oracle"], gpu["binding"], gpu["orc"]
    shape = wl.shape
    B, cap, ids = len(act["kv_len"]), act["kv_capacity"], subsets[0]
    rng = np.random.default_rng(seed)
    std = float(synth.bf16_bits_to_f32(act["hidden_in"]).std())
    okc, ovc = act["k_cache"].copy(), act["v_cache"].copy()
    kv = act["kv_len"].astype(np.int32).copy()
    for b in range(B):
        okc[b][:, kv[b]:] = NAN_BITS
        ovc[b][:, kv[b]:] = NAN_BITS
    eng = binding.DraftEngine(shape, w_dev, subsets, 2 * B, cap, K)
    dkc, dvc = eng.to_device_bits(okc), eng.to_device_bits(ovc)
    dkv = eng.to_device_i32(kv)
    orc = Oracle(shape, w_host, cap, "f32")
    pending = np.zeros(B, dtype=np.int32)
    tok_next = act["token_in"].astype(np.int32).copy()   # the token the next cycle starts from
    tok_pending = np.zeros(B, dtype=np.int32)            # the accepted draft whose cache entry is missing
    worst = 0.0
    for c in range(cycles):
        ext_len = (1 + pending).astype(np.int32)
        hid = synth.f32_to_bf16_bits((rng.standard_normal((2, B, shape.d_model)) * std).astype(np.float32))
        tok = np.zeros((2, B), dtype=np.int32)
        for b in range(B):
            if pending[b]:
                tok[0, b], tok[1, b] = tok_pending[b], tok_next[b]
            else:
                tok[0, b] = tok_next[b]
        # ---- first step over the new positions -------------------------------------------------------------------
        ref = orc.extend(hid, tok, ext_len, okc, ovc, kv, ids)
        ex = eng.extend(0, eng.to_device_bits(hid), eng.to_device_i32(tok), eng.to_device_i32(ext_len), dkc, dvc, dkv,
                        want_logits=True, want_hidden=True)
        torch.cuda.synchronize()
        assert eng.poll_error() == 0
        np.testing.assert_array_equal(dkv.cpu().numpy(), ref["kv_len"])
        lg, hd = ex["logits"].cpu().numpy(), ex["hidden"].cpu().numpy()
        assert np.isfinite(lg[0]).all()
        drafts = np.zeros((B, K), dtype=np.int32)
        own = torch.empty((B, shape.d_model), dtype=torch.float32, device="cuda:0")
        cont = []
        for b in range(B):
            last = int(ext_len[b]) - 1
            gap = float(np.abs(lg[:last + 1, b] - ref["logits"][:last + 1, b]).max())
            worst = max(worst, gap)
            assert gap <= LOGIT_TIGHT, (c, b, gap)
            drafts[b, 0] = ref["draft"][last, b]
            own[b] = ex["hidden"][last, b]
            # ---- K - 1 recursive steps, the oracle's by single steps fed back by hand ------------------------------
            cont.append(orc.chain_from_own_hidden(K - 1, ref["hidden"][last, b], int(drafts[b, 0]), okc[b], ovc[b],
                                                  int(ref["kv_len"][b]), ids))
            drafts[b, 1:] = cont[b]["draft"]
        kv = ref["kv_len"].astype(np.int32).copy()
        forced = np.ascontiguousarray(drafts[:, 1:K - 1]) if K > 2 else None
        out = eng.draft_continue(K - 1, 0, own, eng.to_device_i32(drafts[:, 0].copy()), dkc, dvc, dkv,
                                 forced=eng.to_device_i32(forced) if forced is not None else None, want_logits=True)
        torch.cuda.synchronize()
        assert eng.poll_error() == 0
        lgc, drc = out["logits"].cpu().numpy(), out["draft"].cpu().numpy()
        for b in range(B):
            gap = float(np.abs(lgc[b] - cont[b]["logits"]).max())
            worst = max(worst, gap)
            assert gap <= LOGIT_TIGHT, (c, b, gap)
            clear = cont[b]["margin"] > MARGIN
            np.testing.assert_array_equal(drc[b][clear], cont[b]["draft"][clear])
        # ---- acceptance + rollback: the first of the K drafts came from the block's last position, whose slot the block
        # already counted, so the draft started one slot below the present length -----------------------------------
        tgt = synth.make_targets(wl, drafts, accept_prob=accept_prob, salt=c)
        want = orc_mod.accept(drafts, tgt, kv - 1, 0)
        dkv -= 1
        got = eng.accept(eng.to_device_i32(drafts), eng.to_device_i32(tgt), dkv, 0)
        torch.cuda.synchronize()
        for key in ("accept_len", "out_tokens", "pending", "kv_len"):
            np.testing.assert_array_equal(got[key].cpu().numpy(), want[key])
        np.testing.assert_array_equal(dkv.cpu().numpy(), want["kv_len"])
        kv, pending = want["kv_len"].astype(np.int32).copy(), want["pending"].astype(np.int32).copy()
        a = want["accept_len"]
        for b in range(B):
            tok_next[b] = tgt[b, a[b]]          # the target's own token after the accepted run
            tok_pending[b] = drafts[b, K - 1]
            # live entries agree (up to a bf16 step where the recursive steps wrote them), dead ones become NaN again
            hk, hv = dkc[b].cpu().numpy().view(np.uint16), dvc[b].cpu().numpy().view(np.uint16)
            assert appended_entries_close(hk[:, :kv[b]], okc[b][:, :kv[b]], recursive_from=0)
            assert appended_entries_close(hv[:, :kv[b]], ovc[b][:, :kv[b]], recursive_from=0)
            okc[b][:, kv[b]:] = NAN_BITS
            ovc[b][:, kv[b]:] = NAN_BITS
            # the library's own live entries stay as they are; only the dead slots are overwritten
            dkc[b][:, kv[b]:] = int(NAN_BITS.view(np.int16))
            dvc[b][:, kv[b]:] = int(NAN_BITS.view(np.int16))
            okc[b][:, :kv[b]] = hk[:, :kv[b]]   # both sides continue from the same live entries
            ovc[b][:, :kv[b]] = hv[:, :kv[b]]
    eng.close()
    return worst, pending


def test_tiny_drafting_loop_with_poisoned_dead_slots(gpu, tiny):
    act = synth.make_activations(tiny["wl"], ctx=np.array([40, 0, 120], dtype=np.int32), capacity=192)
    worst, _ = drafting_loop(gpu, tiny["wl"], tiny["w"], tiny["w"], act, [tiny["ids"]], 3, 5, 901)
    print("tiny loop: largest logit gap", worst)
    # acceptance probability 1: every cycle accepts all K drafts and leaves a pending entry for the next block to close
    worst, pending = drafting_loop(gpu, tiny["wl"], tiny["w"], tiny["w"], act, [tiny["ids"]], 3, 4, 902,
                                   accept_prob=1.0)
    assert pending.all()


def test_7b_drafting_loop_with_poisoned_dead_slots(gpu, big):
    """Config 2, four cycles: the recursive steps run through the single-launch kernel."""
    wl = synth.WORKLOADS["c2_7b_b1"]
    act = synth.make_activations(wl, capacity=2112)
    worst, _ = drafting_loop(gpu, wl, big["w"], big["dev"], act, synth.make_subsets(wl), 3, 4, 903,
                             accept_prob=0.8)
    print("c2 loop: largest logit gap", worst)


# ------------------------------------------------------------------------------ workspace guards, HIP-graph capture
def exercise_every_entry_point(gpu, eng, wl, act, K, tiny_ids=None):
    """One call of every draft entry point on `eng` (results are checked elsewhere)."""
    torch, binding = gpu["torch"], gpu["binding"]
    B = len(act["kv_len"])
    hid, tok = eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"])
    kc, vc = eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"])
    for mode in (0, 1, 2, 3):
        if mode == 3 and B > 4:
            continue
        assert binding.mtp_set_launch_mode(eng.handle, mode) == 0
        kv = eng.to_device_i32(act["kv_len"])
        o = eng.draft(K, 0, hid, tok, kc, vc, kv, want_logits=True, want_hidden=True)
        tgt = synth.make_targets(wl, o["draft"].cpu().numpy(), accept_prob=0.7)
        eng.accept(o["draft"], eng.to_device_i32(tgt), kv, 0)
    assert binding.mtp_set_launch_mode(eng.handle, 2) == 0
    kv = eng.to_device_i32(act["kv_len"])
    eng.draft_lists(K, [0] * B, hid, tok, kc, vc, kv)
    hid2, tok2 = extend_inputs(wl.shape, act, 2, seed=5)
    kv = eng.to_device_i32(act["kv_len"])
    ex = eng.extend(0, eng.to_device_bits(hid2), eng.to_device_i32(tok2), eng.to_device_i32(np.full(B, 2, np.int32)),
                    kc, vc, kv, want_hidden=True)
    own = ex["hidden"][1].contiguous()
    eng.draft_continue(K - 1, 0, own.clone(), ex["draft"][1].clone(), kc, vc, kv)
    torch.cuda.synchronize()
    assert eng.poll_error() == 0


@pytest.mark.parametrize("B", [1, 3, 20])
def test_tiny_nothing_is_written_outside_the_workspace(gpu, tiny, B):
    """The workspace sits between two guard areas of a fixed byte pattern; after every entry point has run in every
    launch mode both are unchanged."""
    binding = gpu["binding"]
    wl, K = tiny["wl"], 3
    ctx = (np.arange(B, dtype=np.int32) * 37) % 150 + 1
    act = synth.make_activations(wl, ctx=ctx, capacity=192)
    eng = binding.DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], 2 * B, 192, K, guard_bytes=1 << 16)
    assert eng.guards_intact()
    exercise_every_entry_point(gpu, eng, wl, act, K)
    assert eng.guards_intact()
    eng.close()


def test_7b_nothing_is_written_outside_the_workspace(gpu, big):
    binding = gpu["binding"]
    wl = synth.WORKLOADS["c2_7b_b1"]
    act = synth.make_activations(wl)
    eng = binding.DraftEngine(big["shape"], big["dev"], synth.make_subsets(wl), 2, act["kv_capacity"], wl.draft_steps,
                              guard_bytes=1 << 20)
    exercise_every_entry_point(gpu, eng, wl, act, wl.draft_steps)
    assert eng.guards_intact()
    eng.close()


def graph_replays_match_eager(gpu, wl, eng, act, K):
    """mtp_draft_steps + mtp_accept captured into a HIP graph on a stream of default priority and replayed four times,
    with eager work of the same engine and synchronisations between the replays: every replay must give what the eager
    calls (one launch per phase, the form a captured call takes) give on the same inputs: drafts, logits, the appended
    cache entries, accept results, bit for bit."""
    torch, binding = gpu["torch"], gpu["binding"]
    B = len(act["kv_len"])
    hid, tok = eng.to_device_bits(act["hidden_in"]), eng.to_device_i32(act["token_in"])
    kc0, vc0 = eng.to_device_bits(act["k_cache"]), eng.to_device_bits(act["v_cache"])
    kv0 = eng.to_device_i32(act["kv_len"])

    def fresh():
        return kc0.clone(), vc0.clone(), kv0.clone()

    # eager reference
    assert binding.mtp_set_launch_mode(eng.handle, binding.LAUNCH_PER_PHASE) == 0
    kc, vc, kv = fresh()
    o = eng.draft(K, 0, hid, tok, kc, vc, kv, want_logits=True)
    torch.cuda.synchronize()
    tgt = eng.to_device_i32(synth.make_targets(wl, o["draft"].cpu().numpy(), accept_prob=0.7))
    a = eng.accept(o["draft"], tgt, kv, 0)
    torch.cuda.synchronize()
    want = [o["draft"].cpu().numpy(), o["logits"].cpu().numpy(), kc.cpu().numpy(), vc.cpu().numpy(),
            kv.cpu().numpy()] + [a[k].cpu().numpy() for k in ("accept_len", "out_tokens", "pending")]
    assert binding.mtp_set_launch_mode(eng.handle, binding.LAUNCH_AUTO) == 0  # the default, as a caller would capture it

    # static buffers of the graph
    gkc, gvc, gkv = fresh()
    n = eng.subset_size(0)
    draft = torch.empty((B, K), dtype=torch.int32, device="cuda:0")
    logits = torch.empty((B, K, n), dtype=torch.float32, device="cuda:0")
    acc = torch.empty(B, dtype=torch.int32, device="cuda:0")
    out = torch.empty((B, K + 1), dtype=torch.int32, device="cuda:0")
    pend = torch.empty(B, dtype=torch.int32, device="cuda:0")
    torch.cuda.synchronize()
    side = torch.cuda.Stream()  # default priority
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        st = torch.cuda.current_stream().cuda_stream
        assert binding.mtp_draft_steps(eng.handle, B, K, 0, hid, tok, gkc, gvc, gkv, None, draft, logits, None, st) == 0
        assert binding.mtp_accept(eng.handle, B, K, draft, tgt, 0, gkv, acc, out, pend, st) == 0
    for replay in range(4):
        k2, v2, l2 = fresh()
        gkc.copy_(k2)
        gvc.copy_(v2)
        gkv.copy_(l2)
        draft.fill_(-7)
        logits.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = [draft.cpu().numpy(), logits.cpu().numpy(), gkc.cpu().numpy(), gvc.cpu().numpy(), gkv.cpu().numpy(),
               acc.cpu().numpy(), out.cpu().numpy(), pend.cpu().numpy()]
        for g, w_ in zip(got, want):
            np.testing.assert_array_equal(g, w_, err_msg=f"replay {replay}")
        # eager work of the same engine between the replays (other inputs, the engine's default launch mode)
        kc, vc, kv = fresh()
        eng.draft(K, 0, hid, torch.roll(tok, 1), kc, vc, kv)
        torch.cuda.synchronize()
    assert eng.poll_error() == 0


@pytest.mark.parametrize("B", [1, 5])
def test_tiny_calls_captured_into_a_hip_graph(gpu, tiny, B):
    binding = gpu["binding"]
    wl, K = tiny["wl"], 3
    ctx = (np.arange(B, dtype=np.int32) * 41) % 120 + 3
    act = synth.make_activations(wl, ctx=ctx, capacity=192)
    eng = binding.DraftEngine(tiny["shape"], tiny["w"], [tiny["ids"]], B, 192, K)
    graph_replays_match_eager(gpu, wl, eng, act, K)
    eng.close()


def test_7b_call_captured_into_a_hip_graph(gpu, big):
    """One sequence at the 7B shape: eager calls take the single-launch kernel, whose tags count calls on the host; a
    captured call must not (its replays would all carry the captured call's tags)."""
    binding = gpu["binding"]
    wl = synth.WORKLOADS["c2_7b_b1"]
    act = synth.make_activations(wl)
    eng = binding.DraftEngine(big["shape"], big["dev"], synth.make_subsets(wl), 1, act["kv_capacity"], wl.draft_steps)
    graph_replays_match_eager(gpu, wl, eng, act, wl.draft_steps)
    eng.close()
