"""GPU parity of lsrm_nsa_backward against the CPU oracle's analytic gradients, element by
element on small cases and on a sample of blocks and heads at the full size of config 5.
Tolerance as for the forward: max-abs <= 2e-2 and relative L2 <= 5e-3 per gradient tensor."""
import dataclasses
import sys

import numpy as np
import pytest

from paper_2604_05182_amd import inputs as I

import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2604_05182_amd import binding
    return binding


def _log(msg):
    print(msg, file=sys.stderr, flush=True)


def _case(B, oracle_lib, cfg, idx=None, seg="default", scale=0.0, window=None, window_mode=0):
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    if idx is None:
        idx, _ = oracle_lib.route(I.make_points(cfg), I.make_cameras(cfg), cfg.grid, cfg.topk)
    seg_arr = cfg.seg_offsets() if isinstance(seg, str) else np.asarray(seg, dtype=np.int32)
    window = cfg.window if window is None else window
    got = G.run_backward(B, cfg, q_bits, k_bits, v_bits, idx, gates, dout_bits, seg_offsets=seg, scale=scale,
                         window=window, window_mode=window_mode)
    q, k, v, dout = (I.bf16_bits_to_f32(a) for a in (q_bits, k_bits, v_bits, dout_bits))
    kc, vc = oracle_lib.pool(k), oracle_lib.pool(v)
    return got, (q, k, v, kc, vc, idx, gates, seg_arr, window, dout)


def _assert_grads(got, ref, tag):
    for name, g, r in zip(("dq", "dk", "dv"), got, ref):
        assert np.isfinite(g).all(), f"{tag} {name}: non-finite values"
        ma, rl = G.attention_errors(g, r)
        _log(f"[backward] {tag} {name}: max-abs {ma:.3e} rel-L2 {rl:.3e}  (|ref| max {np.abs(r).max():.3e})")
        assert ma <= G.MAX_ABS_TOL and rl <= G.REL_L2_TOL, (tag, name, ma, rl)


def test_backward_grouped_heads_large_gradients_elementwise(B, oracle_lib):
    """Sixteen query heads per key/value head with single-token blocks and dout as generated (not divided by the
    group size): dk and dv reach magnitudes where their bf16 storage alone exceeds the absolute bar, so they are
    checked element by element against a bar that grows with the row: 2e-2 for rows of order one plus 2^-7 of the
    largest reference value of the element's (token, head) row -- every channel of a row sums the same contributions
    with the same probabilities, so a channel's error follows the row's magnitude, not its own value (a bf16 result
    is within 2^-9 of its value; the operands' own bf16 roundings and the order of the fp32 sums take the rest) --
    and by relative L2 as everywhere."""
    cfg = I.small_config(name="b-group16-unscaled", n_obj=576, n_views=2, grid=16, heads=32, d=32, topk=4, window=160,
                         seed=71, h_kv=2, gate_channels=False)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    rng = np.random.default_rng(13)
    cnt = rng.integers(1, 65, size=cfg.nb).astype(np.int32)
    cnt[:6] = (64, 1, 33, 32, 31, 64)
    idx = np.stack([rng.choice(cfg.nb, size=cfg.topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[:, 0] = np.minimum(np.arange(cfg.nb), 5)
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    q, k, v, dout = (I.bf16_bits_to_f32(a) for a in (q_bits, k_bits, v_bits, dout_bits))
    got = G.run_backward(B, cfg, q_bits, k_bits, v_bits, idx, gates, dout_bits, window_mode=1, block_count=cnt)
    kc, vc = oracle_lib.pool(k, cnt), oracle_lib.pool(v, cnt)
    ref = oracle_lib.nsa_backward(q, k, v, kc, vc, idx, gates, cfg.seg_offsets(), cfg.window, dout, window_mode=1,
                                  block_count=cnt)
    active = (np.arange(cfg.n) % 64) < np.repeat(cnt, 64)
    for name, g, r in zip(("dq", "dk", "dv"), got, ref):
        g, r = g[active], r[active]
        assert np.isfinite(g).all(), name
        excess = np.abs(g - r) - (G.MAX_ABS_TOL + np.abs(r).max(axis=-1, keepdims=True) * 2.0 ** -7)
        _, rl = G.attention_errors(g, r)
        _log(f"[backward] {cfg.name} {name}: |ref| max {np.abs(r).max():.3e}, worst excess over the bar "
             f"{excess.max():.3e}, rel-L2 {rl:.3e}")
        assert excess.max() <= 0.0 and rl <= G.REL_L2_TOL, (name, float(excess.max()), rl)


def test_backward_small(B, oracle_lib):
    cfg = I.small_config(name="b-small", n_obj=512, n_views=2, grid=16, heads=2, d=64, topk=3, window=128)
    _log(f"[backward] {cfg.name}")
    got, args = _case(B, oracle_lib, cfg)
    _assert_grads(got, oracle_lib.nsa_backward(*args), cfg.name)


def test_backward_ragged_and_holes(B, oracle_lib):
    """NB not a multiple of 32, odd head count, -1 holes, an empty routed row, key blocks nobody routes
    to, a window that is not a multiple of the block, explicit scale."""
    cfg = I.small_config(name="b-ragged", n_obj=1088, n_views=3, grid=24, heads=3, d=64, topk=5, window=200, seed=21)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    rng = np.random.default_rng(5)
    idx = np.stack([rng.choice(cfg.nb // 2, size=cfg.topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[rng.random(idx.shape) < 0.2] = -1
    idx[2] = -1
    got, args = _case(B, oracle_lib, cfg, idx=idx, scale=0.2)
    _assert_grads(got, oracle_lib.nsa_backward(*args, scale=0.2), cfg.name)


@pytest.mark.parametrize("d", [64, 128, 32])
def test_backward_repeated_and_popular_blocks(B, oracle_lib, d):
    """Rows that list a block twice (it is attended twice) and one block that every row lists (a reverse list
    longer than one 64-entry chunk, and by far the longest walk), with per-channel gates on grouped heads
    (the gradient rows change between branches even where a branch is empty)."""
    cfg = I.small_config(name=f"b-repeat-d{d}", n_obj=4096, n_views=2, grid=16, heads=4, d=d, topk=4, window=128,
                         seed=27, h_kv=2, gate_channels=True)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    rng = np.random.default_rng(11)
    idx = np.stack([rng.choice(cfg.nb, size=cfg.topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[:, 0] = 5                      # a popular block: nb entries in its reverse list
    idx[3::7, 2] = idx[3::7, 1]        # repeats inside a row
    idx[4::9, 3] = 5                   # the popular block twice in a row
    idx[6] = -1
    got, args = _case(B, oracle_lib, cfg, idx=idx)
    _assert_grads(got, oracle_lib.nsa_backward(*args), cfg.name)
    # no routed blocks and no window at all: only the compressed branch is left
    cfg0 = I.small_config(name="b-cmp-only", n_obj=512, n_views=2, grid=16, heads=4, d=64, topk=2, window=0, seed=28,
                          h_kv=2, gate_channels=True)
    idx0 = np.full((cfg0.nb, cfg0.topk), -1, dtype=np.int32)
    got, args = _case(B, oracle_lib, cfg0, idx=idx0)
    _assert_grads(got, oracle_lib.nsa_backward(*args), cfg0.name)


@pytest.mark.parametrize("d,topk", [(64, 128), (128, 80), (32, 100)])
def test_backward_wide_routing_rows(B, oracle_lib, d, topk):
    """Routing rows of 65..128 entries (the paper's stage-3 budgets at 16 views need 80), with holes on either
    side of entry 64 and a row whose valid entries all sit past it."""
    cfg = I.small_config(name=f"b-topk{topk}-d{d}", n_obj=8192, n_views=2, grid=16, heads=2, d=d, topk=topk, window=64,
                         seed=63)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    rng = np.random.default_rng(14)
    idx = np.stack([rng.choice(cfg.nb, size=topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[1::3][rng.random(idx[1::3].shape) < 0.3] = -1
    idx[5, :70] = -1
    got, args = _case(B, oracle_lib, cfg, idx=idx)
    # every block and head through the sampled function (the same arithmetic, spread over the host's threads)
    every = np.arange(cfg.nb, dtype=np.int32)
    _assert_grads(got, oracle_lib.nsa_backward_sampled(*args, every, every, list(range(cfg.heads))), cfg.name)


def test_backward_own_block_window(B, oracle_lib):
    """The window branch over the query's own block (App. A) instead of the sliding window."""
    cfg = I.small_config(name="b-ownblock", n_obj=1088, n_views=3, grid=24, heads=3, d=64, topk=5, window=200, seed=23)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    rng = np.random.default_rng(9)
    idx = np.stack([rng.choice(cfg.nb, size=cfg.topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[rng.random(idx.shape) < 0.2] = -1
    got, args = _case(B, oracle_lib, cfg, idx=idx, window_mode=1)
    _assert_grads(got, oracle_lib.nsa_backward(*args, window_mode=1), cfg.name)


@pytest.mark.parametrize("d,heads,h_kv,gate_channels", [(64, 6, 2, False), (64, 2, 2, True), (64, 4, 1, True),
                                                        (32, 2, 2, False), (128, 2, 2, False), (128, 4, 2, True),
                                                        # the paper's heads in small: 16 query heads per key/value head
                                                        (32, 32, 2, True),
                                                        # 9 query heads per key/value head: head ranges of 2, 2, 2, 2, 1
                                                        (32, 18, 2, False)])
def test_backward_head_shapes_and_gates(B, oracle_lib, d, heads, h_kv, gate_channels):
    """Head dimensions 32 / 64 / 128, query heads sharing key/value heads (a key/value head collects the
    gradients of its whole group), one gate per output channel; ragged block count, holes in the table."""
    cfg = I.small_config(name=f"b-d{d}-h{heads}-kv{h_kv}-ch{int(gate_channels)}", n_obj=576, n_views=2, grid=16,
                         heads=heads, d=d, topk=4, window=160, seed=51, h_kv=h_kv, gate_channels=gate_channels)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    rng = np.random.default_rng(11)
    idx = np.stack([rng.choice(cfg.nb, size=cfg.topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[rng.random(idx.shape) < 0.2] = -1
    got, args = _case(B, oracle_lib, cfg, idx=idx)
    assert got[1].shape == (cfg.n, h_kv, d)
    _assert_grads(got, oracle_lib.nsa_backward(*args), cfg.name)


@pytest.mark.parametrize("d,window_mode,heads,h_kv,gate_channels",
                         [(64, 0, 3, 3, False), (64, 1, 3, 3, False), (128, 1, 3, 3, False), (32, 0, 3, 3, False),
                          # grouped heads: the pass that adds the head ranges finishes the rows
                          (64, 0, 4, 2, False), (32, 1, 16, 2, False),
                          # per-channel gates: the gate * dout rows of padding slots (NaN dout) must never be read
                          (64, 0, 3, 3, True), (128, 1, 2, 2, True), (32, 0, 4, 2, True)])
def test_backward_with_active_counts(B, oracle_lib, d, window_mode, heads, h_kv, gate_channels):
    """Blocks with fewer than 64 active tokens: padding slots are neither queries nor keys (whatever sits in
    their rows of k, v and dout -- NaN here -- is never looked at) and get zero gradients."""
    cfg = I.small_config(name=f"b-counts-d{d}-w{window_mode}-h{heads}-kv{h_kv}-ch{int(gate_channels)}", n_obj=576,
                         n_views=2, grid=16, heads=heads, d=d, topk=4, window=160, seed=71, h_kv=h_kv,
                         gate_channels=gate_channels)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    rng = np.random.default_rng(13)
    cnt = rng.integers(1, 65, size=cfg.nb).astype(np.int32)
    cnt[:6] = (64, 1, 33, 32, 31, 64)
    idx = np.stack([rng.choice(cfg.nb, size=cfg.topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[rng.random(idx.shape) < 0.2] = -1
    idx[:, 0] = np.minimum(np.arange(cfg.nb), 5)
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    if heads != h_kv:
        # a key/value head sums the gradients of its group: dout / group (a power of two, exact in bf16) keeps
        # dk, dv at the magnitude the absolute tolerance was set for
        dout_bits = I.f32_to_bf16_bits(I.bf16_bits_to_f32(dout_bits) * np.float32(h_kv / heads))
    q, k, v, dout = (I.bf16_bits_to_f32(a) for a in (q_bits, k_bits, v_bits, dout_bits))
    inactive = (np.arange(cfg.n) % 64) >= np.repeat(cnt, 64)
    k_bits, v_bits, dout_bits = k_bits.copy(), v_bits.copy(), dout_bits.copy()
    for bits in (k_bits, v_bits, dout_bits):
        bits[inactive] = 0x7FC0
    got = G.run_backward(B, cfg, q_bits, k_bits, v_bits, idx, gates, dout_bits, window_mode=window_mode, block_count=cnt)
    kc, vc = oracle_lib.pool(k, cnt), oracle_lib.pool(v, cnt)
    ref = oracle_lib.nsa_backward(q, k, v, kc, vc, idx, gates, cfg.seg_offsets(), cfg.window, dout,
                                  window_mode=window_mode, block_count=cnt)
    _assert_grads(got, ref, cfg.name)
    for g in got:
        assert np.all(g[inactive] == 0)


def test_backward_zero_window_and_topk_one(B, oracle_lib):
    cfg = I.small_config(name="b-w0", n_obj=256, n_views=1, grid=16, heads=1, d=64, topk=1, window=0)
    got, args = _case(B, oracle_lib, cfg)
    _assert_grads(got, oracle_lib.nsa_backward(*args), cfg.name)


def test_backward_single_segment_wide_window(B, oracle_lib):
    """One segment, window wider than the sequence, every block routed by every block."""
    cfg = I.small_config(name="b-dense", n_obj=512, n_views=0, grid=0, heads=2, d=64, topk=8, window=1024)
    idx = np.tile(np.arange(8, dtype=np.int32), (8, 1))
    got, args = _case(B, oracle_lib, cfg, idx=idx, seg=[0, 512])
    _assert_grads(got, oracle_lib.nsa_backward(*args), cfg.name)


def test_backward_config5_full_size_sampled(B, oracle_lib):
    """Full-size launch of config 5; the oracle evaluates dq on sampled query blocks and dk, dv on
    sampled key blocks (contributions of every query of the sequence), three heads."""
    cfg = I.CONFIGS[5]
    qblocks = I.sample_query_blocks(cfg, 3)
    kblocks = I.sample_query_blocks(cfg, 2, seed=5)[::2]
    heads = [0, 7, cfg.heads - 1]
    _log(f"[backward] config 5 full-size launch; oracle on {len(qblocks)} query blocks, {len(kblocks)} key blocks, "
         f"heads {heads}")
    got, args = _case(B, oracle_lib, cfg)
    (q, k, v, kc, vc, idx, gates, seg_arr, window, dout) = args
    ref = oracle_lib.nsa_backward_sampled(q, k, v, kc, vc, idx, gates, seg_arr, window, dout, qblocks, kblocks, heads)
    rows_q = (np.asarray(qblocks)[:, None] * 64 + np.arange(64)[None]).reshape(-1)
    rows_k = (np.asarray(kblocks)[:, None] * 64 + np.arange(64)[None]).reshape(-1)
    sub = (got[0][rows_q][:, heads], got[1][rows_k][:, heads], got[2][rows_k][:, heads])
    _assert_grads(sub, ref, "config5-sampled")
    assert all(np.isfinite(g).all() for g in got)


def test_backward_wide_heads_many_tiles_sampled(B, oracle_lib):
    """Head dimension 128 (the shape of config 4's heads) on a sequence long enough for thousands of workgroups,
    several window tiles per key block and reverse lists of uneven length: sampled like the test above, plus
    two runs compared bit for bit."""
    cfg = I.small_config(name="b-d128-mid", n_obj=32768, n_views=4, grid=64, heads=2, d=128, topk=16, window=512,
                         seed=61)
    qblocks = I.sample_query_blocks(cfg, 3)
    kblocks = I.sample_query_blocks(cfg, 2, seed=5)[::2]
    heads = [0, 1]
    _log(f"[backward] {cfg.name}: N {cfg.n}; oracle on {len(qblocks)} query blocks, {len(kblocks)} key blocks")
    got, args = _case(B, oracle_lib, cfg)
    (q, k, v, kc, vc, idx, gates, seg_arr, window, dout) = args
    ref = oracle_lib.nsa_backward_sampled(q, k, v, kc, vc, idx, gates, seg_arr, window, dout, qblocks, kblocks, heads)
    rows_q = (np.asarray(qblocks)[:, None] * 64 + np.arange(64)[None]).reshape(-1)
    rows_k = (np.asarray(kblocks)[:, None] * 64 + np.arange(64)[None]).reshape(-1)
    sub = (got[0][rows_q][:, heads], got[1][rows_k][:, heads], got[2][rows_k][:, heads])
    _assert_grads(sub, ref, cfg.name)
    assert all(np.isfinite(g).all() for g in got)
    again, _ = _case(B, oracle_lib, cfg)
    for x, y in zip(got, again):
        assert np.array_equal(x, y)


def test_backward_is_deterministic(B, oracle_lib):
    cfg = I.small_config(name="b-det", n_obj=1024, n_views=2, grid=16, heads=2, d=64, topk=4, window=256)
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    idx, _ = oracle_lib.route(I.make_points(cfg), I.make_cameras(cfg), cfg.grid, cfg.topk)
    a = G.run_backward(B, cfg, q_bits, k_bits, v_bits, idx, gates, dout_bits)
    b = G.run_backward(B, cfg, q_bits, k_bits, v_bits, idx, gates, dout_bits)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


def test_backward_full_size_is_deterministic(B, oracle_lib):
    """Config 5 at full size, three calls in a row (workspaces reused with whatever the call before left
    in them, the chip fully loaded): a tile read before its copy has landed shows up as a difference."""
    cfg = I.CONFIGS[5]
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    idx, _ = oracle_lib.route(I.make_points(cfg), I.make_cameras(cfg), cfg.grid, cfg.topk)
    _log("[backward] config 5, three runs")
    runs = [G.run_backward(B, cfg, q_bits, k_bits, v_bits, idx, gates, dout_bits) for _ in range(3)]
    for other in runs[1:]:
        for x, y in zip(runs[0], other):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("d,heads,h_kv", [(64, 2, 2), (32, 6, 2), (128, 1, 1)])
def test_backward_lists_cut_into_parts(B, oracle_lib, d, heads, h_kv):
    """Walks at the edges of the parts they are cut into (16 tiles at this size, 6 of them the window's away from the ends of
    the sequence): lists of 4, 5, 6 and 13, 14 entries and one of an entry per row, without grouped heads and with
    three to a key/value head, a workgroup each."""
    cfg = I.small_config(name=f"b-parts-d{d}", n_obj=45 * 64, n_views=1, grid=16, heads=heads, d=d, topk=6, window=96,
                         seed=29, h_kv=h_kv)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    idx = np.full((cfg.nb, cfg.topk), -1, dtype=np.int32)
    for col, (block, rows) in enumerate(((3, cfg.nb), (5, 4), (7, 5), (11, 6), (12, 13), (30, 14))):
        idx[(np.arange(rows) * 3) % cfg.nb, col] = block
    assert [int((idx == b).sum()) for b in (3, 5, 7, 11, 12, 30)] == [49, 4, 5, 6, 13, 14]
    got, args = _case(B, oracle_lib, cfg, idx=idx)
    _assert_grads(got, oracle_lib.nsa_backward(*args), cfg.name)


@pytest.mark.parametrize("d,heads,h_kv", [(64, 2, 2), (32, 4, 1), (128, 1, 1)])
def test_backward_unlimited_window(B, oracle_lib, d, heads, h_kv):
    """The largest even window there is (2^31 - 2) means "the whole segment": the same gradients, bit for bit, as a window
    of twice the sequence, and the oracle's."""
    cfg = I.small_config(name=f"b-unlimited-d{d}", n_obj=21 * 64, n_views=1, grid=16, heads=heads, d=d, topk=3, window=64,
                         seed=31, h_kv=h_kv)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    got, _ = _case(B, oracle_lib, cfg, window=2147483646)
    covering, args = _case(B, oracle_lib, cfg, window=2 * cfg.n)
    for x, y in zip(got, covering):
        assert np.array_equal(x, y)
    _assert_grads(got, oracle_lib.nsa_backward(*args), cfg.name)


@pytest.mark.parametrize("d,heads,h_kv,window", [(64, 1, 1, 1024), (128, 1, 1, 962), (32, 4, 2, 962)])
def test_backward_walks_cut_inside_the_window(B, oracle_lib, d, heads, h_kv, window):
    """Windows of two and more parts (at this size a walk is cut every 16 tiles, every 20 with two heads to a key/value
    head): parts of window tiles only, one that holds the window's end and list entries, and the odd tile by which a window
    of an odd number of tiles falls short of its even share.  Lists of 0, 1, 8 and 14 entries behind it; without grouped
    heads and with two to a key/value head, a workgroup each."""
    cfg = I.small_config(name=f"b-window-parts-d{d}-w{window}", n_obj=45 * 64, n_views=1, grid=16, heads=heads, d=d, topk=3,
                         window=window, seed=33, h_kv=h_kv)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    # tiles that see block b in the window: queries of its segment from 64 b - W/2 + 1 to 64 b + 63 + W/2
    b = np.arange(cfg.nb_obj)
    first = np.maximum(0, 64 * b - window // 2 + 1) // 32
    tiles = (np.minimum(cfg.n_obj, 64 * b + 64 + window // 2) - 1) // 32 + 1 - first
    assert tiles.max() == {1024: 34, 962: 33}[window]
    idx = np.full((cfg.nb, cfg.topk), -1, dtype=np.int32)
    for col, (block, rows) in enumerate(((22, 14), (2, 8), (23, 1))):
        idx[(np.arange(rows) * 3) % cfg.nb, col] = block
    got, args = _case(B, oracle_lib, cfg, idx=idx)
    _assert_grads(got, oracle_lib.nsa_backward(*args), cfg.name)


def test_backward_of_more_tiles_than_one_grid_direction_holds(B):
    """358 M tokens of one head: three images per 64-token block are more workgroups than a launch takes in one direction.
    q, k, v, dout and the branch outputs are ones in the same memory, and every query sees itself and the key before it
    (window 2, the other branches gated off): probabilities of a half, dq = dk = 0, and dv[j] = 1/2 from query j + 1/2
    from query j + 1, which the last token does not have."""
    import torch
    nb, d = 5_600_000, 32
    assert 3 * nb * 256 >= 2 ** 32
    n = nb * 64
    if torch.cuda.mem_get_info()[0] < 230 << 30:
        pytest.skip("needs 230 GiB of free GPU memory")
    _log(f"[backward] {nb} blocks of one head")
    dev = torch.device("cuda")
    goff = (torch.arange(65, device=dev) * (nb // 64)).to(torch.int32)   # (64 pooled pairs)
    goff[-1] = nb
    p = B.make_params(n, 0, 0, 1, d, 0, 2, group_offsets=goff)
    branches = torch.ones((3, n, 1, d), dtype=torch.bfloat16, device=dev)
    ones = branches[0]
    kc = torch.ones((64, 1, d), dtype=torch.bfloat16, device=dev)
    idx = torch.zeros((nb, 1), dtype=torch.int32, device=dev)
    gates = torch.zeros((n, 1, 3), dtype=torch.float32, device=dev)
    gates[:, :, 2] = 1.0
    lse = torch.full((3, n, 1), d ** 0.5 + float(np.log(2.0)), dtype=torch.float32, device=dev)
    dq, dv = (torch.full((n, 1, d), float("nan"), dtype=torch.bfloat16, device=dev) for _ in range(2))
    ws = B.alloc_workspace(p, B.LSRM_WS_BACKWARD)
    B.lsrm_nsa_backward(p, ones, ones, ones, kc, kc, idx, gates, lse, branches, ones, dq, dq, dv, ws)
    torch.cuda.synchronize()
    # (extremes instead of a comparison with a tensor of the same size; NaN fails both)
    rest, last = dv[:-1], dv[-1]
    found = [float(x) for x in (dq.min(), dq.max(), rest.min(), rest.max(), last.min(), last.max())]
    del branches, ones, gates, lse, dq, dv, ws, rest, last
    torch.cuda.empty_cache()
    assert found == [0.0, 0.0, 1.0, 1.0, 0.5, 0.5]


@pytest.mark.parametrize("d,heads,h_kv,n_blocks,channels", [(64, 2, 2, 148, False), (32, 3, 1, 133, True), (128, 1, 1, 140, False)])
def test_backward_same_problem_on_both_sides_of_the_small_ones(B, oracle_lib, d, heads, h_kv, n_blocks, channels):
    """A table of few entries goes through the joint launches of small problems, the same table with columns of holes up to more
    than 16384 entries through the general ones: both against the oracle.  Popular blocks (walks of many parts), blocks
    that nobody lists, a block listed twice in a row, rows of holes."""
    topk, wide = 4, 127
    cfg = I.small_config(name=f"b-routes-d{d}", n_obj=64 * (n_blocks - 1), n_views=1, grid=8, heads=heads, d=d, topk=topk,
                         window=160, seed=77, h_kv=h_kv, gate_channels=channels)
    assert cfg.nb == n_blocks and n_blocks * topk <= 16384 < n_blocks * wide
    rng = np.random.default_rng(6)
    idx = np.stack([rng.choice(cfg.nb // 2, size=topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[:, 0] = 5          # every row: a walk of many parts
    idx[::3, 1] = 5        # and twice in some
    idx[1::4, 2:] = -1
    idx[7] = -1
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    got, args = _case(B, oracle_lib, cfg, idx=idx)
    ref = oracle_lib.nsa_backward(*args)
    _assert_grads(got, ref, cfg.name + " small")
    holes = np.full((cfg.nb, wide - topk), -1, dtype=np.int32)
    padded = dataclasses.replace(cfg, topk=wide)
    got, _ = _case(B, oracle_lib, padded, idx=np.concatenate([idx[:, :2], holes, idx[:, 2:]], axis=1))
    _assert_grads(got, ref, cfg.name + " general")


@pytest.mark.parametrize("n_blocks,topk", [(768, 3), (769, 3), (300, 54), (300, 55)])
def test_backward_preparation_on_both_sides_of_its_sizes(B, oracle_lib, n_blocks, topk):
    """Up to 768 blocks and 16384 table entries one launch prepares the walks, above that five do (with more pairs of a block
    and a head than the joint launches of small problems take): a popular block, whose walk has many parts, and
    rows with holes; sampled against the oracle, and the same twice."""
    cfg = I.small_config(name=f"b-table{n_blocks}-{topk}", n_obj=64 * (n_blocks - 1), n_views=1, grid=8, heads=11, d=32, topk=topk,
                         window=64, seed=78)
    assert cfg.nb == n_blocks and cfg.nb * cfg.heads > 3072
    rng = np.random.default_rng(9)
    idx = np.full((cfg.nb, topk), -1, dtype=np.int32)
    idx[:, :3] = rng.integers(0, cfg.nb, size=(cfg.nb, 3))
    idx[:, topk - 1] = 17
    idx[::5, 0] = -1
    qblocks, kblocks, heads = [0, 17, cfg.nb - 2, cfg.nb - 1], [0, 5, 17, cfg.nb - 2, cfg.nb - 1], [0, 10]
    _log(f"[backward] {cfg.name} nb={cfg.nb} entries={cfg.nb * topk}")
    got, args = _case(B, oracle_lib, cfg, idx=idx)
    ref = oracle_lib.nsa_backward_sampled(*args, qblocks, kblocks, heads)
    rows_q, rows_k = ((np.asarray(b)[:, None] * 64 + np.arange(64)[None]).reshape(-1) for b in (qblocks, kblocks))
    _assert_grads((got[0][rows_q][:, heads], got[1][rows_k][:, heads], got[2][rows_k][:, heads]), ref, cfg.name)
    again, _ = _case(B, oracle_lib, cfg, idx=idx)
    for x, y in zip(got, again):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("d,n_blocks,heads,h_kv", [(128, 64, 21, 3), (128, 65, 21, 3), (128, 128, 21, 7), (128, 129, 11, 11), (128, 193, 7, 7),
                                                   (128, 65, 3, 3), (64, 300, 11, 11), (32, 129, 26, 13), (128, 511, 2, 2),
                                                   (128, 512, 4, 2), (128, 513, 2, 1), (128, 575, 1, 1), (128, 609, 2, 2)])
def test_backward_pooled_keys_at_the_edges_of_their_groups(B, oracle_lib, d, n_blocks, heads, h_kv):
    """Numbers of pooled keys around those a workgroup takes (64; 128 from 512 keys on at d = 128, the last workgroup with one
    to four wavefronts that have any), and of walks that eight does not divide, above the limits of the joint launches and
    once below: sampled against the oracle, first and last blocks, keys and heads."""
    cfg = I.small_config(name=f"b-pooled{n_blocks}-{heads}-{d}", n_obj=64 * (n_blocks - 1), n_views=1, grid=8, heads=heads, d=d, topk=4,
                         window=96, seed=79, h_kv=h_kv)
    assert cfg.nb == n_blocks
    rng = np.random.default_rng(10)
    idx = np.stack([rng.choice(cfg.nb, size=4, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    blocks, some = sorted({0, 63, min(64, cfg.nb - 1), cfg.nb - 2, cfg.nb - 1}), sorted({0, heads // 2, heads - 1})
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    got, args = _case(B, oracle_lib, cfg, idx=idx)
    kv = sorted({h // (heads // h_kv) for h in some})
    ref = oracle_lib.nsa_backward_sampled(*args, blocks, blocks, some, kv_heads=kv)
    rows = (np.asarray(blocks)[:, None] * 64 + np.arange(64)[None]).reshape(-1)
    _assert_grads((got[0][rows][:, some], got[1][rows][:, kv], got[2][rows][:, kv]), ref, cfg.name)


@pytest.mark.parametrize("d,heads,h_kv,channels", [(32, 9, 1, False), (64, 8, 1, False), (32, 7, 1, True), (128, 4, 2, False)])
def test_backward_heads_of_a_group_dealt_to_two_or_to_one(B, oracle_lib, d, heads, h_kv, channels):
    """Groups of eight and more heads in the general launches go to two workgroups (nine: five and four), smaller ones stay
    together; the joint launches deal groups of seven and more to two here; walks cut into parts of few tiles by many heads,
    the most popular into dozens.
    Bar: 2e-2 plus 2^-7 of the largest reference value of the row, as for the other large sums over a group."""
    n_blocks, topk, wide = 130, 4, 127
    cfg = I.small_config(name=f"b-dealt-d{d}-h{heads}", n_obj=64 * (n_blocks - 1), n_views=1, grid=8, heads=heads, d=d, topk=topk,
                         window=224, seed=79, h_kv=h_kv, gate_channels=channels)
    rng = np.random.default_rng(8)
    idx = np.stack([rng.choice(cfg.nb // 2, size=topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[:, 0] = np.where(np.arange(cfg.nb) % 2, 5, 70)
    idx[3] = -1
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    holes = np.full((cfg.nb, wide - topk), -1, dtype=np.int32)
    ref = None
    for what, c, table in (("small", cfg, idx), ("general", dataclasses.replace(cfg, topk=wide), np.concatenate([idx, holes], axis=1))):
        got, args = _case(B, oracle_lib, c, idx=table)
        ref = oracle_lib.nsa_backward(*args) if ref is None else ref
        for name, g, r in zip(("dq", "dk", "dv"), got, ref):
            excess = np.abs(g - r) - (G.MAX_ABS_TOL + np.abs(r).max(axis=-1, keepdims=True) * 2.0 ** -7)
            _, rl = G.attention_errors(g, r)
            _log(f"[backward] {cfg.name} {what} {name}: worst excess over the bar {excess.max():.3e}, rel-L2 {rl:.3e}")
            assert excess.max() <= 0.0 and rl <= G.REL_L2_TOL, (what, name, float(excess.max()), rl)


@pytest.mark.parametrize("d,n_blocks,topk,channels", [(32, 2049, 4, True), (64, 2049, 65, False), (64, 2080, 4, True), (128, 2049, 4, False),
                                                      (128, 2048, 66, True)])
def test_backward_two_query_blocks_to_a_workgroup(B, oracle_lib, d, n_blocks, topk, channels):
    """From 2048 pooled keys on a workgroup of the dQ pass has two query blocks of a head (at d = 32 one): an odd number of blocks,
    partners with rows of very different numbers of valid entries, in narrow and wide tables; heads with key/value heads of their own."""
    heads = 3
    cfg = I.small_config(name=f"b-two-blocks{n_blocks}-{d}", n_obj=64 * (n_blocks - 1), n_views=1, grid=8, heads=heads, d=d, topk=topk,
                         window=224, seed=80, gate_channels=channels)
    assert cfg.nb == n_blocks
    rng = np.random.default_rng(14)
    idx = rng.integers(0, cfg.nb // topk, size=(cfg.nb, topk)) * topk + np.arange(topk)  # (no block twice in a row)
    idx = np.where(idx < cfg.nb, idx, -1).astype(np.int32)
    idx[1::4, 1:] = -1
    idx[2] = idx[-1] = -1
    blocks = sorted({0, 1, 2, 3, 4, 5, cfg.nb - 2, cfg.nb - 1})
    _log(f"[backward] {cfg.name} nb={cfg.nb}")
    got, args = _case(B, oracle_lib, cfg, idx=idx)
    dq, _, _ = oracle_lib.nsa_backward_sampled(*args, blocks, [], [0, 2])
    rows = (np.asarray(blocks)[:, None] * 64 + np.arange(64)[None]).reshape(-1)
    _assert_grads((got[0][rows][:, [0, 2]],), (dq,), cfg.name)


@pytest.mark.parametrize("d,heads,h_kv,n_blocks,n_groups,topk,window,window_mode,with_counts,channels", [
    (64, 1, 1, 2049, 0, 4, 224, 1, True, False),     # the window is the query's own block
    (128, 3, 1, 2051, 0, 66, 224, 0, True, True),
    (64, 3, 1, 2500, 2049, 5, 224, 1, True, False),  # the window is the spatial block: partners of very different lengths
    (128, 1, 1, 2701, 2048, 3, 160, 1, True, True),
    (128, 5, 1, 2048, 0, 1, 0, 0, False, False),     # half of the blocks have the pooled keys only
    (64, 3, 3, 2047, 0, 4, 224, 0, True, False),     # one pooled key too few
])
def test_backward_two_query_blocks_and_two_heads_to_a_workgroup(B, d, heads, h_kv, n_blocks, n_groups, topk, window, window_mode,
                                                                with_counts, channels):
    """The dQ pass with two query blocks to a workgroup and, every query head given twice, with two heads to one: the same
    bits in every row, and again in a second run.  Active counts, both windows, spatial blocks, groups of three and five."""
    cfg = I.small_config(name=f"b-both-pairs{n_blocks}-{d}", n_obj=64 * (n_blocks - 1), n_views=1, grid=8, heads=heads, d=d, topk=topk,
                         window=window, seed=81, h_kv=h_kv, gate_channels=channels)
    rng = np.random.default_rng(15)
    goff = None
    if n_groups:   # (the last spatial block of more than one block and an image tile of its own)
        ends = np.sort(rng.choice(np.arange(1, n_blocks - 1), size=n_groups - 2, replace=False))
        goff = np.concatenate([[0], ends, [n_blocks - 1, n_blocks]]).astype(np.int32)
    cnt = rng.integers(1, 65, size=n_blocks).astype(np.int32) if with_counts else None
    idx = rng.integers(0, cfg.nb, size=(cfg.nb, topk)).astype(np.int32)
    idx[1::4, 1:] = -1
    idx[::2] = np.where(rng.random(idx[::2].shape) < 0.5, -1, idx[::2])
    idx[2] = idx[-1] = -1
    if topk == 1:
        idx[1::2] = -1
    q, k, v = I.make_qkv(cfg)
    gates, dout = I.make_gates(cfg), I.make_dout(cfg)
    twice = dataclasses.replace(cfg, heads=2 * heads)
    _log(f"[backward] {cfg.name} nb={cfg.nb}")

    def run(c, copies):
        def of(x, axis):
            return np.ascontiguousarray(np.repeat(x, copies, axis=axis))
        return G.run_backward(B, c, of(q, 1), k, v, idx, of(gates, 2 if channels else 1), of(dout, 1), window_mode=window_mode,
                              block_count=cnt, group_offsets=goff)

    runs, pairs = [run(cfg, 1) for _ in range(2)], [run(twice, 2) for _ in range(2)]
    for one, other in (runs, pairs):
        for x, y in zip(one, other):
            assert np.isfinite(x).all() and np.array_equal(x, y)
    assert np.array_equal(pairs[0][0], np.repeat(runs[0][0], 2, axis=1))
