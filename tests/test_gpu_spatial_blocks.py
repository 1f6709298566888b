"""GPU parity with spatial blocks larger than 64 tokens (Sec. 3.2: 8 x 8 x 8 volume blocks hold up to 512 active
tokens), given as groups of consecutive 64-slot blocks: one compressed pair per spatial block, the own-block window
over the whole spatial block, gradients handed back to all its active tokens.  Compress, forward and backward
against the oracle, element by element."""
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


def _groups(nb, rng, max_blocks=8):
    """Random spatial blocks of 1..max_blocks 64-slot blocks covering nb blocks; a few sizes forced in."""
    sizes = [1, max_blocks, 2, 3]
    while sum(sizes) < nb:
        sizes.append(int(rng.integers(1, max_blocks + 1)))
    over = sum(sizes) - nb
    while over > 0:                      # trim from the end
        take = min(over, sizes[-1] - 1) if sizes[-1] > 1 else 1
        if sizes[-1] - take <= 0:
            sizes.pop()
        else:
            sizes[-1] -= take
        over = sum(sizes) - nb
    assert sum(sizes) == nb and min(sizes) >= 1
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)


def _case(cfg, seed, with_counts, topk, min_count=1):
    rng = np.random.default_rng(seed)
    goff = _groups(cfg.nb, rng)
    idx = np.stack([rng.choice(cfg.nb, size=topk, replace=False) for _ in range(cfg.nb)]).astype(np.int32)
    idx[rng.random(idx.shape) < 0.15] = -1
    cnt = None
    if with_counts:
        # a spatial block fills its 64-slot blocks in order: only its last block is partly filled; two blocks in the
        # middle of groups are made partial as well (the kernels mask per 64-slot block)
        cnt = np.full(cfg.nb, 64, dtype=np.int32)
        cnt[goff[1:] - 1] = rng.integers(min_count, 65, size=len(goff) - 1)
        cnt[goff[1] + 2] = 31
        cnt[goff[2]] = max(5, min_count)
    return goff, idx, cnt


def _poison(cfg, cnt, *bits):
    if cnt is None:
        return bits
    inactive = (np.arange(cfg.n) % 64) >= np.repeat(cnt, 64)
    out = []
    for b in bits:
        b = b.copy()
        b[inactive] = 0x7FC0
        out.append(b)
    return out


@pytest.mark.parametrize("d,heads,h_kv,window_mode,with_counts", [(64, 2, 2, 1, False), (128, 2, 2, 1, True),
                                                                  (64, 4, 2, 0, True), (32, 4, 1, 1, True),
                                                                  (128, 3, 3, 0, False),
                                                                  # more than 256 workgroups: the general kernel
                                                                  (64, 10, 2, 1, False), (128, 6, 2, 1, True), (64, 12, 2, 0, True),
                                                                  (32, 12, 1, 1, True), (128, 6, 3, 0, False)])
def test_forward_with_spatial_blocks(B, oracle_lib, d, heads, h_kv, window_mode, with_counts):
    cfg = I.small_config(name=f"g-fwd-d{d}-w{window_mode}-cnt{int(with_counts)}", n_obj=2368, n_views=2, grid=24,
                         heads=heads, d=d, topk=6, window=160, seed=91, h_kv=h_kv)
    goff, idx, cnt = _case(cfg, 3, with_counts, cfg.topk)
    _log(f"[spatial blocks] {cfg.name}: {cfg.nb} blocks of 64 slots in {len(goff) - 1} spatial blocks of "
         f"{np.diff(goff).min()}..{np.diff(goff).max()}")
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates = I.make_gates(cfg)
    k_bits, v_bits = _poison(cfg, cnt, k_bits, v_bits)
    for fused in (False, True):
        res = G.run_forward(B, cfg, q_bits, k_bits, v_bits, idx, gates, want_aux=True, window_mode=window_mode,
                            block_count=cnt, group_offsets=goff, fused_pack=fused)
        q, k, v = (I.bf16_bits_to_f32(a) for a in (q_bits, k_bits, v_bits))
        kc, vc = oracle_lib.pool(k, cnt, goff), oracle_lib.pool(v, cnt, goff)
        assert res["kc"].shape == kc.shape == (len(goff) - 1, h_kv, d)
        for got, ref in ((res["kc"], kc), (res["vc"], vc)):
            assert np.all(np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 + 1e-6)
        ref_out, ref_lse, ref_ob = oracle_lib.nsa_forward(q, k, v, kc, vc, idx, gates, cfg.seg_offsets(), cfg.window,
                                                          want_lse=True, want_branches=True, window_mode=window_mode,
                                                          block_count=cnt, group_offsets=goff)
        act = np.ones(cfg.n, dtype=bool) if cnt is None else (np.arange(cfg.n) % 64) < np.repeat(cnt, 64)
        for name, got, ref in (("out", res["out"], ref_out), ("cmp", res["ob"][0], ref_ob[0]),
                               ("sel", res["ob"][1], ref_ob[1]), ("win", res["ob"][2], ref_ob[2])):
            ma, rl = G.attention_errors(got[act], ref[act])
            _log(f"    fused={fused} {name}: max-abs {ma:.3e} rel-L2 {rl:.3e}")
            assert ma <= G.MAX_ABS_TOL and rl <= G.REL_L2_TOL
        fin = np.isfinite(ref_lse[:, act])
        assert np.array_equal(np.isfinite(res["lse"][:, act]), fin)
        assert np.abs(res["lse"][:, act][fin] - ref_lse[:, act][fin]).max() <= 2e-2


@pytest.mark.parametrize("d,heads,h_kv,window_mode,with_counts", [(64, 2, 2, 1, False), (128, 2, 2, 1, True),
                                                                  (64, 4, 2, 0, True), (32, 4, 1, 1, True)])
def test_backward_with_spatial_blocks(B, oracle_lib, d, heads, h_kv, window_mode, with_counts):
    cfg = I.small_config(name=f"g-bwd-d{d}-w{window_mode}-cnt{int(with_counts)}", n_obj=1088, n_views=2, grid=16,
                         heads=heads, d=d, topk=4, window=160, seed=93, h_kv=h_kv)
    # (spatial blocks hold at least 8 active tokens here: a pooled pair hands the gradient it collects from every
    # query of the sequence to its tokens, divided by their number -- with a single token nothing averages the bf16
    # noise of those 1600 contributions down, and it reaches 0.03-0.05 on that one row)
    goff, idx, cnt = _case(cfg, 5, with_counts, cfg.topk, min_count=8)
    _log(f"[spatial blocks] {cfg.name}: {cfg.nb} blocks in {len(goff) - 1} spatial blocks")
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    if heads != h_kv:   # keep the summed gradients of a key/value head at the magnitude the absolute bar was set for
        dout_bits = I.f32_to_bf16_bits(I.bf16_bits_to_f32(dout_bits) * np.float32(h_kv / heads))
    q, k, v, dout = (I.bf16_bits_to_f32(a) for a in (q_bits, k_bits, v_bits, dout_bits))
    k_bits, v_bits, dout_bits = _poison(cfg, cnt, k_bits, v_bits, dout_bits)
    got = G.run_backward(B, cfg, q_bits, k_bits, v_bits, idx, gates, dout_bits, window_mode=window_mode,
                         block_count=cnt, group_offsets=goff)
    kc, vc = oracle_lib.pool(k, cnt, goff), oracle_lib.pool(v, cnt, goff)
    ref = oracle_lib.nsa_backward(q, k, v, kc, vc, idx, gates, cfg.seg_offsets(), cfg.window, dout,
                                  window_mode=window_mode, block_count=cnt, group_offsets=goff)
    for name, g, r in zip(("dq", "dk", "dv"), got, ref):
        assert np.isfinite(g).all(), name
        ma, rl = G.attention_errors(g, r)
        _log(f"    {name}: max-abs {ma:.3e} rel-L2 {rl:.3e} (|ref| max {np.abs(r).max():.3e})")
        assert ma <= G.MAX_ABS_TOL and rl <= G.REL_L2_TOL, (name, ma, rl)
    if cnt is not None:
        inactive = (np.arange(cfg.n) % 64) >= np.repeat(cnt, 64)
        for g in got:
            assert np.all(g[inactive] == 0)


def _heads(x, n_copies, axis):
    return np.ascontiguousarray(np.concatenate([x] * n_copies, axis=axis))


@pytest.mark.parametrize("d,heads,h_kv,window_mode,grouped_blocks,channels", [
    (64, 2, 2, 1, True, False), (64, 4, 2, 0, False, True), (32, 2, 2, 0, True, False), (32, 4, 2, 1, True, True),
    (32, 2, 2, 1, False, False), (128, 2, 2, 1, True, False), (128, 4, 2, 0, True, True), (128, 2, 2, 1, False, False)])
def test_backward_options_on_every_set_of_launches(B, oracle_lib, d, heads, h_kv, window_mode, grouped_blocks, channels):
    """Active counts, both windows, blocks alone and in spatial blocks, with a block that every row lists (walks of many
    parts): the joint launches of a small problem; the general kernels behind five launches of preparation (holes in the
    table up to more than 16384 entries); the general kernels behind one (copies of the heads)."""
    cfg = I.small_config(name=f"g-sets-d{d}-h{heads}-w{window_mode}-g{int(grouped_blocks)}", n_obj=64 * 139, n_views=1, grid=8,
                         heads=heads, d=d, topk=4, window=160, seed=97, h_kv=h_kv, gate_channels=channels)
    assert cfg.nb == 140
    goff, idx, cnt = _case(cfg, 7, True, cfg.topk, min_count=8)
    idx[:, 1] = np.where(np.arange(cfg.nb) % 5 == 0, -1, 11)
    if not grouped_blocks:
        goff = None
        cnt = np.random.default_rng(8).integers(8, 65, size=cfg.nb).astype(np.int32)
        cnt[:4] = (32, 33, 64, 31)
    _log(f"[sets of launches] {cfg.name}")
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    # (a popular block and a group of heads add up gradients: keep them at the magnitude the absolute bar was set for)
    dout_bits = I.f32_to_bf16_bits(I.bf16_bits_to_f32(dout_bits) * np.float32(0.5 * h_kv / heads))
    q, k, v, dout = (I.bf16_bits_to_f32(a) for a in (q_bits, k_bits, v_bits, dout_bits))
    k_bits, v_bits, dout_bits = _poison(cfg, cnt, k_bits, v_bits, dout_bits)
    ref = oracle_lib.nsa_backward(q, k, v, oracle_lib.pool(k, cnt, goff), oracle_lib.pool(v, cnt, goff), idx, gates,
                                  cfg.seg_offsets(), cfg.window, dout, window_mode=window_mode, block_count=cnt,
                                  group_offsets=goff)
    active = (np.arange(cfg.n) % 64) < np.repeat(cnt, 64)

    def check(cfg, idx, copies, tag):
        got = G.run_backward(B, cfg, _heads(q_bits, copies, 1), _heads(k_bits, copies, 1), _heads(v_bits, copies, 1), idx,
                             _heads(gates, copies, 2 if channels else 1), _heads(dout_bits, copies, 1), window_mode=window_mode,
                             block_count=cnt, group_offsets=goff)
        for name, g, r in zip(("dq", "dk", "dv"), got, ref):
            n_heads = r.shape[1]
            for c in range(1, copies):
                assert np.array_equal(g[:, c * n_heads:(c + 1) * n_heads], g[:, :n_heads]), (tag, name, c)
            g = g[:, :n_heads]
            assert np.isfinite(g).all() and np.all(g[~active] == 0), (tag, name)
            ma, rl = G.attention_errors(g, r)
            _log(f"    {tag} {name}: max-abs {ma:.3e} rel-L2 {rl:.3e} (|ref| max {np.abs(r).max():.3e})")
            assert ma <= G.MAX_ABS_TOL and rl <= G.REL_L2_TOL, (tag, name, ma, rl)

    check(cfg, idx, 1, "joint")
    wide = 120
    assert cfg.nb * wide > 16384
    holes = np.full((cfg.nb, wide - cfg.topk), -1, dtype=np.int32)
    check(dataclasses.replace(cfg, topk=wide), np.concatenate([idx[:, :2], holes, idx[:, 2:]], axis=1), 1, "general, five")
    copies = -(-1281 // (cfg.nb * heads)) if d == 128 else -(-3073 // (cfg.nb * h_kv))
    check(dataclasses.replace(cfg, heads=copies * heads, h_kv=copies * h_kv), idx, copies, "general, one")


@pytest.mark.parametrize("n_groups,with_counts", [(511, True), (512, False), (513, True), (576, True), (641, False)])
def test_backward_many_pairs_of_spatial_blocks(B, n_groups, with_counts):
    """At d = 128 workgroups of 128 pooled keys from 512 on, here fewer pairs than blocks: the compressed branch alone (no
    routed blocks, no window) against its formulas in float64."""
    import torch
    cfg = I.small_config(name=f"g-pairs{n_groups}", n_obj=64 * 699, n_views=1, grid=8, heads=2, d=128, topk=1, window=0, seed=98,
                         h_kv=1)
    assert cfg.nb == 700
    rng = np.random.default_rng(n_groups)
    goff = np.concatenate([[0], np.sort(rng.choice(np.arange(1, cfg.nb), size=n_groups - 1, replace=False)), [cfg.nb]]).astype(np.int32)
    cnt = rng.integers(8, 65, size=cfg.nb).astype(np.int32) if with_counts else np.full(cfg.nb, 64, dtype=np.int32)
    _log(f"[spatial blocks] {cfg.name}")
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    idx = np.full((cfg.nb, 1), -1, dtype=np.int32)
    count = cnt if with_counts else None
    _, _, kc, vc = G.run_compress(B, cfg, k_bits, v_bits, count, goff)
    k_in, v_in, do_in = _poison(cfg, count, k_bits, v_bits, dout_bits)
    got = G.run_backward(B, cfg, q_bits, k_in, v_in, idx, gates, do_in, block_count=count, group_offsets=goff)

    active = torch.from_numpy((np.arange(cfg.n) % 64) < np.repeat(cnt, 64)).cuda()
    group = torch.from_numpy(np.repeat(np.repeat(np.arange(n_groups), np.diff(goff)), 64)).cuda()
    q, do = (torch.from_numpy(I.bf16_bits_to_f32(a)).cuda().double() for a in (q_bits, dout_bits))
    gate = torch.from_numpy(gates[:, :, 0]).cuda().double()
    kc, vc = kc[:, 0].double(), vc[:, 0].double()
    scale = cfg.d ** -0.5
    dq, dkc, dvc = torch.zeros_like(q), torch.zeros_like(kc), torch.zeros_like(vc)
    for h in range(cfg.heads):
        qh, doh = q[active][:, h], (do * gate[:, :, None])[active][:, h]
        p = torch.softmax(qh @ kc.T * scale, dim=1)
        dp = doh @ vc.T
        ds = p * (dp - (p * dp).sum(1, keepdim=True)) * scale
        dq[active, h] = ds @ kc
        dkc += ds.T @ qh
        dvc += p.T @ doh
    n_tok = torch.zeros(n_groups, dtype=torch.float64, device="cuda").index_add_(0, group, active.double())
    dk, dv = ((x / n_tok[:, None])[group] * active[:, None] for x in (dkc, dvc))
    for name, g, r in zip(("dq", "dk", "dv"), got, (dq, dk[:, None], dv[:, None])):
        r = r.cpu().numpy()
        assert np.isfinite(g).all() and np.all(g[~active.cpu().numpy()] == 0), name
        # (gradients of pairs are far below the absolute bar here: the relative one, and a tenth of the largest row's size)
        ma, rl = G.attention_errors(g, r)
        _log(f"    {name}: max-abs {ma:.3e} rel-L2 {rl:.3e} (|ref| max {np.abs(r).max():.3e})")
        assert rl <= G.REL_L2_TOL and ma <= 0.1 * np.abs(r).max(), (name, ma, rl)


def test_group_arguments_are_checked(B):
    import torch
    off = torch.tensor([0, 2, 8], dtype=torch.int32, device="cuda")
    ok = B.make_params(512, 0, 16, 2, 64, 3, 128, group_offsets=off)
    assert B.lsrm_workspace_bytes(ok, B.LSRM_WS_FORWARD) > 0 and B.lsrm_workspace_bytes(ok, B.LSRM_WS_BACKWARD) > 0
    bad = B.make_params(512, 0, 16, 2, 64, 3, 128, group_offsets=off)
    bad.n_groups = 9          # more spatial blocks than 64-slot blocks
    assert B.lsrm_workspace_bytes(bad, B.LSRM_WS_FORWARD) == 0
    none = B.make_params(512, 0, 16, 2, 64, 3, 128)
    none.n_groups = 2         # a count without offsets
    assert B.lsrm_workspace_bytes(none, B.LSRM_WS_FORWARD) == 0


@pytest.mark.parametrize("d,h_kv,with_counts", [(32, 1, True), (64, 3, True), (64, 2, False), (128, 5, True)])
def test_pooling_of_spatial_blocks_edges(B, oracle_lib, d, h_kv, with_counts):
    """Spatial blocks of 1, 2, 3, 8, 16 and 17 blocks (one pass over 128 slots, several, one past a whole number) at rows
    of 4, 24, 16 and 80 chunks of 8 channels (16 share a workgroup); one active token in the last block."""
    import torch
    cfg = I.small_config(name=f"g-pool-d{d}-h{h_kv}", n_obj=64 * 47, n_views=0, grid=0, heads=h_kv, d=d, topk=1, window=64)
    goff = np.concatenate([[0], np.cumsum([1, 2, 3, 8, 16, 17])]).astype(np.int32)
    rng = np.random.default_rng(5)
    cnt = None
    if with_counts:
        cnt = np.full(cfg.nb, 64, dtype=np.int32)
        cnt[goff[1:] - 1] = [1, 17, 64, 33, 2, 1]
    bits = [I.f32_to_bf16_bits(rng.standard_normal((cfg.n, h_kv, d)).astype(np.float32)) for _ in range(2)]
    bits = _poison(cfg, cnt, *bits)
    dev = torch.device("cuda")
    p = B.make_params(cfg.n_obj, 0, 0, h_kv, d, 1, 64, h_kv=h_kv, group_offsets=torch.from_numpy(goff).to(dev),
                      block_count=None if cnt is None else torch.from_numpy(cnt).to(dev))
    k, v = (torch.from_numpy(b.view(np.int16)).to(dev).view(torch.bfloat16) for b in bits)
    kc = torch.empty((len(goff) - 1, h_kv, d), dtype=torch.bfloat16, device=dev)
    vc = torch.empty_like(kc)
    _log(f"[pool] {cfg.name}")
    B.lsrm_nsa_compress(p, k, v, kc, vc)
    torch.cuda.synchronize()
    active = np.arange(cfg.n) % 64 < (64 if cnt is None else np.repeat(cnt, 64))
    for got, b in ((kc, bits[0]), (vc, bits[1])):
        x = I.bf16_bits_to_f32(b).astype(np.float64)
        for g in range(len(goff) - 1):
            sl = slice(64 * goff[g], 64 * goff[g + 1])
            ref = x[sl][active[sl]].mean(axis=0)
            assert np.all(np.abs(got[g].double().cpu().numpy() - ref) <= np.abs(ref) * 2.0 ** -8 + 1e-6)


@pytest.mark.parametrize("d,h_kv,n_groups,max_size", [
    (32, 1, 10, 8),       # rows of 4 chunks: four groups side by side, two of the last four missing
    (64, 1, 7, 1), (32, 2, 9, 2),  # of 8, short groups: two side by side, one missing
    (32, 2, 7, 17),       # of 8, long groups: one, half of the lanes idle
    (32, 3, 6, 3),        # of 12
    (128, 4, 2048, 3),    # of 64, as many groups as the wide form starts from
    (64, 24, 700, 3),     # of 192, wide: three sets of chunks
    (128, 4, 2047, 2),    # one group less
], ids=lambda v: str(v))
def test_pooling_of_spatial_blocks_layouts(B, d, h_kv, n_groups, max_size):
    """Every layout of the pooling kernel, at the shapes where its workgroups are partly filled."""
    import torch
    rng = np.random.default_rng(n_groups + max_size)
    sizes = rng.integers(1, max_size + 1, size=n_groups)
    sizes[-1] = max_size
    goff = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    nb = int(goff[-1])
    cnt = np.full(nb, 64, dtype=np.int32)
    cnt[goff[1:] - 1] = rng.integers(1, 65, size=n_groups)
    _log(f"[pool] {n_groups} groups in {nb} blocks, {h_kv} heads of {d}")
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(n_groups)
    k, v = (torch.randn((nb * 64, h_kv, d), generator=gen, device=dev, dtype=torch.bfloat16) for _ in range(2))
    slot = torch.arange(nb * 64, device=dev) % 64
    active = slot < torch.from_numpy(cnt).to(dev).repeat_interleave(64)
    k[~active] = float("nan")   # (whatever sits in padding slots is never read)
    v[~active] = float("inf")
    p = B.make_params(nb * 64, 0, 0, h_kv, d, 1, 64, h_kv=h_kv, group_offsets=torch.from_numpy(goff).to(dev),
                      block_count=torch.from_numpy(cnt).to(dev))
    kc = torch.full((n_groups, h_kv, d), -1.0, dtype=torch.bfloat16, device=dev)
    vc = torch.full_like(kc, -1.0)
    B.lsrm_nsa_compress(p, k, v, kc, vc)
    torch.cuda.synchronize()
    group = torch.from_numpy(np.repeat(np.arange(n_groups), 64 * sizes)).to(dev)
    tokens = torch.zeros(n_groups, dtype=torch.float64, device=dev).index_add_(0, group, active.double())
    for got, x in ((kc, k), (vc, v)):
        x = torch.where(active[:, None, None], x, torch.zeros_like(x)).double()
        ref = torch.zeros((n_groups, h_kv, d), dtype=torch.float64, device=dev).index_add_(0, group, x)
        ref /= tokens[:, None, None]
        assert bool(((got.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-6).all())


@pytest.mark.parametrize("nb,h_kv,d", [(1 << 24, 1, 32), ((1 << 20) + 3, 1, 128), ((1 << 20) + 3, 4, 128)])
def test_pooling_of_as_many_spatial_blocks_as_there_can_be(B, nb, h_kv, d):
    """2^30 tokens, the longest sequence the calls take, every 64-slot block a spatial block of its own: 2^24 of them;
    and a few more of rows of 16 and 64 chunks than there are workgroups, so that some take two in turn.
    (k and v are the same 64 GiB.)  All tokens of a block hold its number modulo 251 in every channel, which is its
    mean exactly."""
    import torch
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GiB of free GPU memory")
    _log(f"[pool] {nb} spatial blocks of one block")
    dev = torch.device("cuda")
    value = (torch.arange(nb, device=dev) % 251).to(torch.bfloat16)
    k = torch.empty((nb * 64, h_kv, d), dtype=torch.bfloat16, device=dev)
    k.view(nb, 64 * h_kv * d).copy_(value[:, None].expand(nb, 64 * h_kv * d))
    goff = torch.arange(nb + 1, dtype=torch.int32, device=dev)
    p = B.make_params(nb * 64, 0, 0, h_kv, d, 1, 64, group_offsets=goff)
    kc, vc = (torch.full((nb, h_kv, d), -1.0, dtype=torch.bfloat16, device=dev) for _ in range(2))
    B.lsrm_nsa_compress(p, k, k, kc, vc)
    torch.cuda.synchronize()
    want = value[:, None, None].expand(nb, h_kv, d)
    same = torch.equal(kc, want) and torch.equal(vc, want)
    del k, kc, vc
    torch.cuda.empty_cache()
    assert same


@pytest.mark.parametrize("d,heads,h_kv", [(64, 2, 2), (128, 1, 1), (32, 6, 2)])
def test_backward_lists_cut_into_parts_with_spatial_blocks(B, oracle_lib, d, heads, h_kv):
    """The window is the spatial block: it goes uncounted to a walk's first part, and walks are cut by their lists alone
    (every 16 tiles at this size).  Lists of 7, 8, 9, 16, 17 and 44 entries on blocks of different spatial blocks, full
    and partly filled: whole walks, two parts and more, each finished with its own group's divisor; without grouped heads and
    with three to a key/value head, a workgroup each."""
    cfg = I.small_config(name=f"g-parts-d{d}", n_obj=40 * 64, n_views=1, grid=16, heads=heads, d=d, topk=6, window=64,
                         seed=95, h_kv=h_kv)
    goff = np.concatenate([[0], np.cumsum([1, 8, 2, 3, 5, 8, 8, 5, 1, 1, 1, 1])]).astype(np.int32)
    assert goff[-1] == cfg.nb == 44
    cnt = np.full(cfg.nb, 64, dtype=np.int32)
    cnt[goff[1:] - 1] = [40, 9, 64, 33, 1, 32, 31, 50, 64, 64, 20, 64]
    cnt[11] = 17                         # (in the middle of a spatial block)
    lists = {8: 7, 0: 8, 11: 9, 18: 16, 26: 17, 30: 44}
    idx = np.full((cfg.nb, cfg.topk), -1, dtype=np.int32)
    for col, (block, rows) in enumerate(lists.items()):
        idx[(np.arange(rows) * 3 + col) % cfg.nb, col] = block
    assert all(int((idx == block).sum()) == rows for block, rows in lists.items())
    _log(f"[spatial blocks] {cfg.name}: {cfg.nb} blocks in {len(goff) - 1} spatial blocks")
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    if heads != h_kv:   # (three query heads per key/value head: see test_backward_with_spatial_blocks)
        dout_bits = I.f32_to_bf16_bits(I.bf16_bits_to_f32(dout_bits) * np.float32(0.25))
    q, k, v, dout = (I.bf16_bits_to_f32(a) for a in (q_bits, k_bits, v_bits, dout_bits))
    k_bits, v_bits, dout_bits = _poison(cfg, cnt, k_bits, v_bits, dout_bits)
    got = G.run_backward(B, cfg, q_bits, k_bits, v_bits, idx, gates, dout_bits, window_mode=1, block_count=cnt,
                         group_offsets=goff)
    kc, vc = oracle_lib.pool(k, cnt, goff), oracle_lib.pool(v, cnt, goff)
    ref = oracle_lib.nsa_backward(q, k, v, kc, vc, idx, gates, cfg.seg_offsets(), cfg.window, dout, window_mode=1,
                                  block_count=cnt, group_offsets=goff)
    active = (np.arange(cfg.n) % 64) < np.repeat(cnt, 64)
    for name, g, r in zip(("dq", "dk", "dv"), got, ref):
        assert np.isfinite(g).all() and np.all(g[~active] == 0), name
        ma, rl = G.attention_errors(g, r)
        _log(f"    {name}: max-abs {ma:.3e} rel-L2 {rl:.3e} (|ref| max {np.abs(r).max():.3e})")
        assert ma <= G.MAX_ABS_TOL and rl <= G.REL_L2_TOL, (name, ma, rl)


@pytest.mark.parametrize("d,heads,h_kv,window_mode,grouped_blocks", [(32, 12, 1, 1, True), (64, 5, 1, 0, True), (64, 10, 2, 1, False),
                                                                     (32, 7, 1, 1, True), (128, 32, 2, 1, True), (128, 6, 2, 0, False)])
def test_backward_of_few_blocks_deals_the_heads_of_a_group(B, oracle_lib, d, heads, h_kv, window_mode, grouped_blocks):
    """In the joint launch of small problems up to eight workgroups share the heads of a group, one or more each and the
    last one fewer (twelve and sixteen by twos, five and seven one each, five of ten by twos and one, three by two and one), and walks
    are cut into parts of eight, ten and sixteen tiles; windows that are a spatial block go uncut."""
    cfg = I.small_config(name=f"g-few-d{d}-h{heads}-w{window_mode}", n_obj=64 * 21, n_views=1, grid=16, heads=heads, d=d, topk=5,
                         window=160, seed=99, h_kv=h_kv)
    goff, idx, cnt = _case(cfg, 9, True, cfg.topk, min_count=8)
    idx[:, 1] = np.where(np.arange(cfg.nb) % 5 == 0, -1, 11)
    if not grouped_blocks:
        goff = None
        cnt = np.random.default_rng(10).integers(8, 65, size=cfg.nb).astype(np.int32)
    _log(f"[few blocks] {cfg.name} nb={cfg.nb}")
    q_bits, k_bits, v_bits = I.make_qkv(cfg)
    gates, dout_bits = I.make_gates(cfg), I.make_dout(cfg)
    # (a popular block and a group of heads add up gradients: keep them at the magnitude the absolute bar was set for)
    dout_bits = I.f32_to_bf16_bits(I.bf16_bits_to_f32(dout_bits) * np.float32(0.5 * h_kv / heads))
    q, k, v, dout = (I.bf16_bits_to_f32(a) for a in (q_bits, k_bits, v_bits, dout_bits))
    k_bits, v_bits, dout_bits = _poison(cfg, cnt, k_bits, v_bits, dout_bits)
    ref = oracle_lib.nsa_backward(q, k, v, oracle_lib.pool(k, cnt, goff), oracle_lib.pool(v, cnt, goff), idx, gates,
                                  cfg.seg_offsets(), cfg.window, dout, window_mode=window_mode, block_count=cnt,
                                  group_offsets=goff)
    got = G.run_backward(B, cfg, q_bits, k_bits, v_bits, idx, gates, dout_bits, window_mode=window_mode, block_count=cnt,
                         group_offsets=goff)
    inactive = (np.arange(cfg.n) % 64) >= np.repeat(cnt, 64)
    for name, g, r in zip(("dq", "dk", "dv"), got, ref):
        assert np.isfinite(g).all() and np.all(g[inactive] == 0), name
        ma, rl = G.attention_errors(g, r)
        _log(f"    {name}: max-abs {ma:.3e} rel-L2 {rl:.3e} (|ref| max {np.abs(r).max():.3e})")
        assert ma <= G.MAX_ABS_TOL and rl <= G.REL_L2_TOL, (name, ma, rl)
