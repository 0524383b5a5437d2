"""Kernel variants and dispatch edges on the GPU, each against the float64 oracle."""
import numpy as np
import pytest

import oracle as O
from harness import dev_bf16, host_f32
from workloads import BlockShape, make_rng
from workloads.gen import draw_time_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A(gpu):
    from paper_2606_15319_amd import ardit
    return ardit


def _sync():
    import torch
    torch.cuda.synchronize()


@pytest.mark.parametrize("dim,n", [(128, 1), (640, 2), (1152, 9), (2816, 3), (2816, 8)])
def test_time_mod_rows_and_stream_groups(A, dim, n):
    """Rows per wave (four from 16384 outputs: 6 x 2816 = 16896), streams in
    groups of eight, and widths that end inside a 512- or 1024-column step."""
    import torch
    tw = draw_time_weights(make_rng(400), dim)
    ts = [100.0 * i + 37.5 for i in range(n)]   # exact in fp32 (an angle is t times up to 1 rad)
    sh = BlockShape(dim=dim, n_heads=dim // 128, head_dim=128, ffn_dim=128, frames=1, lat_h=8, lat_w=8)
    mod = torch.full((n, 6, dim), float("nan"), device="cuda")
    ws = torch.empty(4 << 20, dtype=torch.uint8, device="cuda")
    A.ardit_time_mod(None, A.dims_from_shape(sh), ts,
                     A.time_weights({k: dev_bf16(v) for k, v in tw.items()}), mod, ws, ws.numel())
    _sync()
    got = host_f32(mod)
    for i, t in enumerate(ts):
        ref = O.time_modulation(t, tw, dim)
        # three chained fp32 sums of K <= 2816 terms: a sum's rounding error is a
        # random walk of about sqrt(K) 2^-24 of its RMS, 3.2e-6; three of them
        # and a factor of two for the largest of 17k values: 2e-5 of the RMS
        assert np.max(np.abs(got[i] - ref)) <= 2e-5 * np.sqrt(np.mean(ref ** 2)), (dim, n, i)


def _ctx_case(A, dim, lens, seed, in_place=False):
    import torch
    from harness import upload_block_weights
    from paper_2606_15319_amd.layout import ctx_from_device_layout
    from workloads import normal_bf16
    from workloads.gen import draw_block_weights
    sh = BlockShape(dim=dim, n_heads=dim // 128, head_dim=128, ffn_dim=128, frames=1, lat_h=8, lat_w=8)
    w = draw_block_weights(make_rng(seed), sh)
    rng = make_rng(seed + 1)
    ctx = [normal_bf16(rng, (n, dim)) for n in lens]
    dims, batch = A.dims_from_shape(sh), A.Batch(ctx_lens=lens)
    src = dev_bf16(np.concatenate(ctx))
    ck = torch.full((sum(lens) * dim,), float("nan"), dtype=torch.bfloat16, device="cuda")
    cv = src.view(-1) if in_place else torch.full_like(ck, float("nan"))
    n = A.ardit_workspace_size(dims, batch)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    A.ardit_ctx_kv(None, dims, batch, src, A.block_weights(upload_block_weights(w)), ck, cv, ws, n)
    _sync()
    kf, vf, off, out = host_f32(ck), host_f32(cv), 0, []
    for b, m in enumerate(lens):
        sl = slice(off * dim, (off + m) * dim)
        out.append((*ctx_from_device_layout(kf[sl], vf[sl], m, sh.n_heads, 128), *O.context_kv(ctx[b], w, sh.eps)))
        off += m
    return out


@pytest.mark.parametrize("dim,lens", [
    (128, [1]),             # one row, two K steps: fewer than the stages in flight
    (256, [31, 33, 1]),     # 32-row tiles with a ragged end, streams meeting inside a tile
    (384, [512, 77]),       # six K steps (the ring wraps once), the last row tile half full
    (1536, [512, 77]),      # 64-row tiles
    (1536, [700, 500]),     # the large tiles, both products in one launch, values transposed after
    (1152, [900, 700]),     # the same, each product's last column tile half full
])
def test_ctx_kv_tiles(A, dim, lens):
    from harness import parity
    for b, (k, v, kr, vr) in enumerate(_ctx_case(A, dim, lens, 410)):
        parity(k, kr, f"k {dim} {b}", quantum=kr)
        parity(v, vr, f"v {dim} {b}", quantum=vr)


def test_ctx_kv_values_over_the_text(A):
    """ctx_v in the memory of ctx: values are placed after both products have read it."""
    from harness import parity
    for b, (k, v, kr, vr) in enumerate(_ctx_case(A, 256, [97, 33], 415, in_place=True)):
        parity(k, kr, f"k {b}", quantum=kr)
        parity(v, vr, f"v {b}", quantum=vr)


@pytest.mark.parametrize("dim,heads,lat_h,lat_w", [(1024, 8, 26, 40), (256, 4, 7, 24)])
def test_block_small_products(A, dim, heads, lat_h, lat_w):
    """The residual epilogues of the small tiles: 1040 rows of 1024 (64-row tiles
    of the D x D products) and 168 rows of 256 (32-row tiles, a ragged end)."""
    import dataclasses
    from harness import BlockRun, parity
    from workloads import WORKLOADS
    sh = BlockShape(dim=dim, n_heads=heads, head_dim=dim // heads, ffn_dim=512, frames=1, lat_h=lat_h,
                    lat_w=lat_w)
    wl = dataclasses.replace(WORKLOADS["tiny"], shape=sh, cache_chunks=(1,), frame_pos0=(1,), ctx_len=40)
    run = BlockRun(wl, A, shuffle_pages_seed=3)
    run.run()
    _sync()
    ref = run.reference(0)
    parity(host_f32(run.out), ref["out"], f"block {dim}")


# 32-query workgroups with the keys split between waves: up to 256 workgroups and
# 31 key tiles (d = 64: 47); past either the items run whole or on a split schedule.
@pytest.mark.parametrize("hd,q_lens,caches", [
    (64, [1, 33], [0, 512]),            # one query, one key; 9 tiles: a wave takes two
    (128, [31, 64, 5], [448, 64, 0]),   # 8 tiles and a ragged end, lengths off every multiple
    (128, [64], [4032]),                # 64 tiles, 4 items: a split of 32 workgroups
    (128, [64], [4096]),                # 65 tiles, the same
    (128, [64, 40], [1920, 96]),        # 31 tiles: the longest taken
    (128, [64, 40], [1984, 96]),        # 32 tiles: a split
    (64, [33], [2944]),                 # 47 tiles: the longest taken
    (64, [33], [3008]),                 # 48 tiles: a split
    (64, [2048, 8], [0, 1920]),         # 260 workgroups: one workgroup per item
    (64, [700], [3840]),                # 71 tiles on 12 items: a split schedule below 256 workgroups
    (128, [203], [4192]),               # the same at d = 128, 43 keys in the last tile
])
def test_attn_few_keys(A, hd, q_lens, caches):
    from harness import parity
    from test_gpu_parity import _attn, _attn_case
    sh = BlockShape(dim=4 * hd, n_heads=4, head_dim=hd, ffn_dim=512, frames=1, lat_h=4, lat_w=8)
    pc, dims, batch, q, o, qs, ks, vs = _attn_case(A, sh, q_lens, caches, 420)
    _attn(A, dims, batch, q, pc.kv(A), o)
    _sync()
    og, off = host_f32(o), 0
    for b, n in enumerate(q_lens):
        ref = O.attention(qs[b], ks[b], vs[b]).reshape(n, -1)
        parity(og[off:off + n], ref, f"hd {hd} stream {b}", quantum=ref)
        off += n


@pytest.mark.parametrize("hd,heads,q_lens,caches,split", [
    (128, 12, [768], [64], False), (128, 12, [768], [128], False),   # 36 items of 13 and 14 tiles
    (128, 12, [768], [256], True),                      # of 16: one piece of 8 tiles a range
    (64, 16, [256] * 4, [448] * 4, False),              # 64 items of 11
    (64, 12, [768], [768], True),                       # 36 items of 24
    (128, 10, [512] * 4 + [256] * 2, [1408, 1472, 768, 128, 64, 0], False),   # 4 to 31 tiles
    (64, 10, [256, 512], [0, 2688], True),              # 4 and 50
])
def test_attn_split_where_it_ends_sooner(A, hd, heads, q_lens, caches, split):
    """Few items of few tiles run whole where the tail ranges would be several short
    pieces.  A dense call writes its workspace only if it splits."""
    import torch
    from harness import parity
    from test_gpu_parity import _attn_case
    sh = BlockShape(dim=heads * hd, n_heads=heads, head_dim=hd, ffn_dim=512, frames=1, lat_h=8, lat_w=8)
    pc, dims, batch, q, o, qs, ks, vs = _attn_case(A, sh, q_lens, caches, 424)
    n = A.ardit_workspace_size(dims, batch)
    ws = torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda")
    A.ardit_attn_fwd(None, dims, batch, q, pc.kv(A), o, ws, n)
    _sync()
    assert bool((ws != 0xA5).any()) == split
    got, off = host_f32(o).reshape(-1, heads, hd), 0
    for b, m in enumerate(q_lens):
        for h in (0, heads - 1):
            ref = O.attention(qs[b][:, h:h + 1], ks[b][:, h:h + 1], vs[b][:, h:h + 1])
            parity(got[off:off + m, h:h + 1], ref, f"stream {b} head {h}", quantum=ref)
        off += m


def test_attn_items_apart(A):
    """d = 64, 280 items of 48, 30 and 18 tiles: the longest take the whole time and the
    others fit beside them, so the launch keeps two workgroups from sharing a CU."""
    from harness import parity
    from test_gpu_parity import _attn, _attn_case
    sh = BlockShape(dim=2560, n_heads=40, head_dim=64, ffn_dim=512, frames=1, lat_h=8, lat_w=8)
    q_lens, caches = [640, 512, 512], [2432, 1408, 640]
    pc, dims, batch, q, o, qs, ks, vs = _attn_case(A, sh, q_lens, caches, 426)
    _attn(A, dims, batch, q, pc.kv(A), o)
    _sync()
    got, off = host_f32(o).reshape(-1, 40, 64), 0
    for b, m in enumerate(q_lens):
        for h in (0, 17, 39):
            ref = O.attention(qs[b][:, h:h + 1], ks[b][:, h:h + 1], vs[b][:, h:h + 1])
            parity(got[off:off + m, h:h + 1], ref, f"stream {b} head {h}", quantum=ref)
        off += m


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("lat,frames", [
    ((4, 8), 150),    # 32 keys a frame: a tile is two frames, the page window moves twice
    ((7, 8), 150),    # 56: tiles straddle frames at every offset
    ((8, 8), 150),    # 64: a frame a tile
    ((12, 16), 30),   # 192: three tiles a frame, one page window
])
def test_attn_page_walk(A, hd, lat, frames):
    """Ranges of a split schedule that start inside a stream and walk its (shuffled)
    pages, tile by tile and page by page."""
    from harness import parity
    from test_gpu_parity import _attn, _attn_case
    T = lat[0] * lat[1]
    sh = BlockShape(dim=8 * hd, n_heads=8, head_dim=hd, ffn_dim=512, frames=1, lat_h=lat[0], lat_w=lat[1])
    q_len = 1025 if frames < 100 else 300   # (over 256 workgroups of 32 queries, or over 47 tiles)
    pc, dims, batch, q, o, qs, ks, vs = _attn_case(A, sh, [q_len], [T * frames], 423)
    _attn(A, dims, batch, q, pc.kv(A), o)
    _sync()
    got = host_f32(o).reshape(q_len, 8, hd)
    for h in (0, 3, 7):
        ref = O.attention(qs[0][:, h:h + 1], ks[0][:, h:h + 1], vs[0][:, h:h + 1])
        parity(got[:, h:h + 1], ref, f"T {T} head {h}", quantum=ref)


@pytest.mark.parametrize("hd,q_len,cache,quant,finite", [
    (64, 40, 448, 0, slice(0, 64)), (128, 40, 448, 0, slice(0, 64)),        # one wave's tile
    (64, 700, 3840, 0, slice(0, 64)), (128, 700, 3840, 0, slice(0, 64)),    # one piece's tile
    (64, 40, 448, 0, slice(256, 320)), (128, 700, 3840, 0, slice(3900, 4000)),
    (128, 40, 448, 1, slice(0, 64)), (128, 40, 448, 1, slice(64, None)),    # the first tile, or all others
    (128, 300, 640, 1, slice(500, 600)),
])
def test_attn_overflowed_scores(A, hd, q_len, cache, quant, finite):
    """Scores of every key outside `finite` overflow to -inf: the waves (40 queries),
    the pieces of a split (700) and the tiles before the first finite score weigh nothing."""
    from harness import fp8_parity, parity
    from oracle import fp8_ref
    from test_gpu_parity import _attn, _attn_case
    sh = BlockShape(dim=4 * hd, n_heads=4, head_dim=hd, ffn_dim=512, frames=1, lat_h=4, lat_w=8)
    pc, dims, _, _, o, qs, ks, vs = _attn_case(A, sh, [q_len], [cache], 425)
    q = host_f32(dev_bf16(np.abs(qs[0]) + 0.5))
    k = np.full_like(ks[0], -np.float32(2.0 ** 127))
    k[finite] = ks[0][finite]
    pc.fill_stream(0, k, vs[0])
    pc.upload()
    _attn(A, dims, A.Batch([q_len], [cache], quant=[quant]), dev_bf16(q.reshape(q_len, -1)), pc.kv(A), o)
    _sync()
    got = host_f32(o).reshape(q_len, 4, hd)
    if quant:
        ref, _, sigma = fp8_ref.fp8_attention(q, k, vs[0], sigma=True)
        fp8_parity(got, ref, sigma, f"fp8 q {q_len}")
    else:
        ref = O.attention(q, k, vs[0])
        parity(got, ref, f"hd {hd} q {q_len}", quantum=ref)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("ctx", [1, 37, 200])
def test_block_few_text_keys(A, hd, ctx):
    """Text attention of a small block: lengths that are no multiple of 8 read
    their values one by one."""
    import dataclasses
    from harness import BlockRun, parity
    from workloads import WORKLOADS
    sh = BlockShape(dim=256, n_heads=256 // hd, head_dim=hd, ffn_dim=256, frames=1, lat_h=8, lat_w=9)
    wl = dataclasses.replace(WORKLOADS["tiny"], shape=sh, cache_chunks=(1,), frame_pos0=(1,), ctx_len=ctx)
    run = BlockRun(wl, A, shuffle_pages_seed=4)
    run.run()
    _sync()
    ref = run.reference(0)
    parity(host_f32(run.out), ref["out"], f"block hd {hd} ctx {ctx}")


@pytest.mark.parametrize("ctx", [1, 64, 100, 192, 264, 448])
def test_block_text_tiles(A, ctx):
    """Text attention on 256-query items over 1 to 7 key tiles: fewer than the
    tiles in flight, whole and partial ends, and a length (100) whose values are
    not 16-byte aligned."""
    import dataclasses
    from harness import BlockRun, parity
    from workloads import WORKLOADS
    sh = BlockShape(dim=1024, n_heads=8, head_dim=128, ffn_dim=256, frames=1, lat_h=26, lat_w=40)
    wl = dataclasses.replace(WORKLOADS["tiny"], shape=sh, cache_chunks=(0,), frame_pos0=(0,), ctx_len=ctx)
    run = BlockRun(wl, A, shuffle_pages_seed=3)
    run.run()
    _sync()
    ref = run.reference(0)
    parity(host_f32(run.out), ref["out"], f"ctx {ctx}")


@pytest.mark.parametrize("quant", [0, 1])
@pytest.mark.parametrize("keys", [64, 100, 128, 192, 250, 320, 384])
def test_attn_sparse_few_tiles(A, quant, keys):
    """Lists of 1 to 6 tiles (fewer than the pairs in flight), the last one whole
    or partial, on the bf16 and FP8 kernels: every tile kept but one."""
    import oracle.sparse_ref as SR
    from harness import fp8_parity, parity
    from oracle import fp8_ref
    from test_gpu_parity import _attn, _attn_case
    T = 32
    sh = BlockShape(dim=256, n_heads=2, head_dim=128, ffn_dim=256, frames=1, lat_h=4, lat_w=8)
    cache = (keys - 1) // T * T
    q_len = keys - cache
    pc, dims, batch, q, o, qs, ks, vs = _attn_case(A, sh, [q_len], [cache], 430)
    n = -(-keys // 64)
    rho = 1.0 / n if n > 1 else 0.25
    _attn(A, dims, A.Batch([q_len], [cache], sparsity=[rho], quant=[quant]), q, pc.kv(A), o)
    _sync()
    lists = SR.select_blocks(SR.block_scores(qs[0], ks[0]), SR.keep_count(n, rho))
    got = host_f32(o).reshape(q_len, 2, 128)
    if quant:
        mask = np.stack([SR.block_mask(lists[h], q_len, keys) for h in range(2)])
        ref, _, sigma = fp8_ref.fp8_attention(qs[0], ks[0], vs[0], mask=mask, sigma=True)
        fp8_parity(got, ref, sigma, f"fp8 {keys}")
    else:
        ref = SR.sparse_attention(qs[0], ks[0], vs[0], lists)
        parity(got, ref, f"keys {keys}", quantum=ref)


@pytest.mark.parametrize("tiles", [256, 257, 512, 513, 1024, 1025])
def test_sparse_select_key_registers(A, tiles):
    """The selection holds a stream's scores in 4, 8 or 16 registers a lane, or in LDS,
    by the longest stream: both sides of each line, beside a short stream."""
    from test_gpu_parity import _attn_case, _check_selection, _sparse_rows
    import oracle.sparse_ref as SR
    sh = BlockShape(dim=128, n_heads=2, head_dim=64, ffn_dim=128, frames=1, lat_h=8, lat_w=8)
    q_lens, caches, rho = [40, 70], [64 * (tiles - 1), 640], [0.9, 0.6]
    pc, dims, _, q, o, qs, ks, vs = _attn_case(A, sh, q_lens, caches, 431)
    batch = A.Batch(q_lens, caches, sparsity=rho)
    rows = _sparse_rows(A, dims, batch, q, pc.kv(A), row_stride=SR.keep_count(tiles, rho[0]))
    _sync()
    for b in range(2):
        _check_selection(rows[2 * b:2 * b + 2], qs[b], ks[b], rho[b], 2, f"{tiles} tiles stream {b}")


@pytest.mark.parametrize("hd,quant", [(64, 0), (128, 0), (128, 1)])
def test_attn_sparse_long_lists(A, hd, quant):
    """Lists of 155 tiles: the kernels hold 64 entries at a time and refill twice."""
    import oracle.sparse_ref as SR
    from harness import fp8_parity, parity
    from oracle import fp8_ref
    from test_gpu_parity import _attn, _attn_case
    sh = BlockShape(dim=2 * hd, n_heads=2, head_dim=hd, ffn_dim=256, frames=1, lat_h=8, lat_w=12)
    q_len, cache, rho = 41, 16416, 0.4
    n, keys = 258, q_len + cache
    pc, dims, _, q, o, qs, ks, vs = _attn_case(A, sh, [q_len], [cache], 432)
    _attn(A, dims, A.Batch([q_len], [cache], sparsity=[rho], quant=[quant]), q, pc.kv(A), o)
    _sync()
    keep = SR.keep_count(n, rho)
    assert -(-keys // 64) == n and keep == 155
    lists = SR.select_blocks(SR.block_scores(qs[0], ks[0]), keep)
    got = host_f32(o).reshape(q_len, 2, hd)
    if quant:
        mask = np.stack([SR.block_mask(lists[h], q_len, keys) for h in range(2)])
        ref, _, sigma = fp8_ref.fp8_attention(qs[0], ks[0], vs[0], mask=mask, sigma=True)
        fp8_parity(got, ref, sigma, "fp8")
    else:
        ref = SR.sparse_attention(qs[0], ks[0], vs[0], lists)
        parity(got, ref, f"hd {hd}", quantum=ref)


@pytest.mark.parametrize("q_lens,caches", [
    ([3328, 3328], [0, 0]),     # 52 tiles each: the last four of 260 items, in the second stream
    ([2300, 2304, 2290, 2304], [384] * 4),   # 42 tiles: the last 104 of 360, from the middle of one stream on
    ([2500, 4096], [0, 0]),     # 40 and 64 tiles: no split
    ([3072, 3500], [0, 0]),     # 48 and 55
])
def test_attn_full_rounds_and_split_rest(A, q_lens, caches):
    """More items (of 10 heads) than a round holds: with equal tiles the full rounds run
    whole and the rest is split; streams of different length run one workgroup per item."""
    from harness import parity
    from test_gpu_parity import _attn, _attn_case
    sh = BlockShape(dim=640, n_heads=10, head_dim=64, ffn_dim=512, frames=1, lat_h=8, lat_w=8)
    pc, dims, batch, q, o, qs, ks, vs = _attn_case(A, sh, q_lens, caches, 440)
    _attn(A, dims, batch, q, pc.kv(A), o)
    _sync()
    og, off = host_f32(o), 0
    for b, n in enumerate(q_lens):
        got = og[off:off + n].reshape(n, 10, 64)
        for h in (0, 5, 9):
            ref = O.attention(qs[b][:, h:h + 1], ks[b][:, h:h + 1], vs[b][:, h:h + 1])
            parity(got[:, h:h + 1], ref, f"stream {b} head {h}", quantum=ref)
        off += n
