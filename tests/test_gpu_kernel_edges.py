"""GPU parity of kernels at the sizes where their tiling, splitting or dispatch changes."""
import numpy as np
import pytest

from oracle import litevggt_oracle as O
from paper_2512_04939_amd import synth

from helpers import hip_params, oracle_params, stored_inputs, to_dev_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2512_04939_amd import binding
    binding.lib()
    return binding


def _i32(t):
    return t.cpu().numpy().astype(np.int64)


# ------------------------------------------------------------------------------- partition
# a wave's 64-token steps that end on, before and behind a frame's end; one wave and all sixteen;
# the largest grid; score maps without ties, with many, and all equal (the threshold's ties go by
# token number), with infinities and values that differ in their last bit only
@pytest.mark.parametrize("h,w,special,ratio", [(8, 8, 0, 0.5), (9, 11, 5, 0.75), (16, 16, 5, 0.9), (32, 31, 32, -1.0),
                                               (37, 37, 5, 0.9), (31, 33, 1, 0.25), (75, 80, 5, 0.6), (1, 7, 3, 0.5)])
@pytest.mark.parametrize("kind", ["plain", "ties", "equal", "extremes"])
def test_select_edges(B, h, w, special, ratio, kind):
    import torch
    wl = synth.Workload("t", frames=3, grid_h=h, grid_w=w, dim=64, heads=1, n_special=special, merge_ratio=ratio)
    rng = np.random.default_rng(h * w + special)
    score = rng.random((3, h * w)).astype(np.float32)
    if kind == "ties":
        score = (np.floor(score * 7) / 7).astype(np.float32)
    elif kind == "equal":
        score[:] = np.float32(0.25)
    elif kind == "extremes":
        score = (np.float32(1.0) + np.float32(2.0 ** -23) * np.floor(score * 5)).astype(np.float32)
        score[:, ::3] *= -1.0
        score[1, ::5], score[2, ::4] = np.inf, -np.inf
    po, ph = oracle_params(wl), hip_params(wl)
    ref = O.select_anchors(score, po)
    pl = B.litevggt_plan(ph)
    ib = B.alloc_index(pl)
    B.litevggt_select_anchors(ph, torch.from_numpy(score).cuda(), ib)
    torch.cuda.synchronize()
    assert np.array_equal(ib.role.cpu().numpy(), ref["role"])
    for got, want in ((ib.kept_idx, "kept_idx"), (ib.dst_idx, "dst_idx"), (ib.src_idx, "src_idx")):
        assert np.array_equal(_i32(got)[:len(ref[want])], ref[want])
    kept = ref["kept_idx"].astype(np.int64)
    assert np.array_equal(_i32(ib.anchor_of)[kept], kept)
    assert np.array_equal(_i32(ib.slot_of)[kept], np.arange(len(kept)))


# 8 waves per frame: up to 512 patches, and one more; more than 512 frames, up to 2048 patches and one row
# more; the last GA token's ties decided in the last digit
@pytest.mark.parametrize("frames,h,w", [(3, 16, 32), (3, 19, 27), (512, 8, 65), (513, 8, 65), (513, 32, 64), (513, 33, 64)])
def test_select_waves_per_frame(B, frames, h, w):
    import torch
    wl = synth.Workload("t", frames=frames, grid_h=h, grid_w=w, dim=64, heads=1, n_special=5, merge_ratio=0.75)
    rng = np.random.default_rng(frames + h)
    score = (np.float32(1.0) + np.float32(2.0 ** -23) * rng.integers(0, h * w, (frames, h * w))).astype(np.float32)
    ref = O.select_anchors(score, oracle_params(wl))
    ph = hip_params(wl)
    ib = B.alloc_index(B.litevggt_plan(ph))
    B.litevggt_select_anchors(ph, torch.from_numpy(score).cuda(), ib)
    torch.cuda.synchronize()
    assert np.array_equal(ib.role.cpu().numpy(), ref["role"])
    for got, want in ((ib.kept_idx, "kept_idx"), (ib.dst_idx, "dst_idx"), (ib.src_idx, "src_idx")):
        assert np.array_equal(_i32(got)[:len(ref[want])], ref[want])


# ------------------------------------------------------------------------------- matching
def _check_index(B, ph, x, near=1e-6):
    """Matching of bf16 rows x against every dst row in float64, and the groups it implies."""
    import torch
    pl = B.litevggt_plan(ph)
    ib = B.alloc_index(pl)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    score = torch.rand(ph.frames, ph.grid_h * ph.grid_w, generator=g, device="cuda")
    best = torch.empty(max(pl.n_src, 1), device="cuda")
    B.litevggt_select_anchors(ph, score, ib)
    B.litevggt_match(ph, x, ib, best, B.alloc_ws(pl.ws_bytes))
    torch.cuda.synchronize()
    xn = x.double()
    xn = xn / xn.norm(dim=1, keepdim=True).clamp_min(1e-12)
    src, dst = ib.src_idx[:pl.n_src].long(), ib.dst_idx[:pl.n_dst].long()
    dn = xn[dst].t().contiguous()
    for i in range(0, pl.n_src, 8192):
        sim = xn[src[i:i + 8192]] @ dn
        top, at = sim.topk(2, dim=1)
        got = ib.anchor_of[src[i:i + 8192]].long()
        wrong = got != dst[at[:, 0]]
        assert bool(((top[:, 0] - top[:, 1])[wrong] < near).all())
        pos = torch.searchsorted(dst, got)
        assert torch.equal(dst[pos], got)
        assert float((top[:, 0] - sim.gather(1, pos[:, None])[:, 0]).max()) < near
        assert float((best[i:i + 8192].double() - top[:, 0]).abs().max()) < 2e-5
    # groups: members ascending inside every slot, slots in the order of the kept tokens
    slot = ib.slot_of.long()
    kept = ib.kept_idx.long()
    assert torch.equal(kept[slot], ib.anchor_of.long())
    order = torch.sort(slot, stable=True)[1]
    assert torch.equal(ib.group_mem.long(), order)
    off = torch.zeros(pl.M + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(torch.bincount(slot, minlength=pl.M), 0)
    assert torch.equal(ib.group_off.long(), off)


# src x dst tiles of 256 rows: 1 x 2 and 1 x 30 (one src tile, a sweep per dst tile), 12 x 3 (no full
# round), 83 x 8 (the same with ragged sweeps), 252 x 20 (three full rounds of 8 x 4 teams, a rest of
# 60), 143 x 57 (a full round of 16 x 2 teams, a rest of 15 tiles by 17 sweeps)
@pytest.mark.parametrize("frames,h,w,ratio,dim", [(2, 16, 16, 0.5, 64), (2, 77, 77, 0.01, 64), (9, 20, 20, 0.9, 192),
                                                  (60, 20, 20, 0.9, 64), (180, 20, 20, 0.9, 128), (141, 20, 20, -1.0, 64)])
def test_match_schedules(B, frames, h, w, ratio, dim):
    import torch
    ph = B.make_params(frames, h, w, dim, dim // 64, merge_ratio=ratio)
    pl = B.litevggt_plan(ph)
    g = torch.Generator(device="cuda")
    g.manual_seed(frames)
    x = torch.randn(pl.N, ph.dim, generator=g, device="cuda").to(torch.bfloat16)
    _check_index(B, ph, x)


def test_match_near_equal_rows_of_many_sweeps(B):
    """Every dst row appears in several dst tiles (exact copies): float64 ties over sweeps go to
    the lowest token number."""
    import torch
    ph = B.make_params(40, 16, 16, 128, 2, merge_ratio=0.5)
    pl = B.litevggt_plan(ph)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    frame = torch.randn(pl.N // 40, 128, generator=g, device="cuda").to(torch.bfloat16)
    x = frame.repeat(40, 1).contiguous()
    ib = B.alloc_index(pl)
    score = torch.rand(1, 256, generator=g, device="cuda").repeat(40, 1).contiguous()
    B.litevggt_select_anchors(ph, score, ib)
    B.litevggt_match(ph, x, ib, None, B.alloc_ws(pl.ws_bytes))
    torch.cuda.synchronize()
    src = ib.src_idx[:pl.n_src].long()
    # frame 0 is all dst, so every src token has its exact copy there, and no dst precedes it
    assert torch.equal(ib.anchor_of[src].long(), src % (pl.N // 40))


def _near_equal_families(rng, count, dim):
    """(row, [best, second, third]): bf16 rows whose cosines with `row` are exactly 1 and, for the other
    two, one or two fp32 steps below it in float64, while fp32 products with fp32 inverse norms rank the
    best one last or level with the others.  (Small integers times an odd factor: every product sum is exact in fp32, so the fp32
    values follow from the rounding of the inverse norm alone.)"""
    f32, out = np.float32, []
    while len(out) < count:
        row = rng.integers(-31, 32, dim).astype(np.float64)
        n2 = float((row * row).sum())
        va, k = min((f32(f * n2) * f32(1 / np.sqrt(f * f * n2)), f) for f in (1, 3, 5, 7))
        others = []
        for i in np.flatnonzero(np.abs(row) >= 16):
            d = row.copy()
            d[i] += np.sign(d[i]) / 8
            dot, d2 = float((row * d).sum()), float((d * d).sum())
            if f32(dot) * f32(1 / np.sqrt(d2)) >= va and f32(dot / np.sqrt(d2) / np.sqrt(n2)) < f32(1):
                others.append(d)
        if len(others) >= 2:
            out.append((row, [k * row, others[0], others[1]]))
    return out


# one, two and three sweeps per src tile: lists of a quarter, of a half, of a half of the dst rows
@pytest.mark.parametrize("frames,h,w,ratio", [(230, 16, 16, 0.98), (80, 20, 20, 0.9), (60, 20, 20, 0.9)])
def test_match_lists_keep_their_own_candidates(B, frames, h, w, ratio):
    """Two near-equal rows in the first quarter of the first dst tile, the best one in the last quarter of
    a later tile of the same sweep: float64 decides among all three, whatever fp32 made of them."""
    import torch
    ph = B.make_params(frames, h, w, 256, 4, merge_ratio=ratio)
    pl = B.litevggt_plan(ph)
    g = torch.Generator(device="cuda")
    g.manual_seed(frames)
    x = torch.randn(pl.N, 256, generator=g, device="cuda").to(torch.bfloat16)
    ib = B.alloc_index(pl)
    score = torch.rand(frames, h * w, generator=g, device="cuda")
    B.litevggt_select_anchors(ph, score, ib)
    torch.cuda.synchronize()
    src, dst = _i32(ib.src_idx)[:pl.n_src], _i32(ib.dst_idx)[:pl.n_dst]
    rng = np.random.default_rng(frames)
    rows = rng.choice(pl.n_src, 30, replace=False)
    want = []
    for n, (p, (row, cand)) in enumerate(zip(rows, _near_equal_families(rng, 30, 256))):
        at = [dst[256 * (1 + n % 3) + 192 + n], dst[2 * n], dst[2 * n + 1]]
        for t, v in zip([src[p]] + at, [row] + cand):
            b = torch.from_numpy(v).cuda()
            x[t] = b.to(torch.bfloat16)
            assert torch.equal(x[t].double(), b)
        want.append(at[0])
    B.litevggt_match(ph, x, ib, None, B.alloc_ws(pl.ws_bytes))
    torch.cuda.synchronize()
    assert np.array_equal(_i32(ib.anchor_of)[src[rows]], np.array(want))


# groups: the largest sequence one workgroup sorts, the smallest beyond it, one digit pass, a chunk of the general
# sort that ends on a wave's last element, and one slot count above 16 bits (three digit passes); two
# passes in three launches: whole chunks of kept tokens only, large groups of few slots, 16,384 counters and a chunk
# more, the most counters that are summed in the move (65,536) and one chunk more
@pytest.mark.parametrize("frames,h,w,special,ratio", [(20, 15, 17, 1, 0.9), (3, 42, 40, 27, 0.5), (50, 8, 16, 0, 0.99),
                                                      (64, 15, 17, 1, 0.9), (5, 52, 63, 1, 0.5), (2, 1, 1, 0, 0.0),
                                                      (17, 32, 32, 0, 0.75), (70, 32, 32, 2, 0.0),
                                                      (17, 32, 32, 0, 0.0), (40, 20, 21, 0, 0.98), (64, 32, 32, 0, 0.5),
                                                      (65, 32, 32, 0, 0.5), (32, 37, 37, 5, 0.9), (256, 32, 32, 0, 0.8),
                                                      (257, 32, 32, 0, 0.8)])
def test_groups_edges(B, frames, h, w, special, ratio):
    import torch
    ph = B.make_params(frames, h, w, 64, 1, n_special=special, merge_ratio=ratio)
    pl = B.litevggt_plan(ph)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = torch.randn(pl.N, 64, generator=g, device="cuda").to(torch.bfloat16)
    _check_index(B, ph, x)


# ------------------------------------------------------------------------------- linear layers
def _block64(z, t, heads, seen=None):
    """The transformer block in float64, rounded to bf16 where the block stores its intermediates; `seen`
    receives the largest |input| of each linear layer."""
    import torch
    r = lambda a: a.to(torch.bfloat16).double()  # noqa: E731

    def lin(a, w, b):
        return a @ t[w].double().t().contiguous() + t[b].double()

    def ln(a, g, b):
        d = a - a.mean(1, keepdim=True)
        return r(d / torch.sqrt((d * d).mean(1, keepdim=True) + 1e-6) * t[g].double() + t[b].double())

    z, c = z.double(), z.shape[1]
    h1 = ln(z, "ln1_g", "ln1_b")
    qkv = r(lin(h1, "w_qkv", "b_qkv"))
    a = torch.empty_like(z)
    for h in range(heads):
        q, k, v = (qkv[:, i * c + h * 64:i * c + h * 64 + 64] for i in range(3))
        q, k = (r(x / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-6)) for x in (q, k))
        for i in range(0, len(z), 4096):
            a[i:i + 4096, h * 64:h * 64 + 64] = torch.softmax(q[i:i + 4096] @ k.t().contiguous() * 0.125, 1) @ v
    u1 = r(lin(r(a), "w_o", "b_o"))
    h2 = ln(z + u1, "ln2_g", "ln2_b")
    hid = lin(h2, "w_1", "b_1")
    hid = r(0.5 * hid * (1.0 + torch.erf(hid / 2.0 ** 0.5)))
    if seen is not None:
        seen += [float(x.abs().max()) for x in (h1, r(a), h2, hid)]
    return u1 + r(lin(hid, "w_2", "b_2"))


# rows of one tile, around the two tile heights, row tiles by XCD or in plain order (2200 rows at 1024
# channels: both), every tile shape and mixes of them (5776, 9000; the largest tile with its output in
# operand order: test_block_largest_tiles), more tiles than workgroups (33000 at 256), a column count that
# is no multiple of 4 tiles; two K groups: 64 x 64 tiles of one row, whole ones and one row more, the most of
# them in one launch (2048 rows at 256: the first MLP layer) and one row more, 128 x 128 tiles from the fewest rows on
# (4097 at 512: the second MLP layer) to the most (8192) and one row more
@pytest.mark.parametrize("m,dim", [(1, 256), (127, 256), (129, 256), (257, 768), (640, 1024), (2200, 1024), (5776, 1024),
                                   (9000, 1024), (17000, 256), (33000, 256), (63, 256), (64, 512), (65, 256), (2048, 256),
                                   (2049, 256), (4097, 512), (8192, 512), (8193, 512)])
@pytest.mark.parametrize("linear", ["bf16", "fp8", "fp8-delayed"])
def test_block_tile_shapes(B, m, dim, linear):
    import torch
    w = synth.block_weights(dim, seed=m)
    t = {k: torch.from_numpy(v).cuda() for k, v in w.items()}
    t = {k: v.to(torch.bfloat16) if k.startswith("w_") else v for k, v in t.items()}
    g = torch.Generator(device="cuda")
    g.manual_seed(m)
    z = torch.randn(m, dim, generator=g, device="cuda").to(torch.bfloat16)
    state = torch.zeros(B.FP8_STATE_BYTES, dtype=torch.uint8, device="cuda")
    bw = B.block_weights(t) if linear == "bf16" else B.block_weights(
        t, B.LINEAR_FP8_E4M3, B.FP8_CURRENT if linear == "fp8" else B.FP8_DELAYED, state)
    ph = B.make_params(1, 1, 1, dim, dim // 64, n_special=0, qk_norm=1)
    delta = torch.full_like(z, float("nan"))
    ws = B.alloc_ws(B.litevggt_global_block_ws_bytes(ph, m))
    for _ in range(2 if linear == "fp8-delayed" else 1):     # the second call scales by the first one's amaxes
        B.litevggt_global_block(ph, m, z, bw, delta, ws)
    torch.cuda.synchronize()
    ref = _block64(z, t, dim // 64)
    err = float((delta.double() - ref).abs().max() / ref.abs().max())
    # bf16: one rounding step of an intermediate apart; E4M3 layers: 2^-4 per code, four layers deep
    assert err <= (2e-2 if linear == "bf16" else 1e-1)


# the LayerNorms' rows in LDS, 40 to 132 KB of 32: the fewer channels of one kernel before the most of the same one, whose
# limit of dynamic LDS is raised once per device
@pytest.mark.parametrize("fewer,most", [(1280, 1536), (1792, 2048)])
@pytest.mark.parametrize("linear", ["bf16", "fp8-delayed"])
def test_block_of_more_channels_after_fewer(B, fewer, most, linear):
    for dim in (fewer, most):
        test_block_tile_shapes(B, 100, dim, linear)


@pytest.mark.parametrize("dim", [512, 768, 1024])
def test_block_layernorm_cancels_opposite_lanes_first(B, dim):
    """Two channels 32 lanes apart hold +-2^30: added to each other first they vanish and the mean of the
    rest is kept; in any order that adds something else in between, it is lost to rounding."""
    import torch
    big = 2.0 ** 30
    g = torch.Generator(device="cuda")
    g.manual_seed(dim)
    z = (1.0 + 0.1 * torch.randn(1, dim, generator=g, device="cuda")).to(torch.bfloat16)
    z.view(dim // 8, 8)[torch.arange(0, dim // 8, 32, device="cuda")] = 0.0     # what lanes 0 and 32 hold
    z[0, 0], z[0, 256] = big, -big
    t = {k: torch.zeros(v.shape, device="cuda") for k, v in synth.block_weights(dim, seed=0).items()}
    t["ln1_g"] += big
    t["ln1_g"][[0, 256]] = 0.0
    t["w_qkv"][2 * dim:] = torch.eye(dim, device="cuda")    # q = k = 0 and v = LN(z): one token attends to itself
    t["w_o"][:] = torch.eye(dim, device="cuda")
    t = {k: v.to(torch.bfloat16) if k.startswith("w_") else v for k, v in t.items()}
    ph = B.make_params(1, 1, 1, dim, dim // 64, n_special=0, qk_norm=1)
    delta = torch.full_like(z, float("nan"))
    B.litevggt_global_block(ph, 1, z, B.block_weights(t), delta, B.alloc_ws(B.litevggt_global_block_ws_bytes(ph, 1)))
    torch.cuda.synchronize()
    d = z.double() - z.double().mean()
    ref = d / torch.sqrt((d * d).mean() + 1e-6) * t["ln1_g"].double()
    # one bf16 rounding of a value that went through identity layers
    assert bool(((delta.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4).all())


# the first MLP layer on 256 x 256 tiles with its output in operand order, more tiles than CUs (8 x 61, 12 x 35)
# and a ragged last row tile; tiles of four stages, the ring's fewest, that follow each other (98 x 4)
@pytest.mark.parametrize("m,dim", [(15400, 512), (8900, 768), (25001, 256)])
@pytest.mark.parametrize("linear", ["bf16", "fp8-delayed"])
@pytest.mark.parametrize("attn", ["bf16", "fp8"])
def test_block_largest_tiles(B, m, dim, linear, attn):
    import torch
    t = {k: torch.from_numpy(v).cuda() for k, v in synth.block_weights(dim, seed=m).items()}
    t = {k: v.to(torch.bfloat16) if k.startswith("w_") else v for k, v in t.items()}
    g = torch.Generator(device="cuda")
    g.manual_seed(m)
    z = torch.randn(m, dim, generator=g, device="cuda").to(torch.bfloat16)
    state = torch.zeros(B.FP8_STATE_BYTES, dtype=torch.uint8, device="cuda")
    bw = B.block_weights(t) if linear == "bf16" else B.block_weights(t, B.LINEAR_FP8_E4M3, B.FP8_DELAYED, state)
    ph = B.make_params(1, 1, 1, dim, dim // 64, n_special=0, qk_norm=1, attn_dtype=B.ATTN_FP8_E4M3 if attn == "fp8" else B.ATTN_BF16)
    delta = torch.full_like(z, float("nan"))
    ws = B.alloc_ws(B.litevggt_global_block_ws_bytes(ph, m))
    for _ in range(1 if linear == "bf16" else 2):            # the second call scales by the first one's amaxes
        B.litevggt_global_block(ph, m, z, bw, delta, ws)
    torch.cuda.synchronize()
    seen = []
    ref = _block64(z, t, dim // 64, seen)
    err = float((delta.double() - ref).abs().max() / ref.abs().max())
    assert err <= (2e-2 if linear == attn == "bf16" else 1e-1)   # as in test_block_tile_shapes; E4M3 attention as E4M3 layers
    if linear != "bf16":    # recorded amaxes of the four layers' inputs: LayerNorm of z to a bf16 step, the others behind E4M3 layers
        amax = state.view(torch.float32).reshape(4, -1)[:, 1].tolist()
        assert abs(amax[0] / seen[0] - 1) <= 2.0 ** -8
        assert all(abs(a / s - 1) <= 0.1 for a, s in zip(amax[1:], seen[1:])), (amax, seen)


def _exact_qkv_block(n, dim, seed, far=None):
    """A block's tokens and weights whose q, k and v are exact in every type, and those three; its output is its attention's, as
    the output projection takes it.  Rows of +-1, so LN(z) = z; q and k are selections of it in powers of two that differ from
    head to head, v sums of eight entries.  Keys share 48 of 64 channels.  With `far`, all heads are alike; queries agree with
    the keys in half of these 48, and the rows `far` in none, 8.6 binades below."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    heads = dim // 64
    z = torch.randint(0, 2, (n, dim), generator=g, device="cuda") * 2.0 - 1.0
    z[:, 64:112] = z[0, 64:112].clone()                            # keys: channels 64 .. 127; queries: 0 .. 63
    if far is not None:
        z[:, 0:48] = z[0, 64:112] * (1.0 - 2.0 * (torch.rand(n, 48, generator=g, device="cuda").argsort(1).argsort(1) < 24))
        z[far, 0:48] = -z[0, 64:112]
    ones = (dim - 128 - z[:, :128].sum(1)) / 2                     # mean 0
    rank = torch.rand(n, dim - 128, generator=g, device="cuda").argsort(1).argsort(1)
    z[:, 128:] = (rank < ones[:, None]) * 2.0 - 1.0
    assert bool((z.sum(1) == 0).all())
    t = {k: torch.zeros(v.shape, device="cuda") for k, v in synth.block_weights(dim, seed=0).items()}
    t["ln1_g"] += 1.0
    t["ln2_g"] += 1.0
    i = torch.arange(64, device="cuda")
    for h in range(heads):
        gain_q, gain_k = (torch.ones(64, device="cuda"),) * 2 if far is not None else (
            2.0 ** -(i % 3 + (heads - 1 - h) % 4).float(), 2.0 ** -((i + h) % 3 + h % 4).float())
        t["w_qkv"][h * 64 + i, i] = gain_q
        t["w_qkv"][dim + h * 64 + i, 64 + i] = gain_k
    at = torch.rand(dim, dim, generator=g, device="cuda").argsort(1)[:, :8]
    t["w_qkv"][2 * dim:].scatter_(1, at, 2.0 ** -torch.randint(0, 3, (dim, 8), generator=g, device="cuda").float())
    t["w_o"][:] = torch.eye(dim, device="cuda")
    t = {k: v.to(torch.bfloat16) if k.startswith("w_") else v for k, v in t.items()}
    qkv = (z.double() @ t["w_qkv"].double().t().contiguous()).to(torch.bfloat16)
    return z.to(torch.bfloat16), t, [qkv[:, i * dim:i * dim + dim].contiguous() for i in range(3)]


def _through_e4m3(o, inv):
    """Rows through an identity layer with E4M3 operands (weight: code 448), their scale inv."""
    import torch
    f = lambda x: torch.tensor(x, dtype=torch.float32, device="cuda")  # noqa: E731
    codes = (o.float() * f(inv)).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).float()
    return (codes * 448.0 * ((f(1.0) / f(inv)) * (f(1.0) / f(448.0)))).to(torch.bfloat16)


def _f32(x):
    return float(np.float32(x))


# blocks around E4M3 attention, and bf16 attention: q, k and v from every tile shape of their layer (64 x 64 in two K groups: one
# row, one row more than a tile; 128 x 128 in two K groups with bf16 layers; 128 x 128; 128 x 256; 256 x 256), ragged ends,
# among them ones whose last 512 queries reach beyond the next layer's operand; normalised and as given, the attention's
# output as rows, as bf16 and as E4M3 operand: the attention entry point's bits, rounded as the output layer rounds its input
@pytest.mark.parametrize("n,dim", [(1, 256), (65, 256), (300, 512), (700, 256), (400, 2048), (2200, 1024), (5200, 512),
                                   (5601, 512), (12001, 256)])
@pytest.mark.parametrize("linear", ["bf16", "fp8", "fp8-delayed"])
@pytest.mark.parametrize("attn", ["fp8", "bf16"])
@pytest.mark.parametrize("norm", [1, 0])
def test_block_is_its_attention_between_identity_layers(B, n, dim, linear, attn, norm):
    import torch
    z, t, (q, k, v) = _exact_qkv_block(n, dim, n)
    ph = B.make_params(1, 1, 1, dim, dim // 64, n_special=0, attn_dtype=B.ATTN_FP8_E4M3 if attn == "fp8" else B.ATTN_BF16, qk_norm=norm)
    o = torch.full_like(q, float("nan"))
    B.litevggt_global_attn(ph, n, q, k, v, o, B.alloc_ws(B.litevggt_attn_ws_bytes(ph, n)))
    top = float(o.abs().max())
    state = torch.zeros(B.FP8_STATE_BYTES, dtype=torch.uint8, device="cuda")
    bw = B.block_weights(t) if linear == "bf16" else B.block_weights(
        t, B.LINEAR_FP8_E4M3, B.FP8_CURRENT if linear == "fp8" else B.FP8_DELAYED, state)
    ws = B.alloc_ws(B.litevggt_global_block_ws_bytes(ph, n))
    ws.fill_(0x7f)
    for call in range(2):                                          # (delayed: scale 1, then by the first call's amax)
        delta = torch.full_like(z, float("nan"))
        B.litevggt_global_block(ph, n, z, bw, delta, ws)
        torch.cuda.synchronize()
        scale = 1.0 if linear == "fp8-delayed" and call == 0 else _f32(np.float32(448.0) / np.float32(top))
        assert torch.equal(delta, o if linear == "bf16" else _through_e4m3(o, scale)), call
    if linear == "fp8-delayed":
        amax = state.view(torch.float32).reshape(4, -1)[:, :2].tolist()
        assert amax[0] == [1.0, 1.0] and amax[1] == [top, top]


# E4M3 attention whose blocks' first pass is not enough for some query: the second pass rewrites the output layer's operand, and
# the amax that goes into the history is that of the rows that it leaves, and of other blocks' first pass.  One block of 512 queries,
# flagged in its first half, in its ragged second one, and none of it; a flagged one among others
@pytest.mark.parametrize("n,far", [(200, [10]), (512, [511]), (230, []), (1300, [600, 700])])
@pytest.mark.parametrize("linear", ["bf16", "fp8", "fp8-delayed"])
def test_block_attention_left_to_the_second_pass(B, n, far, linear):
    import torch
    ph = B.make_params(1, 1, 1, 256, 4, n_special=0, attn_dtype=B.ATTN_FP8_E4M3, qk_norm=1)
    ws = B.alloc_ws(B.litevggt_global_block_ws_bytes(ph, n))
    for seed in range(8):
        z, t, (q, k, v) = _exact_qkv_block(n, 256, seed, far)
        o, delta, aws = torch.full_like(q, float("nan")), torch.full_like(q, float("nan")), B.alloc_ws(B.litevggt_attn_ws_bytes(ph, n))
        B.litevggt_global_attn(ph, n, q, k, v, o, aws)
        state = torch.zeros(B.FP8_STATE_BYTES, dtype=torch.uint8, device="cuda")
        bw = B.block_weights(t) if linear == "bf16" else B.block_weights(
            t, B.LINEAR_FP8_E4M3, B.FP8_CURRENT if linear == "fp8" else B.FP8_DELAYED, state)
        B.litevggt_global_block(ph, n, z, bw, delta, ws)
        torch.cuda.synchronize()
        top = float(o.abs().max())
        if linear == "fp8-delayed":
            amax = state.view(torch.float32).reshape(4, -1)[:, 0].tolist()
            assert amax[0] == 1.0 and amax[1] == top, (seed, amax, top)
        scale = 1.0 if linear == "fp8-delayed" else _f32(np.float32(448.0) / np.float32(top))
        assert torch.equal(delta, o if linear == "bf16" else _through_e4m3(o, scale)), seed
        words, nqb = 4 * 2 * ((n + 511) // 512), (n + 255) // 256         # one flag per head and 256 queries, behind K and V twice
        base = (aws.data_ptr() + 255) // 256 * 256 - aws.data_ptr() + 256 + 4 * (4 * 2 * ((n + 63) // 64) * 4 * 64 * 8)
        flags = aws[base:base + words * 4].view(torch.int32).reshape(4, -1)[:, :nqb]
        assert flags.ne(0).nonzero().tolist() == [[h, b] for h in range(4) for b in sorted({f // 256 for f in far})]


# a captured block as it is served in FP8: every replay clears its words, takes its scales from the history and records into it,
# also after eager calls in the same scratch
@pytest.mark.parametrize("attn", ["fp8", "bf16"])
def test_block_replays_from_a_graph(B, attn):
    import torch
    n, dim = 700, 256
    t = {k: torch.from_numpy(v).cuda() for k, v in synth.block_weights(dim, seed=5).items()}
    t = {k: v.to(torch.bfloat16) if k.startswith("w_") else v for k, v in t.items()}
    states = torch.zeros(3, B.FP8_STATE_BYTES, dtype=torch.uint8, device="cuda")
    bws = [B.block_weights(t, B.LINEAR_FP8_E4M3, B.FP8_DELAYED, s) for s in states]
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    z = torch.randn(n, dim, generator=g, device="cuda").to(torch.bfloat16)
    ph = B.make_params(1, 1, 1, dim, 4, n_special=0, qk_norm=1, attn_dtype=B.ATTN_FP8_E4M3 if attn == "fp8" else B.ATTN_BF16)
    ws, got, other = B.alloc_ws(B.litevggt_global_block_ws_bytes(ph, n)), torch.empty_like(z), torch.empty_like(z)
    B.litevggt_global_block(ph, n, z, bws[2], other, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.litevggt_global_block(ph, n, z, bws[0], got, ws)
    for _ in range(4):
        want = torch.full_like(z, float("nan"))
        B.litevggt_global_block(ph, n, z, bws[1], want, ws)
        got.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want) and torch.equal(states[0], states[1])
        z.mul_(1.5)
        B.litevggt_global_block(ph, n, z, bws[2], other, ws)
        ws.fill_(0x7f)
        torch.cuda.synchronize()


# ------------------------------------------------------------------------------- importance
# pixel rows that are no multiple of 4 pixels, planes that are none (one pixel at a time), images
# behind an unaligned address, a single patch row and column, pixel rows wider than a workgroup,
# grids of one row segment per row and of segments of unequal height
@pytest.mark.parametrize("frames,h,w,patch,dim", [(2, 16, 16, 14, 64), (3, 5, 7, 3, 128), (2, 1, 1, 14, 64), (2, 3, 50, 14, 64),
                                                  (1, 37, 5, 14, 192), (3, 9, 2, 7, 1024), (260, 6, 6, 2, 64)])
@pytest.mark.parametrize("kind", ["f32", "f32 at 4", "u8", "u8 at 1"])
def test_importance_edges(B, frames, h, w, patch, dim, kind):
    import torch
    wl = synth.Workload("t", frames=frames, grid_h=h, grid_w=w, dim=dim, heads=dim // 64, patch=patch, canvas=64, seed=h)
    bits, xf, im = stored_inputs(wl)
    u8 = kind.startswith("u8")
    if u8:
        im = np.floor(im * 255).astype(np.uint8)
    flat = torch.zeros(im.size + 8, dtype=torch.uint8 if u8 else torch.float32, device="cuda")
    at = 1 if "at" in kind else 0
    img = flat[at:at + im.size]
    img.copy_(torch.from_numpy(im.reshape(-1)))
    ph = hip_params(wl, img_dtype=B.IMG_U8 if u8 else B.IMG_F32)
    grad = torch.full((frames, h * w), float("nan"), device="cuda")
    score = torch.full((frames, h * w), float("nan"), device="cuda")
    B.litevggt_importance(ph, img, to_dev_bf16(bits), grad, True, score, B.alloc_ws(frames * h * w * 4))
    torch.cuda.synchronize()
    ref, psi_g = O.importance(im.astype(np.float64) / (255.0 if u8 else 1.0), xf, oracle_params(wl))
    assert np.abs(grad.cpu().numpy() - psi_g.reshape(frames, -1)).max() <= 2e-5 * max(1.0, np.abs(psi_g).max())
    assert np.abs(score.cpu().numpy() - ref.reshape(frames, -1)).max() <= 2e-5


# more than 1024 channels: a second pass over the channels adds to the map, with the rows of a strip in
# segments (few frames) and whole; both maps in one launch with whole strips, an odd number of them, of one and three rows
@pytest.mark.parametrize("frames,h,w,dim", [(2, 9, 5, 1536), (1, 37, 6, 1088), (260, 4, 5, 1536), (1, 3, 36, 1088), (3, 1, 60, 1536),
                                            (1, 2, 20, 256)])
def test_importance_two_channel_passes(B, frames, h, w, dim):
    test_importance_edges(B, frames, h, w, 2, dim, "f32")


# White noise has gradients of one size everywhere, so the rounding of single pixels averages out and the
# sums decide: 2^-24, half a step of the result, is more than they may lose together (2-norm)
@pytest.mark.parametrize("h,w,patch", [(37, 37, 14), (5, 50, 7), (9, 11, 31)])
def test_gradient_map_sums_lose_less_than_the_results_rounding(B, h, w, patch):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(patch)
    img = torch.rand(12, 3, h * patch, w * patch, generator=g, device="cuda")
    ph = B.make_params(12, h, w, 64, 1, patch=patch)
    pl = B.litevggt_plan(ph)
    grad, score = (torch.empty(12, h * w, device="cuda") for _ in range(2))
    x = torch.zeros(pl.N, 64, dtype=torch.bfloat16, device="cuda")
    B.litevggt_importance(ph, img, x, grad, True, score, B.alloc_ws(pl.ws_bytes))
    torch.cuda.synchronize()
    v = img.double()
    lum = torch.nn.functional.pad((0.299 * v[:, 0] + 0.587 * v[:, 1] + 0.114 * v[:, 2])[:, None], (1, 1, 1, 1),
                                  mode="replicate")[:, 0]
    t, m, b = lum[:, :-2], lum[:, 1:-1], lum[:, 2:]
    gx = (t + 2 * m + b)[:, :, 2:] - (t + 2 * m + b)[:, :, :-2]
    gy = (b - t)[:, :, :-2] + 2 * (b - t)[:, :, 1:-1] + (b - t)[:, :, 2:]
    ref = torch.sqrt(gx * gx + gy * gy).reshape(12, h, patch, w, patch).mean((2, 4)).reshape(12, h * w)
    assert float((grad.double() - ref).norm() / ref.norm()) <= 2.0 ** -24


# ------------------------------------------------------------------------------- attention
def _attn64(q, k, v, norm, heads):
    import torch
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    for h in range(heads):
        qh, kh, vh = (t[:, h * 64:h * 64 + 64].double() for t in (q, k, v))
        if norm:
            qh, kh = (t / torch.sqrt((t * t).mean(1, keepdim=True) + 1e-6) for t in (qh, kh))
        for i in range(0, len(q), 4096):
            out[i:i + 4096, h * 64:h * 64 + 64] = torch.softmax(qh[i:i + 4096] @ kh.t().contiguous() * 0.125, 1) @ vh
    return out


# short sequences whose blocks are cut along the keys (8 XCDs with 64 slots): 12 blocks per XCD in
# halves (as given: normalised they are 64-query blocks), 17 and 46 (as given; normalised 17 stay whole; 46: three second
# pieces per idle slot, a ragged last block and key stage), 63 (nothing
# to gain, not cut), 65 (more than a round, not cut), 33 with a last block of one query; 28 and 32, cut in halves
# normalised as well
@pytest.mark.parametrize("n,heads", [(1500, 16), (4352, 8), (11709, 8), (5776, 16), (16640, 8), (16128, 8), (8193, 8), (3500, 16),
                                     (4096, 16)])
@pytest.mark.parametrize("kind", ["norm", "plain", "climbing"])
def test_attention_cut_rounds(B, n, heads, kind):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn(n, heads * 64, generator=g, device="cuda") for _ in range(3))
    if kind == "climbing":   # scores grow along the keys: every segment has a reference of its own
        k *= torch.linspace(0.1, 6.0, n, device="cuda")[:, None]
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    ph = B.make_params(1, 1, 1, heads * 64, heads, n_special=0, qk_norm=int(kind == "norm"))
    o = torch.full_like(q, float("nan"))
    B.litevggt_global_attn(ph, n, q, k, v, o, B.alloc_ws(B.litevggt_attn_ws_bytes(ph, n)))
    again = torch.full_like(q, float("nan"))
    B.litevggt_global_attn(ph, n, q, k, v, again, B.alloc_ws(B.litevggt_attn_ws_bytes(ph, n)))
    torch.cuda.synchronize()
    ref = _attn64(q, k, v, kind == "norm", heads)
    assert float((o.double() - ref).abs().max() / ref.abs().max()) <= 2e-2
    assert torch.equal(o, again)     # two partial sums: the same in either order


# Blocks cut in two along the keys whose pieces leave blocks to the per-row kernel (heads by fate: the block
# that holds the one query with a component along a long key's own direction).  n is 5 blocks and two waves, or
# one, of a sixth; its key stages are 11 and 11, or 11 and 10
@pytest.mark.parametrize("n", [1400, 1300])
def test_attention_cut_blocks_left_to_the_second_pass(B, n):
    import torch
    heads, nqb, nkv = 16, (n + 255) // 256, (n + 63) // 64
    split = 64 * (nkv - nkv // 2)                   # the first key of the second piece
    # per head: long keys, score of the query along them in binades (256 is what a reference may reach,
    # a row 60 under its wave's reference is lost), and how many pieces of the block arrive at their sums
    fates = {"reference too large in the first piece": ([100], 360, 1), "... in its first tile": ([5], 360, 1),
             "... in the second piece": ([split + 200], 360, 1), "... in its first tile too": ([split + 5], 360, 1),
             "... in both": ([100, split + 200], 360, 0), "low rows by the second piece": ([split + 200], 120, 2),
             "low rows by the first piece": ([5], 120, 2), "nothing": ([5], 30, 2)}
    plan = [(list(fates.values())[h % len(fates)], (5 * h + h // 8) % nqb) for h in range(heads)]
    assert {b for _, b in plan} == set(range(nqb))
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn(n, heads, 64, generator=g, device="cuda") for _ in range(3))
    q[:, :, 0] = k[:, :, 0] = 0.0
    for h, ((keys, binades, _), blk) in enumerate(plan):
        q[blk * 256 + 7 * h % 16 + (64 * (h % 4) if blk < nqb - 1 else 0), h, 0] = 32.0
        k[keys, h, 0] = binades * np.log(2.0) / (32.0 * 0.125)
    q, k, v = (t.reshape(n, heads * 64).to(torch.bfloat16) for t in (q, k, v))
    ph = B.make_params(1, 1, 1, heads * 64, heads, n_special=0)
    need = B.litevggt_attn_ws_bytes(ph, n)
    per = (heads * 2 * nkv * 4 * 64 * 16 + 255) // 256 * 256
    stride = 2 * ((n + 511) // 512)
    flags_at = 256 + 2 * per                        # behind the packed K and V; then the pieces' words
    sync_at = flags_at + (heads * stride * 4 + 255) // 256 * 256
    assert need > sync_at + heads * nqb * (256 * 64 + 1024) * 4        # room for every block's sums: cut
    ws = B.alloc_ws(need)
    o = torch.full_like(q, float("nan"))
    B.litevggt_global_attn(ph, n, q, k, v, o, ws)
    torch.cuda.synchronize()
    ref = _attn64(q, k, v, False, heads)
    assert float((o.double() - ref).abs().max() / ref.abs().max()) <= 2e-2
    base = (ws.data_ptr() + 255) // 256 * 256 - ws.data_ptr()
    words = ws[base:base + need].cpu().numpy()[:need // 4 * 4].view(np.uint32)
    flags = words[flags_at // 4:][:heads * stride].reshape(heads, stride)[:, :nqb]
    arrived = words[sync_at // 4:][:2 * heads * nqb:2].reshape(heads, nqb)
    want_flags, want_arrived = np.zeros((heads, nqb), np.uint32), np.full((heads, nqb), 2, np.uint32)
    for h, ((_, binades, pieces), blk) in enumerate(plan):
        want_flags[h, blk] = binades > 60
        want_arrived[h, blk] = pieces
    assert np.array_equal(flags != 0, want_flags != 0)
    assert np.array_equal(arrived, want_arrived)


# ------------------------------------------------------------------------------- scratch
# scratch sized for a longer sequence serves a shorter one that would ask for more: cut attention blocks
# (2000 of 2050 tokens as given; normalised they are 64-query blocks; 14800 of 14850, 5776 of 7000) and matching
# schedules with many partial results
@pytest.mark.parametrize("short,long,heads", [(2000, 2050, 16), (14800, 14850, 8), (5776, 7000, 16)])
@pytest.mark.parametrize("norm", [1, 0])
def test_attention_in_scratch_of_a_longer_sequence(B, short, long, heads, norm):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(short)
    q, k, v = (torch.randn(short, heads * 64, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    ph = B.make_params(1, 1, 1, heads * 64, heads, n_special=0, qk_norm=norm)
    need = B.litevggt_attn_ws_bytes(ph, long)
    assert need + 512 < B.litevggt_attn_ws_bytes(ph, short)
    ws = B.alloc_ws(need)
    used = (ws.data_ptr() + 255) // 256 * 256 - ws.data_ptr() + need
    ws[used:] = 0x5a
    o = torch.full_like(q, float("nan"))
    B.litevggt_global_attn(ph, short, q, k, v, o, ws[:used])
    torch.cuda.synchronize()
    ref = _attn64(q, k, v, norm, heads)
    assert float((o.double() - ref).abs().max() / ref.abs().max()) <= 2e-2
    assert bool((ws[used:] == 0x5a).all())


# (the attention of 2000 tokens in 64-query blocks, of 6900 in cut blocks where there is room)
@pytest.mark.parametrize("short,long", [(2000, 2050), (6900, 6950)])
def test_block_in_scratch_of_a_longer_sequence(B, short, long):
    import torch
    w = synth.block_weights(1024, seed=1)
    t = {k: torch.from_numpy(v).cuda() for k, v in w.items()}
    t = {k: v.to(torch.bfloat16) if k.startswith("w_") else v for k, v in t.items()}
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    z = torch.randn(short, 1024, generator=g, device="cuda").to(torch.bfloat16)
    ph = B.make_params(1, 1, 1, 1024, 16, n_special=0, qk_norm=1)
    need = B.litevggt_global_block_ws_bytes(ph, long)
    assert need + 512 < B.litevggt_global_block_ws_bytes(ph, short)
    delta = torch.full_like(z, float("nan"))
    B.litevggt_global_block(ph, short, z, B.block_weights(t), delta, B.alloc_ws(need))
    torch.cuda.synchronize()
    ref = _block64(z, t, 16)
    assert float((delta.double() - ref).abs().max() / ref.abs().max()) <= 2e-2


@pytest.mark.parametrize("frames,h,w,ratio", [(87, 16, 16, 0.5), (55, 20, 20, 0.5), (57, 16, 16, 0.9)])
def test_matching_in_scratch_of_a_longer_sequence(B, frames, h, w, ratio):
    import torch
    ph = B.make_params(frames, h, w, 64, 1, merge_ratio=ratio)
    pl = B.litevggt_plan(ph)
    need = B.litevggt_plan(B.make_params(frames + 1, h, w, 64, 1, merge_ratio=ratio)).ws_bytes
    assert need + 512 < pl.ws_bytes
    g = torch.Generator(device="cuda")
    g.manual_seed(frames)
    x = torch.randn(pl.N, 64, generator=g, device="cuda").to(torch.bfloat16)
    images = torch.rand(frames, 3, h * ph.patch, w * ph.patch, generator=g, device="cuda")
    out = []
    for nbytes in (pl.ws_bytes, need):
        ib, xx = B.alloc_index(pl), x.clone()
        grad, score = (torch.zeros(frames, h * w, device="cuda") for _ in range(2))
        B.litevggt_layers_run(ph, 1, images, xx, ib, grad, score, B.alloc_ws(nbytes))
        torch.cuda.synchronize()
        out.append((ib.anchor_of, ib.group_off, ib.group_mem, xx))
    assert all(torch.equal(a, b) for a, b in zip(*out))


# ------------------------------------------------------------------------------- layers that share an index
# The driver does the unmerge of a layer and the merge of the next in one pass where both use the same
# groups; step by step they give the same bits.  Widths of one piece per lane, a part of one, two; groups
# from one member to more than 64 and 256 (a still scene), a refresh in between, special tokens only.
@pytest.mark.parametrize("frames,h,w,special,ratio,dim,still", [(2, 16, 16, 5, 0.5, 256, False), (40, 9, 11, 3, 0.9, 64, True),
                                                                (300, 3, 4, 1, 0.9, 576, True), (5, 12, 13, 5, -1.0, 1024, False),
                                                                (3, 2, 2, 0, 0.0, 128, False)])
def test_layers_in_one_pass_equal_the_single_steps(B, frames, h, w, special, ratio, dim, still):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(frames + dim)
    wl = synth.Workload("t", frames=frames, grid_h=h, grid_w=w, dim=dim, heads=dim // 64, n_special=special, merge_ratio=ratio,
                        refresh_interval=3)
    ph = hip_params(wl)
    pl = B.litevggt_plan(ph)
    x = torch.randn(frames, h * w + special, dim, generator=g, device="cuda")
    if still:   # every frame shows a handful of things: large groups
        x[:, special:] = x[0, special:special + 4].repeat(frames, (h * w + 3) // 4, 1)[:, :h * w] + 0.1 * x[:, special:]
    x = x.reshape(pl.N, dim).to(torch.bfloat16)
    images = torch.rand(frames, 3, h * ph.patch, w * ph.patch, generator=g, device="cuda")
    maps = [torch.empty(frames, h * w, device="cuda") for _ in range(4)]
    ib, ws = B.alloc_index(pl), B.alloc_ws(pl.ws_bytes)
    got = x.clone()
    B.litevggt_layers_run(ph, 5, images, got, ib, maps[0], maps[1], ws)
    want, ix = x.clone(), B.alloc_index(pl)
    z = torch.empty(pl.M, dim, dtype=torch.bfloat16, device="cuda")
    y = torch.empty_like(z)
    largest = 0
    for l in range(5):
        if l % 3 == 0:
            B.litevggt_importance(ph, images, want, maps[2], l == 0, maps[3], ws)
            B.litevggt_select_anchors(ph, maps[3], ix)
            B.litevggt_match(ph, want, ix, None, ws)
            largest = max(largest, int(ix.group_off[1:].sub(ix.group_off[:-1]).max()))
        B.litevggt_merge(ph, want, ix, z)
        B.litevggt_global_attn(ph, pl.M, z, z, z, y, ws)
        B.litevggt_unmerge(ph, y, ix, want, want)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert torch.equal(maps[1], maps[3])         # the score map, fused on its own and with the partition
    assert not still or largest > 64


# The same with large groups whose rows go to several workgroups by channels: 128 at a time up to 512
# channels (two and three slices, the last one of half a slice), 256 at a time beyond; one group with nearly every token
@pytest.mark.parametrize("frames,h,w,special,ratio,dim,blank", [(80, 5, 6, 2, 0.9, 256, False), (70, 4, 4, 0, 0.9, 320, False),
                                                                (80, 4, 4, 1, 0.9, 1024, False), (90, 6, 6, 5, 0.98, 960, False),
                                                                (9, 20, 20, 5, 0.9, 768, True), (9, 20, 20, 0, 0.9, 64, True)])
def test_large_groups_in_one_pass_equal_the_single_steps(B, frames, h, w, special, ratio, dim, blank):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(frames + dim)
    wl = synth.Workload("t", frames=frames, grid_h=h, grid_w=w, dim=dim, heads=dim // 64, n_special=special, merge_ratio=ratio)
    ph = hip_params(wl)
    pl = B.litevggt_plan(ph)
    x = torch.randn(frames, h * w + special, dim, generator=g, device="cuda")
    x[:, special:] = x[0, special:] + (0.0 if blank else 0.1) * x[:, special:]      # a still scene
    if blank:
        x[:, special:] = x[0, special]
    x = x.reshape(pl.N, dim).to(torch.bfloat16)
    images = torch.rand(frames, 3, h * ph.patch, w * ph.patch, generator=g, device="cuda")
    grad, score = (torch.empty(frames, h * w, device="cuda") for _ in range(2))
    ib, ws = B.alloc_index(pl), B.alloc_ws(pl.ws_bytes)
    got, want = x.clone(), x.clone()
    B.litevggt_layers_run(ph, 3, images, got, ib, grad, score, ws)
    z = torch.empty(pl.M, dim, dtype=torch.bfloat16, device="cuda")
    y = torch.empty_like(z)
    for _ in range(3):
        B.litevggt_merge(ph, want, ib, z)
        B.litevggt_global_attn(ph, pl.M, z, z, z, y, ws)
        B.litevggt_unmerge(ph, y, ib, want, want)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    largest = int(ib.group_off[1:].sub(ib.group_off[:-1]).max())
    assert largest > (pl.n_src if blank else 64)


# With a block y is the block's delta, z feeds its LayerNorms and the packed weights are kept across the layers; in bf16, and as it
# is served in FP8 (E4M3 attention, E4M3 layers, delayed scaling: a history each)
@pytest.mark.parametrize("frames,h,w,dim,still", [(2, 16, 16, 256, False), (80, 5, 6, 256, True), (3, 12, 13, 768, False)])
@pytest.mark.parametrize("fp8", [False, True])
def test_layers_with_a_block_in_one_pass_equal_the_single_steps(B, frames, h, w, dim, still, fp8):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(frames + dim)
    t = {k: torch.from_numpy(v).cuda() for k, v in synth.block_weights(dim, seed=frames).items()}
    t = {k: v.to(torch.bfloat16) if k.startswith("w_") else v for k, v in t.items()}
    states = torch.zeros(2, B.FP8_STATE_BYTES, dtype=torch.uint8, device="cuda")
    bws = [B.block_weights(t, B.LINEAR_FP8_E4M3, B.FP8_DELAYED, s) if fp8 else B.block_weights(t) for s in states]
    wl = synth.Workload("t", frames=frames, grid_h=h, grid_w=w, dim=dim, heads=dim // 64, n_special=5, merge_ratio=0.9,
                        refresh_interval=3)
    ph = hip_params(wl, block=bws[0], attn_dtype=B.ATTN_FP8_E4M3 if fp8 else B.ATTN_BF16)
    pl = B.litevggt_plan(ph)
    x = torch.randn(frames, h * w + 5, dim, generator=g, device="cuda")
    if still:
        x[:, 5:] = x[0, 5:] + 0.1 * x[:, 5:]
    x = x.reshape(pl.N, dim).to(torch.bfloat16)
    images = torch.rand(frames, 3, h * ph.patch, w * ph.patch, generator=g, device="cuda")
    maps = [torch.empty(frames, h * w, device="cuda") for _ in range(4)]
    ib, ix, ws = B.alloc_index(pl), B.alloc_index(pl), B.alloc_ws(pl.ws_bytes)
    got, want = x.clone(), x.clone()
    B.litevggt_layers_run(ph, 5, images, got, ib, maps[0], maps[1], ws)
    z = torch.empty(pl.M, dim, dtype=torch.bfloat16, device="cuda")
    y = torch.empty_like(z)
    for l in range(5):
        if l % 3 == 0:
            B.litevggt_importance(ph, images, want, maps[2], l == 0, maps[3], ws)
            B.litevggt_select_anchors(ph, maps[3], ix)
            B.litevggt_match(ph, want, ix, None, ws)
        B.litevggt_merge(ph, want, ix, z)
        B.litevggt_global_block(ph, pl.M, z, bws[1], y, B.alloc_ws(B.litevggt_global_block_ws_bytes(ph, pl.M)))
        B.litevggt_unmerge(ph, y, ix, want, want)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert torch.equal(states[0], states[1]) and bool(states.any()) == fp8
    assert not still or int(ix.group_off[1:].sub(ix.group_off[:-1]).max()) > 64


# ------------------------------------------------------------------------------- short sequences, attention
# 64-query blocks whose waves share the keys out: waves without a key tile (1 to 96 tokens), the last tile
# with one key, whole tiles, one tile more for one wave, the most blocks that are taken this way and one
# token more (16 heads: 2048 normalised, 1024 as given; 4 and 12 heads, never cut: 8192 and 2688)
@pytest.mark.parametrize("n,heads", [(1, 4), (31, 1), (32, 8), (33, 4), (64, 16), (65, 3), (96, 8), (97, 4), (129, 4), (394, 4),
                                     (522, 4), (1024, 16), (1025, 16), (2048, 16), (2049, 16), (2688, 12), (2689, 12),
                                     (8192, 4), (8193, 4)])
@pytest.mark.parametrize("kind", ["norm", "plain", "climbing", "falling"])
def test_attention_short_sequences(B, n, heads, kind):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn(n, heads * 64, generator=g, device="cuda") for _ in range(3))
    if kind in ("climbing", "falling"):   # every wave's keys have a reference of their own
        ramp = torch.linspace(0.1, 6.0, n, device="cuda")[:, None]
        k *= ramp if kind == "climbing" else ramp.flip(0)
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    ph = B.make_params(1, 1, 1, heads * 64, heads, n_special=0, qk_norm=int(kind == "norm"))
    ws = B.alloc_ws(B.litevggt_attn_ws_bytes(ph, n))
    ws.fill_(0x7f)                        # flags are cleared by the call
    o, again = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    B.litevggt_global_attn(ph, n, q, k, v, o, ws)
    B.litevggt_global_attn(ph, n, q, k, v, again, ws)
    torch.cuda.synchronize()
    ref = _attn64(q, k, v, kind == "norm", heads)
    assert float((o.double() - ref).abs().max() / ref.abs().max()) <= 2e-2
    assert torch.equal(o, again)


# queries along long keys: references beyond what serves in one wave's keys or another's, rows far below their
# wave's reference, in the first, a middle and the last 64-query block of a 256-query flag and across two flags
@pytest.mark.parametrize("n,heads", [(700, 8), (394, 4)])
def test_attention_short_blocks_left_to_the_second_pass(B, n, heads):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn(n, heads, 64, generator=g, device="cuda") for _ in range(3))
    q[:, :, 0] = k[:, :, 0] = 0.0
    spots = [(5, 3, 360), (n - 1, 70, 120), (n // 2, 255, 360), (7, n - 1, 30), (n // 3, 256, 20)]   # key, query, binades
    for h in range(heads):
        for key, query, binades in spots[h % 4:h % 4 + 2]:
            q[query, h, 0] = 32.0
            k[key, h, 0] = binades * np.log(2.0) / (32.0 * 0.125)
    q, k, v = (t.reshape(n, heads * 64).to(torch.bfloat16) for t in (q, k, v))
    ph = B.make_params(1, 1, 1, heads * 64, heads, n_special=0)
    need = B.litevggt_attn_ws_bytes(ph, n)
    ws = B.alloc_ws(need)
    o = torch.full_like(q, float("nan"))
    B.litevggt_global_attn(ph, n, q, k, v, o, ws)
    torch.cuda.synchronize()
    ref = _attn64(q, k, v, False, heads)
    assert float((o.double() - ref).abs().max() / ref.abs().max()) <= 2e-2
    nqb, stride, nkv = (n + 255) // 256, 2 * ((n + 511) // 512), (n + 63) // 64
    base = (ws.data_ptr() + 255) // 256 * 256 - ws.data_ptr() + 256 + 2 * ((heads * 2 * nkv * 4 * 64 * 16 + 255) // 256 * 256)
    flags = ws[base:base + heads * stride * 4].cpu().numpy().view(np.uint32).reshape(heads, stride)[:, :nqb]
    want = np.zeros((heads, nqb), bool)
    for h in range(heads):
        for _, query, _ in spots[h % 4:h % 4 + 2]:      # a query meets both keys of its head
            want[h, query // 256] |= max(b for _, _, b in spots[h % 4:h % 4 + 2]) > 60
    assert np.array_equal(flags != 0, want)
    # o in q's place: the second pass starts again from q, so no block of a flag may have been stored
    B.litevggt_global_attn(ph, n, q, k, v, q, ws)
    torch.cuda.synchronize()
    assert float((q.double() - ref).abs().max() / ref.abs().max()) <= 2e-2


# K and V read from their rows (up to 768 tokens) and from their re-layout (the output takes V's place): the same bits; fewer
# keys than waves have tiles for, ragged tiles, waves with one to six tiles, the longest sequence and one token more, an
# infinite value of the last key, whose neighbours beyond the end count as zeros
@pytest.mark.parametrize("n,heads", [(1, 1), (31, 2), (32, 1), (33, 3), (64, 1), (65, 8), (127, 4), (129, 2), (257, 3), (394, 16),
                                     (511, 8), (640, 4), (767, 8), (768, 16), (769, 8)])
def test_attention_short_rows_equal_relaid(B, n, heads):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn(n, heads * 64, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    v[-1, 5] = float("inf")
    ph = B.make_params(1, 1, 1, heads * 64, heads, n_special=0, qk_norm=1)
    ws = B.alloc_ws(B.litevggt_attn_ws_bytes(ph, n))
    o = torch.full_like(q, float("nan"))
    B.litevggt_global_attn(ph, n, q, k, v, o, ws)
    relaid = v.clone()
    B.litevggt_global_attn(ph, n, q, k, relaid, relaid, ws)
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), relaid.view(torch.int16))
    fine = torch.ones(heads * 64, dtype=torch.bool, device="cuda")
    fine[5] = False
    v[-1, 5] = 0.0
    ref = _attn64(q, k, v, True, heads)
    assert bool(torch.isinf(o[:, 5]).all())
    assert float((o.double() - ref)[:, fine].abs().max() / ref.abs().max()) <= 2e-2


# V read from its rows: what lies beyond a sequence's end counts as zeros, whatever it is.  Frames between frames of NaN
# and of infinity and before rows of NaN give what the re-layout (the output takes V's place) gives among zeros: in 64-query
# blocks and in a stream, last tiles and stages of 1, 2, 9, 10, 30 and 33 keys, so that rows, and whole parts of a stage, lie beyond
@pytest.mark.parametrize("frames,h,w,heads", [(3, 4, 7, 4), (3, 6, 6, 4), (3, 4, 23, 4), (3, 13, 25, 4), (2, 12, 61, 16),
                                              (33, 4, 79, 8), (33, 13, 25, 8), (33, 12, 29, 8), (33, 5, 89, 8), (20, 37, 37, 8)])
@pytest.mark.parametrize("res", [0, 1])
def test_attention_values_end_with_their_sequence(B, frames, h, w, heads, res):
    import torch
    n, c = h * w + 5, heads * 64
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, x = (torch.randn(frames * n, c, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    room = torch.full((frames * n + 64, c), float("nan"), dtype=torch.bfloat16, device="cuda")
    v = room[:frames * n]
    v.copy_(torch.randn(frames * n, c, generator=g, device="cuda"))
    relaid = v.clone()
    relaid.view(frames, n, c)[1::2] = 0.0
    v.view(frames, n, c)[1::4] = float("nan")
    v.view(frames, n, c)[3::4] = float("inf")
    ph = B.make_params(frames, h, w, c, heads, qk_norm=1)
    ws = B.alloc_ws(B.litevggt_frame_attn_ws_bytes(ph))
    got = torch.full_like(q, float("nan"))
    B.litevggt_frame_attn(ph, q, k, v, x if res else None, got, ws)
    B.litevggt_frame_attn(ph, q, k, relaid, x if res else None, relaid, ws)
    torch.cuda.synchronize()
    got, relaid = (t.view(torch.int16).view(frames, n, c)[::2] for t in (got, relaid))
    assert torch.equal(got, relaid)


# frames of a few hundred tokens with the residual added in place, in 64-query blocks and one frame beyond
@pytest.mark.parametrize("frames,h,w,heads,norm", [(2, 16, 16, 4, 1), (25, 15, 17, 4, 1), (26, 15, 17, 4, 1), (2, 37, 37, 8, 1),
                                                   (2, 5, 5, 1, 0)])
def test_frame_attention_short_frames_in_place(B, frames, h, w, heads, norm):
    import torch
    n = h * w + 5
    g = torch.Generator(device="cuda")
    g.manual_seed(frames)
    x = torch.randn(frames * n, heads * 64, generator=g, device="cuda").to(torch.bfloat16)
    ph = B.make_params(frames, h, w, heads * 64, heads, qk_norm=norm)
    got = x.clone()
    B.litevggt_frame_attn(ph, got, got, got, got, got, B.alloc_ws(B.litevggt_frame_attn_ws_bytes(ph)))
    torch.cuda.synchronize()
    ref = torch.cat([f.double() + _attn64(f, f, f, norm, heads) for f in x.reshape(frames, n, -1)])
    assert float((got.double() - ref).abs().max() / ref.abs().max()) <= 2e-2


# ------------------------------------------------------------------------------- blocks that follow each other
# more 256-query blocks than slots, in workgroups that stay: the fewest key stages (4) and one fewer, a
# last stage of one key and a whole one, last blocks with one, two and all waves at work, one list for all
# XCDs (pairs no multiple of 8), tails of the last round up to half of the slots and beyond, residual in
# place and none, an output that is 8-byte aligned only; six blocks per slot (priorities that come round again) with
# one list and with eight
@pytest.mark.parametrize("frames,h,w,heads,res", [(65, 14, 18, 8, 1), (65, 12, 16, 8, 1), (65, 11, 17, 8, 1), (90, 14, 18, 3, 1),
                                                  (33, 16, 16, 16, 1), (43, 17, 18, 7, 0), (40, 24, 25, 6, 1), (20, 37, 37, 8, 1),
                                                  (20, 37, 37, 8, 8), (13, 28, 37, 12, 1), (300, 11, 23, 5, 1),
                                                  (200, 15, 17, 8, 0)])
def test_attention_blocks_in_a_stream(B, frames, h, w, heads, res):
    import torch
    n = h * w + 5
    g = torch.Generator(device="cuda")
    g.manual_seed(frames * heads)
    x = torch.randn(frames * n, heads * 64, generator=g, device="cuda").to(torch.bfloat16)
    ph = B.make_params(frames, h, w, heads * 64, heads, qk_norm=1)
    ws = B.alloc_ws(B.litevggt_frame_attn_ws_bytes(ph))
    ws.fill_(0x7f)                              # counters are cleared by the call
    outs = []
    for _ in range(2):
        if res == 1:
            got = x.clone()
            B.litevggt_frame_attn(ph, got, got, got, got, got, ws)
        else:
            got = torch.full((x.numel() + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")[res // 2:][:x.numel()].view_as(x)
            B.litevggt_frame_attn(ph, x, x, x, x if res else None, got, ws)
        torch.cuda.synchronize()
        outs.append(got.clone())
    ref = torch.cat([_attn64(f, f, f, True, heads) + (f.double() if res else 0.0) for f in x.reshape(frames, n, -1)])
    assert float((outs[0].double() - ref).abs().max() / ref.abs().max()) <= 2e-2
    assert torch.equal(outs[0], outs[1])


# last blocks whose waves take 32 queries each: 127 and 128 queries (and 129, where they take 64), whole waves and one more query;
# the bits of the re-laid form (the output takes V's place), whose waves take 64
@pytest.mark.parametrize("frames,h,w,heads", [(33, 18, 21, 8), (33, 1, 379, 8), (33, 19, 20, 8), (33, 15, 21, 8), (33, 4, 79, 8),
                                              (22, 11, 49, 8), (22, 20, 27, 8), (30, 9, 67, 6), (30, 4, 151, 6)])
@pytest.mark.parametrize("res", [0, 1])
def test_attention_stream_narrow_last_blocks(B, frames, h, w, heads, res):
    import torch
    n = h * w + 5
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn(frames * n, heads * 64, generator=g, device="cuda").to(torch.bfloat16)
    ph = B.make_params(frames, h, w, heads * 64, heads, qk_norm=1)
    got = torch.full_like(x, float("nan"))
    B.litevggt_frame_attn(ph, x, x, x, x if res else None, got, B.alloc_ws(B.litevggt_frame_attn_ws_bytes(ph)))
    torch.cuda.synchronize()
    relaid = x.clone()
    B.litevggt_frame_attn(ph, x, x, relaid, x if res else None, relaid, B.alloc_ws(B.litevggt_frame_attn_ws_bytes(ph)))
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), relaid.view(torch.int16))
    ref = torch.cat([_attn64(f, f, f, True, heads) + (f.double() if res else 0.0) for f in x.reshape(frames, n, -1)])
    # bf16 weights and outputs: 2^-8 of a value twice, as for the other blocks
    assert float((got.double() - ref).abs().max() / ref.abs().max()) <= 2e-2


# the same rows alone (one launch per block) and as one of many blocks have the same bits
@pytest.mark.parametrize("n,heads", [(8200, 16), (13500, 16), (11200, 12)])
def test_attention_stream_equals_single_blocks(B, n, heads):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    q, k, v = (torch.randn(n, heads * 64, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    ph = B.make_params(1, 1, 1, heads * 64, heads, n_special=0, qk_norm=1)
    ws = B.alloc_ws(B.litevggt_attn_ws_bytes(ph, n))
    o = torch.full_like(q, float("nan"))
    B.litevggt_global_attn(ph, n, q, k, v, o, ws)
    odd = torch.full((q.numel() + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")[4:][:q.numel()].view_as(q)
    B.litevggt_global_attn(ph, n, q, k, v, odd, ws)
    torch.cuda.synchronize()
    assert torch.equal(o, odd)


# a captured call: its counters are cleared in every replay, also after eager calls in the same scratch
def test_attention_stream_replays_from_a_graph(B):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    x = torch.randn(40 * 261, 512, generator=g, device="cuda").to(torch.bfloat16)
    ph = B.make_params(40, 16, 16, 512, 8, qk_norm=1)
    ws, want, got = B.alloc_ws(B.litevggt_frame_attn_ws_bytes(ph)), torch.empty_like(x), torch.empty_like(x)
    B.litevggt_frame_attn(ph, x, x, x, x, want, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.litevggt_frame_attn(ph, x, x, x, x, got, ws)
    for _ in range(3):
        got.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        B.litevggt_frame_attn(ph, x, x, x, None, got, ws)
        ws.fill_(0x7f)
        torch.cuda.synchronize()


# ------------------------------------------------------------------------------- matching of few tokens
# 64 x 64 row tiles: one src row, whole tiles of both, one row more; one, three and five channel batches per
# half, sixteen; the most dst tiles that are lists (4096 dst rows) and one more, and near the most workgroups; 128,
# 256 and 258 src rows
@pytest.mark.parametrize("frames,h,w,special,ratio,dim", [(2, 1, 2, 0, 0.5, 64), (2, 8, 16, 0, 0.5, 192), (3, 8, 8, 0, 0.5, 320),
                                                          (2, 64, 63, 0, 0.016, 64), (2, 64, 64, 0, 0.016, 64), (4, 37, 37, 5, 0.9, 128),
                                                          (2, 37, 37, 5, 0.9, 1024), (30, 16, 16, 5, 0.9, 64),
                                                          (2, 16, 16, 5, 0.5, 256), (3, 16, 16, 5, 0.5, 128), (2, 16, 17, 5, 0.95, 128)])
def test_match_of_few_tokens(B, frames, h, w, special, ratio, dim):
    import torch
    ph = B.make_params(frames, h, w, dim, dim // 64, n_special=special, merge_ratio=ratio)
    pl = B.litevggt_plan(ph)
    g = torch.Generator(device="cuda")
    g.manual_seed(frames * dim)
    x = torch.randn(pl.N, dim, generator=g, device="cuda").to(torch.bfloat16)
    _check_index(B, ph, x)
