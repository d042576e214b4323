"""GPU parity of kernels at the sizes where their tiling, splitting or dispatch changes."""
import numpy as np
import pytest

from oracle import litevggt_oracle as O
from paper_2512_04939_amd import synth

from helpers import hip_params, oracle_params

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


# groups: the largest sequence one workgroup sorts, the smallest beyond it, a chunk of the general
# sort that ends on a wave's last element, and one slot count above 16 bits (three digit passes)
@pytest.mark.parametrize("frames,h,w,special,ratio", [(64, 15, 17, 1, 0.9), (5, 52, 63, 1, 0.5), (2, 1, 1, 0, 0.0),
                                                      (17, 32, 32, 0, 0.75), (70, 32, 32, 2, 0.0)])
def test_groups_edges(B, frames, h, w, special, ratio):
    import torch
    ph = B.make_params(frames, h, w, 64, 1, n_special=special, merge_ratio=ratio)
    pl = B.litevggt_plan(ph)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = torch.randn(pl.N, 64, generator=g, device="cuda").to(torch.bfloat16)
    _check_index(B, ph, x)
