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
