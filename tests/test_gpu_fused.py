"""The kernels that run several merge levels at once, at every grid size whose
plan differs (8^2: none; 16^2, 32^2: the top kernel with two and three levels;
64^2: with four, in one window; 128^2: two windows and single levels beside it;
256^2, 512^2, 1024^2: merge-up and merge-down groups of each length, windows that
do not divide the grid).  The reference is the level-by-level pass of every
level, which the batch's persistent kernel runs: the same arithmetic in the same
order, so every result is bitwise the same."""
import numpy as np
import pytest
import torch

from scenes import scene_like_512

pytestmark = pytest.mark.gpu

from gpu_common import log, to_dev  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    from paper_2505_02041_amd import Context
    return Context(0)


def _scene(S):
    sc = scene_like_512(S, 300 + S, max(2, S // 16), max(2, S // 16), box_sigma=3.0)
    rng = np.random.default_rng(S)
    # light everywhere, so that every lookup carries a value
    eps = sc.eps + rng.uniform(0.01, 0.1, sc.eps.shape).astype(np.float32)
    return to_dev(eps), to_dev(sc.sigma), to_dev(rng.normal(size=(S, S)))


@pytest.mark.parametrize("S", [8, 16, 32, 64, 128, 256, 512, 1024])
def test_fused_levels_match_single_levels(ctx, S):
    from paper_2505_02041_amd import Batch, _lib
    log(f"fused merges S={S}")
    e, s, g = _scene(S)
    F, ge, gs = (torch.empty_like(e) for _ in range(3))
    b = Batch([{"emission": e, "sigma_t": s, "fluence": F, "grad_fluence": g,
                "grad_emission": ge, "grad_sigma_t": gs}], ctx,
              flags=_lib.HRC_FLAG_BATCH_PERSISTENT)
    b.launch()
    b.status()
    N = S.bit_length() - 1
    assert torch.equal(ctx.hrc_forward(e, s), F)
    for quadrants in (_lib.HRC_FLAG_QUADRANTS_1, _lib.HRC_FLAG_QUADRANTS_2):
        assert torch.equal(ctx.hrc_forward(e, s, flags=quadrants), F)
    # a workspace of NaNs: nothing a kernel leaves out is read
    ws = ctx.reserve(N)
    ws.view(torch.float32).fill_(float("nan"))
    assert torch.equal(ctx.hrc_forward(e, s, flags=_lib.HRC_FLAG_KEEP_PYRAMID, reserve=ws), F)
    got = ctx.hrc_backward(e, s, g, flags=_lib.HRC_FLAG_REUSE_PYRAMID, reserve=ws)
    assert torch.equal(got[0], ge) and torch.equal(got[1], gs)
    ctx.workspace(N, True).view(torch.float32).fill_(float("nan"))
    got = ctx.hrc_backward(e, s, g)
    assert torch.equal(got[0], ge) and torch.equal(got[1], gs)
    ctx.release_workspaces()


@pytest.mark.parametrize("S", [16, 32, 64, 128, 256, 512, 1024])
@pytest.mark.parametrize("half", [False, True], ids=["f32", "f16"])
def test_fused_rgb_matches_channels(ctx, S, half):
    from paper_2505_02041_amd import _lib
    log(f"fused RGB merges S={S} half={half}")
    N = S.bit_length() - 1
    H = _lib.HRC_FLAG_HALF_INTERVALS if half else 0
    e, s, g = _scene(S)
    e3 = torch.stack([e, torch.roll(e, 3, 1), 0.25 * e]).contiguous()
    g3 = torch.stack([g, -g, torch.roll(g, 5, 0)]).contiguous()
    ws = ctx.reserve_rgb(N, H)
    ws.fill_(0xff)
    F3 = ctx.hrc_forward_rgb(e3, s, flags=H | _lib.HRC_FLAG_KEEP_PYRAMID, reserve=ws)
    ge3, _ = ctx.hrc_backward_rgb(e3, s, g3, flags=H | _lib.HRC_FLAG_REUSE_PYRAMID, reserve=ws)
    assert torch.equal(ctx.hrc_forward_rgb(e3, s, flags=H), F3)
    for c in range(3):
        e1, g1 = e3[c].contiguous(), g3[c].contiguous()
        assert torch.equal(F3[c], ctx.hrc_forward(e1, s, flags=H))
        ge, _ = ctx.hrc_backward(e1, s, g1, flags=H)
        assert torch.equal(ge3[c], ge)
    ctx.release_workspaces()
