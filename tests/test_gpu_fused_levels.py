"""The kernels that run several merge levels at once where test_gpu_fused.py does
not reach: the plans of 2048^2 and 4096^2 (two merge-up kernels in a row, several
merge-down pairs), bitwise against the level-by-level passes of the persistent
kernel, with an environment map across quadrant groups, and the 16-bit storage's
rounding points, which no level-by-level pass of the library shows.

Rounding points.  The model is the oracle's FP64 steps with T_2 .. T_(N-1) rounded
to half where the kernels store or would store them.  d_n is the change of the
model's fluence when level n is left unrounded.  Were the kernels to leave level n
unrounded, their difference from the model would hold d_n once; rounding all
levels, it holds only values that FP32 sends to the other neighbouring half, which
are uncorrelated with d_n.  So the projection of the difference on d_n is 1 or 0 up
to that noise, and 0.25 separates the two.  (The noise: a value within its FP32
error, about 2^-22, of a midpoint goes the other way, one in 2^11 of those stored,
by 2^-11 at most twice: a mean square of 2^-32 of the value against 2^-24.6 for the
rounding itself, so 0.08 of the length of all d_n together, and its projection on
any one direction of some 10^4 pixels is a hundredth of that.)"""
import numpy as np
import pytest
import torch

from oracle import hrc as O
from scenes import scene_like_512

pytestmark = pytest.mark.gpu

from gpu_common import log, to_dev  # noqa: E402


@pytest.fixture()
def ctx():
    from paper_2505_02041_amd import Context
    c = Context(0)
    yield c
    c.set_environment(None)
    c.release_workspaces()


def _scene(S):
    sc = scene_like_512(S, 300 + S, max(2, S // 16), max(2, S // 16), box_sigma=3.0)
    rng = np.random.default_rng(S)
    # light everywhere, so that every lookup carries a value
    eps = sc.eps + rng.uniform(0.01, 0.1, sc.eps.shape).astype(np.float32)
    return eps, sc.sigma, rng.normal(size=(S, S)).astype(np.float32)


@pytest.mark.parametrize("S,grad", [(2048, True), (4096, False)])
def test_large_plans_match_single_levels(ctx, S, grad):
    from paper_2505_02041_amd import Batch, _lib
    log(f"fused merges S={S}")
    e, s, g = (to_dev(a) for a in _scene(S))
    item = {"emission": e, "sigma_t": s, "fluence": torch.empty_like(e)}
    if grad:
        item.update(grad_fluence=g, grad_emission=torch.empty_like(e),
                    grad_sigma_t=torch.empty_like(e))
    b = Batch([item], ctx, flags=_lib.HRC_FLAG_BATCH_PERSISTENT)
    b.launch()
    b.status()
    del b
    torch.cuda.empty_cache()
    for quadrants in (0, _lib.HRC_FLAG_QUADRANTS_1):
        assert torch.equal(ctx.hrc_forward(e, s, flags=quadrants), item["fluence"])
    if grad:
        ge, gs = ctx.hrc_backward(e, s, g)
        assert torch.equal(ge, item["grad_emission"]) and torch.equal(gs, item["grad_sigma_t"])


@pytest.mark.parametrize("half", [False, True], ids=["f32", "f16"])
def test_large_rgb_matches_channels(ctx, half):
    from paper_2505_02041_amd import _lib
    log(f"fused RGB merges S=2048 half={half}")
    H = _lib.HRC_FLAG_HALF_INTERVALS if half else 0
    e, s, _ = (to_dev(a) for a in _scene(2048))
    e3 = torch.stack([e, torch.roll(e, 3, 1), 0.25 * e]).contiguous()
    F3 = ctx.hrc_forward_rgb(e3, s, flags=H)
    for c in range(3):
        assert torch.equal(F3[c], ctx.hrc_forward(e3[c].contiguous(), s, flags=H))


@pytest.mark.parametrize("S", [32, 64, 128, 256, 512])
@pytest.mark.parametrize("half", [False, True], ids=["f32", "f16"])
def test_environment_across_quadrant_groups(ctx, S, half):
    from paper_2505_02041_amd import _lib
    log(f"environment S={S} half={half}")
    e, s, _ = (to_dev(a) for a in _scene(S))
    ctx.set_environment(np.random.default_rng(S).uniform(0.2, 2.0, 61).astype(np.float32))
    H = _lib.HRC_FLAG_HALF_INTERVALS if half else 0
    F = ctx.hrc_forward(e, s, flags=H)
    for quadrants in (_lib.HRC_FLAG_QUADRANTS_1, _lib.HRC_FLAG_QUADRANTS_2):
        assert torch.equal(ctx.hrc_forward(e, s, flags=H | quadrants), F)


def _model(eps, sig, rounded, env):
    """The oracle's fluence with the levels in `rounded` stored as halves."""
    N = O.log2_size(eps.shape[0])
    F = np.zeros(eps.shape)
    for d in O.QUADRANTS:
        E, G = (np.asarray(O.to_frame(np.asarray(a, np.float64), d)) for a in (eps, sig))
        half = lambda t, n: tuple(a.astype(np.float16).astype(np.float64) for a in t) if n in rounded else t
        T = [O.seed_level(E, G, n) for n in range(3)]
        Q = [None, None, half(T[2], 2)]
        for n in range(3, N + 1):
            Q.append(half(O.merge_up(Q[n - 1], n), n))
        light = None if env is None else O.environment_fluence(env, d, N)
        R = np.zeros((1, 1 << N, eps.shape[0]))
        if light is not None:
            R += light[N][None, :, None]
        for n in range(N - 1, -1, -1):
            # (levels 0 and 1 are folded on chip, from the unrounded T_0 .. T_2)
            R = O.merge_down(R, *((Q[n], Q[n + 1]) if n >= 2 else (T[n], T[n + 1])), n,
                             None if light is None else light[n + 1])
        F += O.from_frame(O.gather(R, 0.0 if light is None else float(light[0][0])), d)
    return F


@pytest.mark.parametrize("S", [32, 64, 128, 256])
@pytest.mark.parametrize("K", [0, 61])
def test_half_rounds_every_level_once(ctx, S, K):
    from paper_2505_02041_amd import _lib
    log(f"16-bit rounding points S={S} environment {K}")
    eps, sig, _ = _scene(S)
    env = np.random.default_rng(K + S).uniform(0.2, 2.0, K).astype(np.float32) if K else None
    if K:
        ctx.set_environment(env)
    F = ctx.hrc_forward(to_dev(eps), to_dev(sig), flags=_lib.HRC_FLAG_HALF_INTERVALS)
    levels = set(range(2, O.log2_size(S)))
    want = _model(eps, sig, levels, env)
    diff = F.cpu().numpy().astype(np.float64) - want
    for n in sorted(levels):
        d = _model(eps, sig, levels - {n}, env) - want
        c = float((diff * d).sum() / (d * d).sum())
        log(f"  level {n}: {c:.4f}")
        assert abs(c) < 0.25, f"level {n}: projection {c}"
