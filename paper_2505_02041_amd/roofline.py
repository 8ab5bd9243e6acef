"""Algorithmic HBM bytes of each kernel launch (the roofline's numerator).

Every level a launch is defined to read is counted as read once, and every level
it stores as written once, over the four quadrant solves, in FP32: an interval
<L, T> is 8 bytes, an angular fluence 4 bytes, a scene value 4 bytes.  Levels that
a kernel builds and consumes on chip are not counted, and neither are re-reads
that a cache may or may not absorb (neighbouring blocks sharing rows): they are
what the kernels must keep on chip to reach the roofline.

Counts per quadrant follow Section 4.3: T_n has X^2 (1 + 2^-n) entries, R_n has
X^2, with X = S = 2^N.  ``iv`` is the bytes of a stored interval: 8 in FP32, 4
with the 16-bit storage of ``HRC_FLAG_HALF_INTERVALS``, twice that with RGB
intervals.

``forward_launches`` and ``backward_launches`` list the launches the library
makes: (kernel, the passes of Algorithm 1 it runs as (name, level), bytes), in
order, so that the per-pass times of ``hrc_profile_solve`` (where a kernel's
time is shared equally by its passes) add up to launches.
"""
from __future__ import annotations

HBM_PEAK_GBPS = 8000.0  # MI355X HBM3E, AMD's published figure

_Q = 4  # quadrants


def _t(N: int, n: int, iv: int) -> float:
    return _Q * iv * 4.0 ** N * (1.0 + 2.0 ** -n)


def _r(N: int, ch: int = 1) -> float:
    return _Q * 4.0 * ch * 4.0 ** N


def _forward(N: int, iv: int, ch: int, keep: bool, with_f: bool):
    SS = 4.0 ** N
    rgb, rgb_f32 = ch == 3, ch == 3 and iv == 16
    fields = 4 * (ch + 1) * SS  # the emission planes and sigma
    out = [("hrc_seed", [("seed", -1)], fields + _t(N, 2, iv))]
    top = min(3 if rgb else 4, N - 2)
    n_top = N - top
    pairs = not rgb_f32 or (not keep and N >= 10)
    n = 2
    while n < n_top:
        g = min(n_top - n, 3 if rgb else 4)
        if n_top - n - g == 1 and g > 2:
            g -= 1
        stored = [j for j in range(1, g + 1)
                  if keep or j == g or not pairs or (n_top - n - j) % 2 == 0]
        out.append(("hrc_fuse_up" if g > 1 else "hrc_merge_up",
                    [("merge_up", n + j) for j in range(1, g + 1)],
                    _t(N, n, iv) + sum(_t(N, n + j, iv) for j in stored)))
        n += g
    kept = sum(_t(N, j, iv) + _r(N, ch) for j in range(n_top + 1, N)) if keep else 0.0
    out.append(("hrc_fuse_top" if top > 1 else "hrc_merge_down",
                [("merge_up", j) for j in range(n_top + 1, N)] +
                [("merge_down", j) for j in range(N - 1, n_top - 1, -1)],
                _t(N, n_top, iv) + _r(N, ch) + kept))
    n = n_top
    while n > 2:
        if n >= 4 and pairs:
            n -= 2
            out.append(("hrc_fuse_down", [("merge_down", n + 1), ("merge_down", n)],
                        _t(N, n, iv) + (3 if keep else 2) * _r(N, ch)))
        else:
            # half of T_n (odd columns) and the even directions of T_{n+1}
            n -= 1
            out.append(("hrc_merge_down", [("merge_down", n)], _t(N, n, iv) + 2 * _r(N, ch)))
    out.append(("hrc_tail", [("tail", -1) if with_f else ("merge_down", 1)],
                fields + _r(N, ch) * (2 if keep else 1) + (4 * ch * SS if with_f else 0.0)))
    return out


def forward_launches(N: int, iv: int = 8, keep: bool = False):
    return _forward(N, iv, 1, keep, True)


def backward_launches(N: int):
    """hrc_backward: the forward recomputed down to R_1 (every level stored) and
    the reverse."""
    SS = 4.0 ** N
    out = _forward(N, 8, 1, True, False)
    # sigma and dLoss/dF read, dR_0 .. dR_2 (dR_{N-1} at 8^2: N - 1 = 2) written
    out.append(("hrc_tail_adj", [("gather_adj", -1), ("merge_down_adj", 0), ("merge_down_adj", 1)],
                8 * SS + 3 * _r(N)))
    n = 2
    while n + 1 < N:
        g = 2 if n + 2 <= N - 1 else 1
        # dR_n and the transmittances (4 bytes) of T_n read
        out.append(("hrc_fuse_dr" if g == 2 else "hrc_merge_down_adj",
                    [("merge_down_adj", n + j) for j in range(g)],
                    _r(N) + _t(N, n, 4) + g * _r(N)))
        n += g
    for n in range(N, -1, -1):
        b = _t(N, n, 8) if n else _t(N, 0, 4)  # dT_n written (dT_0 at odd columns)
        if 3 <= n + 1 <= N:
            b += _t(N, n, 8) + _t(N, n + 1, 8)  # T_n and dT_{n+1}
        if n < N:
            b += _r(N)  # odd columns of dR_n and R_{n+1}
        if n >= 1:
            b += _r(N)  # even columns of dR_{n-1} and R_n
        out.append(("hrc_interval_adj", [("interval_adj", n)], b))
    # the fields and dT_0 .. dT_2 read, d eps and d sigma written
    out.append(("hrc_seed_adj", [("seed_adj", -1)],
                16 * SS + _t(N, 0, 4) + _t(N, 1, 8) + _t(N, 2, 8)))
    return out


def forward_bytes(N: int, iv: int = 8) -> float:
    return sum(b for _, _, b in forward_launches(N, iv))


def backward_bytes(N: int) -> float:
    return sum(b for _, _, b in backward_launches(N))


def forward_bytes_rgb(N: int, iv: int = 16) -> float:
    """hrc_forward_rgb: intervals (L_r, L_g, L_b, T) of ``iv`` bytes, cascade
    levels, emission and fluence as three planes."""
    return sum(b for _, _, b in _forward(N, iv, 3, False, True))


def group_launches(launches, passes):
    """Per-pass profile rows (name, level, ms), in order, as per-kernel totals:
    {kernel: (launches, ms, bytes)}."""
    rows = iter(passes)
    out: dict[str, tuple[int, float, float]] = {}
    for kernel, covers, nbytes in launches:
        ms = 0.0
        for want in covers:
            name, n, t = next(rows)
            if (name, n) != want:
                raise ValueError(f"pass {(name, n)} where {want} was expected")
            ms += t
        c, m, b = out.get(kernel, (0, 0.0, 0.0))
        out[kernel] = (c + 1, m + ms, b + nbytes)
    if next(rows, None) is not None:
        raise ValueError("more passes than the launches cover")
    return out
