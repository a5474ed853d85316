"""Bits of the closure-off timestep with FP32 arithmetic.

The collision is evaluated as written: every FP32 operation rounds once, the
multiply-adds spelled out in it fuse, and the result is then rounded to the
storage type, for FP16 too (rounding a multiply-add straight to FP16 would skip the
FP32 rounding and change about one stored value in a thousand per step).  The same
operations here in FP64, each rounded to FP32: exact for +, *, / (53 >= 2 * 24 + 2
digits) and, for a multiply-add, but for a double rounding about once in 2^29
operations, some 1e6 of which are compared; so the states must be equal
(tolerance 0).
"""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NU, ETA, GHOST, BREF = 2e-3, 3e-3, (1.6, 1.4, 1.2, 1.7), 0.01
CX = [0, 1, 0, -1, 0, 1, -1, -1, 1]
CY = [0, 0, 1, 0, -1, 1, 1, -1, -1]
W9 = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
W5 = [1 / 3] + [1 / 6] * 4


def _r(x):
    """Rounded to FP32, held in FP64."""
    return x.float().double() if isinstance(x, torch.Tensor) else float(torch.tensor(x, dtype=torch.float64).float())


def _fma(a, b, c):
    return _r(a * b + c)


def _collide(v, swapped):
    """Post-collision deviations of v [19, ny, nx] (sums in the kernels' order)."""
    s3, sm = 2.0 / (6.0 * NU + 1.0), _r(2.0 / (6.0 * ETA + 1.0))
    r3 = _r(s3 / 4.0)
    r5, r6, r7, r8 = (_r(g / n) for g, n in zip(GHOST, (12.0, 12.0, 180.0, 20.0)))
    add = lambda *a: a[0] if len(a) == 1 else _r(add(*a[:-1]) + a[-1])  # noqa: E731
    f = v[:9]
    drho = add(add(add(add(f[0], f[1]), add(f[2], f[3])), add(add(f[4], f[5]), add(f[6], f[7]))), f[8])
    mx = add(add(add(f[1], -f[3]), add(f[5], -f[6])), add(f[8], -f[7]))
    my = add(add(add(f[2], -f[4]), add(f[5], -f[7])), add(f[6], -f[8]))
    dbx = add(add(add(v[9], v[10]), add(v[11], v[12])), v[13])
    dby = add(add(add(v[14], v[15]), add(v[16], v[17])), v[18])
    ir = _r(1.0 / _r(1.0 + drho))
    bx, by = _r(_r(BREF) + dbx), dby
    d56, d78, s56, s78 = add(f[5], -f[6]), add(f[7], -f[8]), add(f[5], f[6]), add(f[7], f[8])
    s14, s58 = add(add(f[1], f[2]), add(f[3], f[4])), add(s56, s78)
    M3, M4 = add(d56, d78), add(add(f[1], f[3]), -add(f[2], f[4]))
    M5 = add(_fma(2.0, add(f[3], -f[1]), d56), -d78)
    M6 = add(_fma(2.0, add(f[4], -f[2]), s56), -s78)
    M7 = _fma(4.0, s58, _fma(4.0, f[0], _r(-5.0 * s14)))
    M8 = _fma(4.0, f[0], -s58)
    q2 = _r(_fma(mx, mx, _r(my * my)) * ir)
    e3 = _fma(_r(mx * my), ir, -_r(bx * by))
    e4 = _fma(_fma(mx, mx, -_r(my * my)), ir, -_fma(bx, bx, -_r(by * by)))
    m3, m5, m6, m7 = add(M3, -e3), add(M5, mx), add(M6, my), _fma(3.0, q2, M7)
    m8 = add(M8, -_fma(_r(5.0 / 3.0), drho, _r(-3.0 * q2)))
    d4, d5, d6, d7, d8 = (_r(a * b) for a, b in ((r3, add(M4, -e4)), (r5, m5), (r6, m6), (r7, m7), (r8, m8)))
    h = _fma(4.0, d7, -d8)
    o = [None] * 19
    o[0] = _fma(-4.0, torch.where(swapped, _fma(r7, m7, d8), _fma(r8, m8, d7)), f[0])
    o[1] = add(f[1], -_fma(-5.0, d7, _fma(-2.0, d5, d4)))
    o[2] = add(f[2], -_fma(-5.0, d7, _fma(-2.0, d6, -d4)))
    o[3] = add(f[3], -_fma(-5.0, d7, _fma(2.0, d5, d4)))
    o[4] = add(f[4], -_fma(-5.0, d7, _fma(2.0, d6, -d4)))
    o[5] = add(f[5], -add(_fma(r6, m6, _fma(r3, m3, d5)), h))
    o[6] = add(f[6], -add(_fma(-r5, m5, _fma(-r3, m3, d6)), h))
    o[7] = add(f[7], -add(_fma(-r6, m6, _fma(r3, m3, -d5)), h))
    o[8] = add(f[8], -add(_fma(-r6, m6, _fma(-r3, m3, d5)), h))
    E = _r(_fma(mx, by, -_r(my * bx)) * ir)
    bxp, bxm, byp, bym = _fma(3.0, E, dbx), _fma(-3.0, E, dbx), _fma(3.0, E, dby), _fma(-3.0, E, dby)
    for i in range(5):
        w = _r(W5[i])
        o[9 + i] = _fma(-sm, _fma(-w, dbx if CY[i] == 0 else (bxm if CY[i] > 0 else bxp), v[9 + i]), v[9 + i])
        o[14 + i] = _fma(-sm, _fma(-w, dby if CX[i] == 0 else (byp if CX[i] > 0 else bym), v[14 + i]), v[14 + i])
    return o


@pytest.mark.parametrize("dtype", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("schedule", ["fused", "aa"])
@pytest.mark.parametrize("nx,ny", [(64, 48), (61, 50), (62, 49)])
def test_one_step(nx, ny, schedule, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1705_09807_amd import Sim
    print("rounding", nx, ny, schedule, dtype, flush=True)
    s = Sim(nx=nx, ny=ny, nu=NU, eta=ETA, s5=GHOST[0], s6=GHOST[1], s7=GHOST[2], s8=GHOST[3], dtype=dtype,
            schedule=schedule, b_ref=(BREF, 0.0))
    g = torch.Generator(device="cuda").manual_seed(nx * 7 + ny)
    m = 0.02 * (2 * torch.rand(5, ny, nx, generator=g, device="cuda", dtype=torch.float64) - 1)
    m[0] += 1.0
    m[3] += BREF
    s.init_from_moments(m)
    rest = torch.tensor(W9 + [w * BREF for w in W5] + [0.0] * 5, device="cuda", dtype=torch.float64)[:, None, None]

    def stored(a):
        # the deviations as the storage type holds them, in FP64
        if dtype == "fp32":
            return a.float().double()
        return (a.float() * 256).half().double() / 256 if dtype == "fp16" else a.float().bfloat16().double()

    before = stored(s.get_state() - rest)
    # 16-bit rows of a multiple of four columns, two-buffer schedule: one column in four sums
    # the two products of its rest population in the other order
    swapped = torch.zeros(nx, dtype=torch.bool, device="cuda")
    if dtype != "fp32" and schedule == "fused" and nx % 4 == 0:
        swapped[(1 if dtype == "bf16" else 2)::4] = True
    for _ in range(3):
        s.step(1)
        o = torch.stack([stored(a) for a in _collide(before, swapped)])
        before = torch.stack([torch.roll(o[q], (cy, cx), (0, 1)) for q, (cx, cy) in
                              enumerate(list(zip(CX, CY)) + list(zip(CX[:5], CY[:5])) * 2)])
        assert torch.equal(stored(s.get_state() - rest), before)
