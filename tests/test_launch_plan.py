"""How many timesteps each launch of a step call takes (host side of the library)."""

import pytest
import test_gpu_launch_plan as G
import test_gpu_multistep as M
from launch_plan import launch_plan

DTYPES = ["fp64", "fp32", "fp16", "bf16"]
GRIDS = [(4, 4), (15, 400), (16, 16), (64, 64), (64, 8000), (512, 512), (724, 724), (1024, 1024), (1000, 1048),
         (2048, 2048), (32768, 20), (4096, 4096)]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kw", [dict(delta=0.0), dict(delta=2.0), dict(delta=2.0, grad_stencil="local_iso9"),
                                dict(delta=2.0, closure="full"), dict(delta=2.0, closure="learned")])
@pytest.mark.parametrize("nx,ny", GRIDS)
def test_fused(nx, ny, kw, dtype):
    for n in (0, 1, 2, 3, 5, 7, 10, 23, 24, 25, 26, 27, 28, 100, 101):
        p, q = launch_plan(nx, ny, n, dtype=dtype, **kw), launch_plan(nx, ny, n, dtype=dtype, recorded=True, **kw)
        assert sum(p) == sum(q) == n and all(1 <= k <= 4 for k in p + q)
        # a graph replays on the buffer that it was recorded on
        assert (n - len(q)) % 2 == 0
        if nx < 16 or ny < 16 or kw.get("closure") == "learned":
            assert len(p) == n


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("schedule,delta", [("aa", 0.0), ("aa", 2.0), ("aa_lagged", 2.0)])
def test_in_place(schedule, delta, dtype):
    for n in (1, 2, 3, 5, 9, 10):
        for t in (0, 1, 2, 3):
            p = launch_plan(4100, 2050, n, t=t, dtype=dtype, schedule=schedule, delta=delta)
            assert sum(p) == n
            at = t
            for k in p:
                assert k == 1 or (k % 2 == 0 and at % 2 == 0)
                at += k
            assert launch_plan(200, 200, n, t=t, dtype=dtype, schedule=schedule, delta=delta) == [1] * n


@pytest.mark.parametrize("dtype,schedule,delta,nx,ny,n,want", [
    # as measured on both sides: FP32 from 10^6 cells, not on strips of few columns
    ("fp32", "aa", 0.0, 1024, 1024, 4, [4]), ("fp32", "aa", 0.0, 1024, 1024, 6, [4, 2]),
    ("fp32", "aa", 2.0, 1024, 1024, 4, [2, 2]), ("fp32", "aa_lagged", 2.0, 5000, 201, 4, [2, 2]),
    ("fp32", "aa", 2.0, 990, 1000, 2, [1, 1]), ("fp32", "aa_lagged", 2.0, 64, 24000, 2, [1, 1]),
    ("fp32", "aa", 2.0, 128, 9000, 2, [1, 1]), ("fp32", "aa", 2.0, 128, 20000, 2, [2]),
    ("fp32", "aa", 0.0, 128, 20000, 6, [4, 1, 1]), ("fp64", "aa", 0.0, 64, 24000, 2, [1, 1]),
    # two steps of 16-bit storage with the closure off are slower than one and one
    ("bf16", "aa", 0.0, 4096, 4096, 6, [4, 1, 1]), ("fp16", "aa", 0.0, 4096, 4096, 2, [1, 1]),
    ("bf16", "aa", 2.0, 128, 32768, 2, [1, 1]), ("bf16", "aa_lagged", 2.0, 128, 32768, 2, [2])])
def test_in_place_sizes(dtype, schedule, delta, nx, ny, n, want):
    assert launch_plan(nx, ny, n, dtype=dtype, schedule=schedule, delta=delta) == want


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_grids_alike_take_alike_launches(dtype):
    """Closure off, about 2^20 cells: no shape keeps to one step."""
    plans = [launch_plan(nx, ny, 12, dtype=dtype, delta=0.0)
             for nx, ny in ((1000, 1048), (1024, 1000), (1024, 1024), (1040, 1010), (2048, 512), (5000, 201))]
    assert plans == [[4, 4, 4]] * len(plans)


# measured slower in sweeps of two or three steps than in as many of one (16-bit, in the caches)
@pytest.mark.parametrize("nx,ny,n,kw,want", [
    (512, 512, 2, dict(delta=0.0), [1, 1]), (512, 512, 5, dict(delta=0.0), [1, 4]),
    (724, 724, 2, dict(delta=0.0), [1, 1]),
    (1024, 1024, 2, dict(delta=2.0), [1, 1]), (1024, 1024, 5, dict(delta=2.0), [1] * 5),
    (1024, 1024, 5, dict(delta=2.0, closure="full"), [1] * 5),
    (1024, 1024, 2, dict(delta=2.0, grad_stencil="local_iso9"), [1, 1]),
    (64, 8000, 12, dict(delta=2.0), [1] * 12), (32768, 20, 4, dict(delta=0.0), [1] * 4)])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_short_calls(nx, ny, n, kw, want, dtype):
    assert sorted(launch_plan(nx, ny, n, dtype=dtype, **kw)) == want


def test_cases_of_several_steps_take_them():
    """The equality tests compare sweeps of several steps with one-step sweeps, not the latter with themselves."""
    def steps(nx, ny, n, **kw):
        return max(launch_plan(nx, ny, n, **kw) + launch_plan(nx, ny, 3, t=n, **kw))

    for nx, ny, n, k, kw in G.CASES:
        assert k in launch_plan(nx, ny, n, **kw), (nx, ny, n, k, kw)
    for dtype in DTYPES:
        for nx, ny, n in M.SMALL + [(600, 517, 11), (4100, 80, 13)]:
            assert steps(nx, ny, n, dtype=dtype, delta=0.0) > 1, (nx, ny, n, dtype)
        for nx, ny, n in M.IN_PLACE[:4]:
            for schedule, delta in (("aa", 0.0), ("aa", 4.0), ("aa_lagged", 4.0)):
                assert steps(nx, ny, n, dtype=dtype, schedule=schedule, delta=delta) > 1, (nx, ny, n, dtype, schedule)
    on = dict(fp64=M.FP64_LES, fp32=M.FP32_LES, fp16=M.LOW_LES, bf16=M.LOW_LES)
    for dtype, cases in on.items():
        for nx, ny, n in cases:
            if nx > 16:  # one 64-column strip keeps to one step
                assert steps(nx, ny, n, dtype=dtype, delta=4.0) > 1, (nx, ny, n, dtype)


@pytest.mark.parametrize("dtype", DTYPES)
def test_work_room_of_the_fused_schedule(dtype):
    """Reduction partials alone: nothing per cell."""
    from paper_1705_09807_amd.sim import make_params, work_bytes
    assert work_bytes(make_params(4096, 4096, 1e-3, 1e-3, delta=4.0, dtype=dtype)) < 1 << 20
