"""Sweeps of several timesteps per launch against one-step sweeps (bit for bit, tolerance
0: see test_gpu_multistep.py), each case with a number of steps per launch that it has
to take: groups of 256 columns with the closure off in every storage type, strips of whole
sectors, two workgroups per compute unit, and 16-bit storage with the closure on at two
and at three steps."""

import pytest
from launch_plan import launch_plan

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# nx, ny, steps, a launch of so many steps among them, run
CASES = [(nx, ny, n, 4, dict(dtype=d, delta=0.0)) for d in ("fp32", "fp16", "bf16")
         for nx, ny, n in ((1021, 1030, 8), (1448, 1501, 11))]
CASES += [(nx, ny, n, k, dict(dtype="fp64", delta=0.0)) for nx, ny, n, k in ((1021, 1030, 7, 3), (1504, 700, 2, 2))]
CASES += [(4099, 2050, 5, 3, dict(dtype="fp32", delta=0.0)), (4100, 2050, 4, 4, dict(dtype="fp32", delta=0.0))]
CASES += [(8000, 4099, 4, 4, dict(dtype="bf16", delta=0.0)), (8000, 4097, 3, 3, dict(dtype="bf16", delta=4.0)),
          (8001, 4097, 2, 2, dict(dtype="fp16", delta=4.0))]
CASES += [(1203, 1201, 6, 3, dict(dtype=d, delta=4.0, grad_stencil=s)) for d in ("fp16", "bf16")
          for s in ("iso9", "central5", "local_iso9", "local_central5")]
CASES += [(1003, 1050, 2, 2, dict(dtype=d, delta=4.0, grad_stencil=s)) for d in ("fp16", "bf16")
          for s in ("iso9", "central5", "local_iso9", "local_central5")]
CASES += [(1203, 1201, 6, 3, dict(dtype="fp16", delta=3.0, closure="full")),
          (701, 703, 4, 2, dict(dtype="bf16", delta=3.0, closure="full", grad_stencil="central5"))]
CASES += [(66, 6001, 5, 3, dict(dtype="fp32", delta=4.0)), (40, 9001, 3, 3, dict(dtype="fp32", delta=3.0, mag_lattice="d2q9")),
          (32768, 20, 4, 2, dict(dtype="fp64", delta=4.0))]
CASES += [(1003, 1000, 6, 4, dict(dtype="fp32", delta=0.0, schedule="aa")),
          (1024, 1000, 2, 2, dict(dtype="fp32", delta=0.0, schedule="aa")),
          (1003, 1000, 5, 2, dict(dtype="fp32", delta=4.0, schedule="aa")),
          (1003, 1000, 5, 2, dict(dtype="fp32", delta=4.0, schedule="aa_lagged"))]


@pytest.mark.parametrize("nx,ny,n,k,kw", CASES)
def test_equals_one_step_sweeps(nx, ny, n, k, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1705_09807_amd import Sim
    print("plan", nx, ny, n, k, kw, flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert k in launch_plan(nx, ny, n, cus=cus, **kw)
    m = 0.02 * (2 * torch.rand(5, ny, nx, generator=torch.Generator(device="cuda").manual_seed(nx * 7 + ny),
                               device="cuda", dtype=torch.float64) - 1)
    m[0] += 1.0
    m[3] += 0.01
    states = []
    for calls in ([n], [1] * n):
        s = Sim(nx=nx, ny=ny, nu=2e-3, eta=3e-3, s5=1.6, s6=1.4, s7=1.2, s8=1.7, b_ref=(0.01, 0.0), **kw)
        s.init_from_moments(m)
        for c in calls:
            s.step(c)
        states.append(s.get_state())
        s.close()
    assert torch.isfinite(states[1]).all()
    assert torch.equal(*states)
