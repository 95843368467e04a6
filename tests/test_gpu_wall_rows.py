"""Lattices whose only non-periodic faces are x or y walls: no row needs the
general rules, and steps and adjoint steps run the wall rows alone. Sizes with
fewer nodes than a workgroup, one node past a workgroup, and rows that
straddle workgroups; walls that move.

Bars: those of the step parity and of the adjoint step, per step of the
largest value: FP64 1e-12, FP32 4e-6 (adjoint 2e-5)."""
import numpy as np
import pytest

import synth
from lbm_cases import P, W, gpu_lattice, oracle_lattice, rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

TYPE = {"f64": np.float64, "f32": np.float32}
MOVING = [[0.0, 0.001, 0.002], [0.0, 0.0, 0.002], [0.001, 0.0, 0.002], [0.0, 0.0, 0.001],
          [0.0, 0.0, 0.0], [0.0, 0.0, 0.0]]
FACES = {"y": [P, P, W, W, P, P], "x": [W, W, P, P, P, P], "xy": [W, W, W, W, P, P]}
SHAPES = [(7, 5, 6), (2, 2, 65), (37, 9, 11), (300, 3, 2)]


def _pair(name, storage, shape, walls):
    kw = dict(faces=FACES[walls], face_u=MOVING)
    print("case wall rows", name, storage, shape, walls, flush=True)
    return gpu_lattice(name, storage, shape, 0.02, **kw), oracle_lattice(name, shape, 0.02, **kw)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("walls", list(FACES))
@pytest.mark.parametrize("shape", SHAPES)
def test_steps(storage, walls, shape):
    nx, ny, nz = shape
    for name in ("fclb", "clb", "mrt_table1", "mrt_dhumieres"):
        g, o = _pair(name, storage, shape, walls)
        f = synth.random_populations(g.Q, (nz, ny, nx), 1e-2, seed=4).astype(TYPE[storage])
        f = f.astype(np.float64)
        g.set_populations(torch.from_numpy(f))
        for n in (1, 3):  # an even step, then two odd ones round an even one
            g.step(n)
        assert rel_err(g.populations().cpu().numpy(), o.run(f, 0, 4)) <= (
            4e-12 if storage == "f64" else 1.6e-5), name


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("walls", list(FACES))
@pytest.mark.parametrize("shape", SHAPES)
def test_adjoint_steps(storage, walls, shape):
    nx, ny, nz = shape
    for name in ("fclb", "mrt_table1", "mrt_dhumieres"):
        g, o = _pair(name, storage, shape, walls)
        f = synth.random_populations(g.Q, (nz, ny, nx), 1e-2, seed=8).astype(TYPE[storage])
        ln = synth.random_populations(g.Q, (nz, ny, nx), 1.0, seed=9).astype(TYPE[storage])
        ref = o.adjoint_step(f.astype(np.float64), ln.astype(np.float64), np.zeros((3, 1, 1)))
        ft, lt = torch.from_numpy(f).cuda(), torch.from_numpy(ln).cuda()
        out = torch.empty_like(ft)
        g.adjoint_step(ft, lt, out, None)
        assert rel_err(out.cpu().numpy(), ref) <= (1e-12 if storage == "f64" else 2e-5), name
