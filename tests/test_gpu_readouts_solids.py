"""Readouts beside solid nodes: populations of fluid nodes against the oracle
with the same mask after an even and an odd number of steps (the wall rules'
odd-parity pull with solids, in waves with and without a node on a face), and
the copy of populations at even parity on lattices beyond the last-level
cache, exactly what is stored outside the body and zero inside.

Bars against the oracle: those of the step parity, FP64 1e-12, FP32 4e-6 and
FP16 2e-3 per step of the largest population."""
import numpy as np
import pytest

import oracle
import synth
from lbm_cases import I, MODELS, O, P, W, face_velocities, gpu_lattice

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

TOL = {"f64": 1e-12, "f32": 4e-6, "f16": 2e-3}
TYPE = {"f64": np.float64, "f32": np.float32, "f16": np.float16}
FACES = {"periodic": None, "jet": [W, W, W, W, I, O], "walls_y": [P, P, W, W, P, P]}


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("name", ["fclb", "mrt_table1"])
@pytest.mark.parametrize("shape,layout", [((64, 9, 7), "jet"), ((66, 62, 5), "periodic"),
                                          ((70, 30, 11), "walls_y"), ((257, 4, 6), "jet")])
def test_populations_beside_solids(name, storage, shape, layout):
    nx, ny, nz = shape
    kw, okw = {}, {}
    if FACES[layout] is not None:
        kw = dict(faces=FACES[layout], face_u=face_velocities(0.002))
        okw = dict(kw)
        if I in FACES[layout]:
            kw["inlet"] = synth.jet_inlet(nx, ny, 3.0, 0.05, 0.002)
            okw.update(inlet_u=kw["inlet"][0], inlet_mask=kw["inlet"][1])
    solid = np.zeros((nz, ny, nx), np.uint8)
    solid[1:4, 1:3, 2:6] = 1           # beside a y face
    solid[2, 0, nx - 4:nx - 1] = 1     # on it
    solid[nz // 2, ny // 2, ::7] = 1   # single nodes in many waves
    fluid = solid == 0
    g = gpu_lattice(name, storage, shape, 0.02, **kw)
    g.set_solids(torch.from_numpy(solid))
    o = oracle.Lattice(MODELS[name][0], nx, ny, nz, nu=0.02, basis=MODELS[name][1], solid=solid,
                       **okw)
    f = synth.random_populations(g.Q, (nz, ny, nx), 1e-2, seed=12)
    f = f.astype(TYPE[storage]).astype(np.float64)
    g.set_populations(torch.from_numpy(f))
    print("case readout solids", name, storage, shape, layout, flush=True)
    for t in (0, 1, 2, 3):
        if t:
            g.step(1)
        ref = o.run(f, 0, t) if t else f
        p = g.populations(torch.float64)
        got = p.cpu().numpy()
        err = np.abs(got[:, fluid] - ref[:, fluid]).max() / np.abs(ref[:, fluid]).max()
        assert err <= t * TOL[storage], t
        assert np.all(got[:, ~fluid] == 0.0)
        assert torch.equal(g.populations(torch.float32), p.to(torch.float32))


@pytest.mark.parametrize("name,storage,shape", [("fclb", "f32", (143, 141, 139)),
                                                ("mrt_table1", "f32", (161, 153, 151)),
                                                ("fclb", "f64", (111, 117, 111)),
                                                ("fclb", "f16", (171, 173, 171))])
def test_copy_with_solids_beyond_the_cache(name, storage, shape):
    nx, ny, nz = shape
    g = gpu_lattice(name, storage, shape, 0.02, faces=FACES["walls_y"],
                    face_u=face_velocities(0.002))
    assert nx * ny * nz * g.Q * np.dtype(TYPE[storage]).itemsize > 2**28
    print("case readout solids large", name, storage, shape, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(8)
    solid = torch.rand((nz, ny, nx), device="cuda", generator=gen) < 0.2
    g.set_solids(solid.to(torch.uint8))
    f = 1e-2 * torch.randn((g.Q, nz, ny, nx), dtype=torch.float32, device="cuda", generator=gen)
    g.set_populations(f)
    want = f.to({"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}[storage])
    want = torch.where(solid, torch.zeros_like(want), want)
    assert torch.equal(g.populations(torch.float32), want.to(torch.float32))
    assert torch.equal(g.populations(torch.float64), want.to(torch.float64))
