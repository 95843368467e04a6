"""Populations, density and velocity, sums and running statistics read after
an even and an odd number of steps, at sizes where the readout kernels can go
wrong: fewer nodes than a workgroup, one node past a workgroup, node counts
that are not a multiple of what a lane copies, waves with and without a node
on a face of each kind, solids on even and odd states, more tiles than the
reduction has blocks, and a lattice beyond the last-level cache.

The populations are held to the oracle (FP64, the step parity's 1e-12 of the
largest; FP32 4e-6 and FP16 2e-3 per step). The other readouts are functions
of the populations read in FP64: density and velocity differ by the rounding
of their sums only, 64 units of FP64 (27 terms, twice, and a division), or
half a unit of FP32 where the fields are FP32; sums over N nodes by N units
of the sum of magnitudes at most, in any order."""
import numpy as np
import pytest

import paper_1206_0389_amd as Pk
import synth
from lbm_cases import F, I, O, P, PR, W, face_velocities, gpu_lattice, oracle_lattice, rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

TOL = {"f64": 1e-12, "f32": 4e-6, "f16": 2e-3}
ROUND = {"f64": np.float64, "f32": np.float32, "f16": np.float16}
U64 = 2.0**-53
FACES = {"periodic": None, "jet": [W, W, W, W, I, O], "walls_y": [P, P, W, W, P, P],
         "slip": [W, W, F, W, I, O], "x_pressure": [PR, PR, P, P, W, O]}


def fields(g, f):
    """Density deviation, velocity and sums of populations f (FP64, on the GPU)."""
    e = torch.tensor(np.array(Pk.VELOCITIES[:g.Q]), dtype=torch.float64, device="cuda")
    d = f.sum(0)
    j = torch.stack([(f * e[:, a].reshape(-1, 1, 1, 1)).sum(0) for a in range(3)])
    return d, j, j / (1.0 + d) if g.Q == 27 else j


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("name", ["fclb", "mrt_table1"])
@pytest.mark.parametrize("shape,layout,solid", [
    ((5, 4, 3), "periodic", False), ((257, 1, 1), "periodic", False),
    ((43, 6, 5), "jet", False), ((64, 9, 7), "jet", True), ((130, 5, 4), "walls_y", False),
    ((21, 8, 9), "slip", False), ((18, 7, 8), "x_pressure", False),
    ((70, 64, 60), "jet", False), ((66, 62, 65), "periodic", True)])
def test_readouts_at_both_parities(name, storage, shape, layout, solid):
    nx, ny, nz = shape
    kw = {}
    if FACES[layout] is not None:
        kw = dict(faces=FACES[layout], face_u=face_velocities(0.002),
                  face_drho=[0.001, -0.001, 0, 0, 0, 0])
        if I in FACES[layout]:
            kw["inlet"] = synth.jet_inlet(nx, ny, 3.0, 0.05, 0.002)
    g = gpu_lattice(name, storage, shape, 0.02, **kw)
    mask = np.zeros((nz, ny, nx), dtype=np.uint8)
    if solid:
        mask[1:3, 1:4, 2:5] = 1
        g.set_solids(torch.from_numpy(mask))
    f = synth.random_populations(g.Q, (nz, ny, nx), 1e-2, seed=3)
    f = f.astype(ROUND[storage]).astype(np.float64)
    g.set_populations(torch.from_numpy(f))
    print("case readout", name, storage, shape, layout, solid, flush=True)
    sums = g.stats_buffer()
    S = [torch.zeros((3, nz, ny, nx), dtype=torch.float64, device="cuda") for _ in range(2)]
    o = None if solid else oracle_lattice(name, shape, 0.02, **kw)
    for t in (1, 2):
        g.step(1)
        p = g.populations(torch.float64)
        assert torch.equal(g.populations(torch.float32), p.to(torch.float32))
        if o is not None:
            assert rel_err(p.cpu().numpy(), o.run(f, 0, t)) <= t * TOL[storage]
        else:
            assert float(p[:, torch.from_numpy(mask).cuda().bool()].abs().max()) == 0.0
        d, j, u = fields(g, p)
        top = float(p.abs().max()) * g.Q
        for dt, unit in ((torch.float64, 64 * U64), (torch.float32, 2.0**-24 * 1.01)):
            rho, v = g.macroscopic(dtype=dt)
            assert float((rho.double() - d).abs().max()) <= unit * (1.0 + top)
            assert float((v.double() - u).abs().max()) <= unit * top * 2
        s = np.array(g.reduce(check=False))
        rho1 = 1.0 + d if g.Q == 27 else torch.ones_like(d)
        ref = [d, j[0], j[1], j[2], 0.5 * (j * j).sum(0) / rho1]
        for k in range(5):
            bar = (64 + d.numel()) * U64 * float(ref[k].abs().sum() + top * 64)
            assert abs(s[k] - float(ref[k].sum())) <= bar, k
        g.stats_accumulate(sums)
        S[0] += u
        S[1] += u * u
        got = sums.reshape(6, nz, ny, nx)
        assert float((got[:3] - S[0]).abs().max()) <= t * 64 * U64 * top * 2
        assert float((got[3:] - S[1]).abs().max()) <= t * 256 * U64 * max(top, top * top)


@pytest.mark.parametrize("name,storage,shape", [("fclb", "f64", (111, 117, 111)),
                                                ("mrt_table1", "f32", (161, 153, 151)),
                                                ("fclb", "f16", (171, 173, 171))])
def test_readouts_beyond_the_last_level_cache(name, storage, shape):
    nx, ny, nz = shape
    g = gpu_lattice(name, storage, shape, 0.02)
    print("case readout large", name, storage, shape, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    f = 1e-2 * torch.randn((g.Q, nz, ny, nx), dtype=torch.float32, device="cuda", generator=gen)
    g.set_populations(f)
    stored = f.to({"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}[storage])
    assert torch.equal(g.populations(torch.float32), stored.to(torch.float32))
    d, _, u = fields(g, stored.double())
    top = float(stored.abs().max()) * g.Q
    rho, v = g.macroscopic(dtype=torch.float64)
    assert float((rho - d).abs().max()) <= 64 * U64 * (1.0 + top)
    assert float((v - u).abs().max()) <= 128 * U64 * top
    s = np.array(g.reduce(check=False))
    assert abs(s[0] - float(d.sum())) <= (64 + d.numel()) * U64 * float(d.abs().sum())
