"""Density, velocity, sums and statistics read with the streaming hint, which they take on
lattices more than a third larger than the last-level cache: node counts that
leave the last workgroup, lane and memory line partly used, at even parity.

Populations come back as they are stored; the other readouts are functions of
them and differ by the rounding of their sums only, 64 units of FP64 (27 terms,
twice, and a division), sums over N nodes by N units of the sum of magnitudes;
squares of velocities by four times the velocities' units."""
import pytest

from lbm_cases import gpu_lattice
from test_gpu_readouts import U64, fields

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("name,storage,shape", [("fclb", "f64", (121, 121, 119)),
                                                ("mrt_table1", "f32", (173, 171, 169)),
                                                ("fclb", "f16", (191, 193, 191))])
def test_readouts_with_the_hint(name, storage, shape):
    nx, ny, nz = shape
    g = gpu_lattice(name, storage, shape, 0.02)
    size = {"f64": 8, "f32": 4, "f16": 2}[storage]
    assert nx * ny * nz * g.Q * size > 4 / 3 * 2**28
    print("case readout hint", name, storage, shape, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(6)
    f = 1e-2 * torch.randn((g.Q, nz, ny, nx), dtype=torch.float32, device="cuda", generator=gen)
    g.set_populations(f)
    stored = f.to({"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}[storage])
    d, j, u = fields(g, stored.double())
    top = float(stored.abs().max()) * g.Q
    for dt, unit in ((torch.float64, 64 * U64), (torch.float32, 2.0**-24 * 1.01)):
        rho, v = g.macroscopic(dtype=dt)
        assert float((rho.double() - d).abs().max()) <= unit * (1.0 + top)
        assert float((v.double() - u).abs().max()) <= unit * top * 2
    s = g.reduce(check=False)
    for k, ref in enumerate([d, j[0], j[1], j[2]]):
        bar = (64 + ref.numel()) * U64 * float(ref.abs().sum() + top * 64)
        assert abs(s[k] - float(ref.sum())) <= bar, k
    sums = g.stats_buffer()
    g.stats_accumulate(sums)
    got = sums.reshape(6, nz, ny, nx)
    assert float((got[:3] - u).abs().max()) <= 128 * U64 * top
    assert float((got[3:] - u * u).abs().max()) <= 512 * U64 * max(top, top * top)
