"""Steps over workgroups of 256 consecutive nodes, where that split can go
wrong: fewer nodes than a workgroup, exactly one, one node more, rows that
straddle workgroups, node counts that leave an XCD without work, odd counts
and odd rows in FP16 (two nodes per lane), y faces whose rows are left out of
the wall rows; and lattices beyond the last-level cache with and without whole
memory lines, as a small pattern repeated over the box.

Bars: those of the step parity and of the full-size tests, per step of the
largest population: FP64 1e-12, FP32 4e-6, FP16 2e-3; the oracle starts from
the state as it is stored."""
import numpy as np
import pytest

import synth
from lbm_cases import F, I, O, P, W, face_velocities, gpu_lattice, oracle_lattice, rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

TOL = {"f64": 1e-12, "f32": 4e-6, "f16": 2e-3}
ROUND = {"f64": np.float64, "f32": np.float32, "f16": np.float16}
BOX = [W, W, W, W, I, O]
SLIP_Y = [P, P, F, W, I, O]


def start(Q, shape, storage, seed):
    nx, ny, nz = shape
    f = synth.random_populations(Q, (nz, ny, nx), 1e-2, seed=seed)
    return f.astype(ROUND[storage]).astype(np.float64)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
@pytest.mark.parametrize("shape,faces", [
    ((5, 4, 3), None), ((16, 4, 4), None), ((257, 1, 1), None), ((37, 5, 7), None),
    ((130, 3, 6), None), ((13, 11, 9), None), ((31, 9, 11), BOX), ((30, 9, 7), BOX),
    ((64, 6, 9), SLIP_Y), ((21, 7, 3), SLIP_Y), ((9, 8, 2), BOX)])
def test_split_of_the_nodes(storage, shape, faces):
    nx, ny, nz = shape
    kw = {}
    if faces is not None:
        fu = face_velocities(0.002)
        kw = dict(faces=faces, face_u=fu, inlet=synth.jet_inlet(nx, ny, 3.0, 0.05, 0.002))
    for name in ("fclb", "mrt_table1"):
        g = gpu_lattice(name, storage, shape, 0.02, **kw)
        o = oracle_lattice(name, shape, 0.02, **kw)
        f = start(g.Q, shape, storage, 5)
        g.set_populations(torch.from_numpy(f))
        print("case split", name, storage, shape, flush=True)
        for n in (1, 2):  # an even step, then an odd and an even one
            g.step(n)
        got = g.populations().cpu().numpy()
        assert rel_err(got, o.run(f, 0, 3)) <= 3 * TOL[storage], name


@pytest.mark.parametrize("name,storage,shape,part", [
    ("fclb", "f64", (112, 112, 112), (14, 14, 14)),    # whole lines
    ("fclb", "f64", (110, 112, 112), (11, 14, 14)),    # whole per population, not per row
    ("fclb", "f64", (111, 117, 111), (37, 13, 111)),   # neither
    ("mrt_table1", "f32", (160, 152, 152), (16, 8, 8)),
    ("fclb", "f32", (133, 143, 133), (19, 13, 133)),
    ("fclb", "f16", (192, 164, 162), (16, 4, 9)),
    ("fclb", "f16", (171, 173, 171), (9, 173, 9)),     # an odd count: one node per lane
])
@pytest.mark.parametrize("walls", [False, True])
def test_beyond_the_last_level_cache(name, storage, shape, part, walls):
    if walls:  # on z, so the pattern repeats along x and y only
        part = (part[0], part[1], shape[2])
    kw = dict(faces=[P, P, P, P, W, W], face_u=face_velocities(0.002, axis=0)) if walls else {}
    g = gpu_lattice(name, storage, shape, 0.02, **kw)
    o = oracle_lattice(name, part, 0.02, **kw)
    assert shape[0] * shape[1] * shape[2] * g.Q * {"f64": 8, "f32": 4, "f16": 2}[storage] > 2**28
    f = start(g.Q, part, storage, 7)
    reps = (1, shape[2] // part[2], shape[1] // part[1], shape[0] // part[0])
    dev = torch.from_numpy(f).cuda().repeat(reps).contiguous()
    print("case large", name, storage, shape, walls, flush=True)
    g.set_populations(dev)
    del dev
    g.step(3)
    ref = torch.from_numpy(np.ascontiguousarray(o.run(f, 0, 3))).cuda()
    got = g.populations()
    worst = 0.0
    for q in range(g.Q):
        d = got[q].double() - ref[q].repeat(reps[1:])
        worst = max(worst, float(d.abs().max()))
    assert worst <= 3 * TOL[storage] * float(ref.abs().max())
