"""The collisions with every relaxation group at its own rate, one step from
noise far from equilibrium on a periodic box, against the oracle (FP64, 1e-12
of the largest population: rounding order only, the bar of the step parity)."""
import pytest

import synth
from lbm_cases import gpu_lattice, oracle_lattice, rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("name,rates,cs", [
    ("mrt_table1", (1.1, 0.8, 1.3, 0.7), 0.15),
    ("mrt_table1", (1.1, 0.8, 1.3, 0.7), 0.0),
    ("mrt_dhumieres", (1.1, 0.7, 1.3, 0.8, 1.9), 0.15),
    ("fclb", None, 0.0),
    ("clb", None, 0.0),
])
def test_distinct_rates_against_the_oracle(name, rates, cs):
    shape = (9, 7, 8)
    nx, ny, nz = shape
    g = gpu_lattice(name, "f64", shape, 0.02, cs=cs, rates=rates)
    o = oracle_lattice(name, shape, 0.02, cs=cs, rates=rates)
    f = synth.random_populations(g.Q, (nz, ny, nx), 3e-2, seed=17)
    g.set_populations(torch.from_numpy(f))
    print("case rates", name, rates, cs, flush=True)
    g.step(1)
    assert rel_err(g.populations().cpu().numpy(), o.run(f, 0, 1)) <= 1e-12
