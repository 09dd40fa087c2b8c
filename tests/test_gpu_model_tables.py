"""Generic models with transition tables of every length class on the GPU,
against the oracle: no transition, one to sixteen (the kernels for at most
eight and for more, groups of four with a remainder), and compartment counts on
both sides of a group of four, with and without catalysts and frequency."""
import numpy as np
import pytest

import oracle
from gpu_util import TOL, max_rel_l2, to_gpu, to_np
from paper_2603_19789_amd import Model, inputs

pytestmark = pytest.mark.gpu


def _model(m, nt, lattice, rng):
    transitions = []
    for r in range(nt):
        src = int(rng.integers(0, m))
        dst = int(rng.integers(-1, m))
        while dst == src:
            dst = int(rng.integers(-1, m))
        cat = int(rng.integers(-1, m))
        transitions.append((src, dst, cat, float(rng.uniform(0.05, 0.4)), int(cat >= 0)))
    d = inputs.lattice_to_physical(rng.uniform(1e-3, 2e-2, m), 1.0, 0.05)
    counted = tuple(int(v) for v in rng.integers(0, 2, m)) if m > 1 else (1,)
    return inputs.GenericModel(tuple("C%d" % c for c in range(m)), d, tuple(transitions),
                               counted if any(counted) else (1,) * m, lattice, 1.0, 0.05)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("lattice", [5, 9])
@pytest.mark.parametrize("m,nt", [(1, 0), (1, 1), (2, 3), (4, 4), (5, 5), (3, 8), (8, 8), (6, 9),
                                  (4, 13), (8, 16)])
def test_tables_against_oracle(m, nt, lattice, dtype):
    rng = np.random.default_rng(100 * m + nt)
    model = _model(m, nt, lattice, rng)
    nx, ny, steps = 131, 23, 7
    rho0 = rng.uniform(0.2, 0.6, size=(m, ny, nx))
    if dtype == "f32":
        rho0 = rho0.astype(np.float32).astype(np.float64)
    got = to_np(Model(nx, ny, model, dtype=dtype, bc="noflux").run(to_gpu(rho0, dtype), steps))
    want = oracle.load().generic_run(rho0, model, steps, bc="noflux")
    assert max_rel_l2(got, want) <= TOL[dtype]
