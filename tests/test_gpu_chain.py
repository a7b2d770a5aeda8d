"""Third-order FP32 streams whose third mode is longer than 16: the projections' sums over
whole modes are FP64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_06958_amd import load_library
    load_library()


@pytest.mark.parametrize("dims", [(512, 480, 20), (500, 24, 510), (36, 512, 18), (192, 192, 192)])
@pytest.mark.parametrize("data", ["f32", "f64"])
def test_long_sums_lose_nothing(dims, data):
    """An explicit Euler step with a constant data derivative c on bases that hold the constant:
    C_dot is c in its first entry and 0 elsewhere. FP32 roundings, 2^-24 each, of that entry:
    the weighted basis and the sums within 16 rows (at most half a unit for each of their
    partial sums, (1 + 2 + ... + 15) / 16 / 2 = 4 units) of the first product, and the two
    stored intermediates: 7 x 2^-24 in all. (FP32 sums of a whole mode of some hundred equal
    terms are off by 15 to 170 of these.)"""
    from paper_2201_06958_amd import Compressor
    print("case", dims, data, flush=True)
    rng = np.random.default_rng(3)
    U = [np.stack([np.ones(n), (-1.0) ** np.arange(n)], axis=1) for n in dims]   # W-orthonormal for weights 1/N
    C = np.zeros((2, 2, 2))
    C[0, 0, 0], C[1, 1, 0], C[0, 1, 1], C[1, 0, 1] = 1.0, 0.5, 0.5, 0.25
    dt = 0.5
    tp = torch.float32 if data == "f32" else torch.float64
    V = torch.zeros(dims, dtype=tp, device="cuda")
    worst = 0.0
    for _ in range(6):
        c = float(np.float32(rng.uniform(1.0, 2.0)))
        g = Compressor(dims, dt, rank_max=(2, 2, 2), rank_init=(2, 2, 2), data_dtype=data, precision="f32",
                       adaptive=False, integrator="euler")
        g.init_from_factors(V, C, U)
        g.ingest_with_derivative(V, torch.full(dims, c, dtype=tp, device="cuda"))
        assert g.stats()["path_used"] == "fused"
        _, C1, _ = g.get_core_and_bases()
        want = C.copy()
        want[0, 0, 0] += dt * c
        worst = max(worst, np.abs(C1 - want).max() / (dt * c))
        g.close()
    print("  worst", worst, flush=True)
    assert worst <= 7 * 2.0 ** -24
