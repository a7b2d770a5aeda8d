"""Core and bases read to the host: the energetic rotation in every order and precision."""
import numpy as np
import pytest

from oracle import tdb_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2201_06958_amd import load_library
    load_library()


def stream(dims, ranks, prec, core):
    """A stream holding `core` and random W-orthonormal bases (weights 1/N)."""
    from paper_2201_06958_amd import Compressor
    rng = np.random.default_rng(sum(dims))
    U = [np.linalg.qr(rng.normal(size=(n, r)))[0] * np.sqrt(n) for n, r in zip(dims, ranks)]
    data = "f64" if prec == "f64" else "f32"
    V = torch.zeros(dims, dtype=torch.float64 if data == "f64" else torch.float32, device="cuda")
    c = Compressor(dims, 1e-2, rank_max=ranks, rank_init=ranks, data_dtype=data, precision=prec, adaptive=False)
    return c.init_from_factors(V, core, U), U


ROTATED = [
    ((4096, 8), (8, 8), "f32"),        # the bases in FP64 take more than the snapshot in FP32
    ((4096, 8), (8, 8), "f64"),
    ((3000, 6), (4, 4), "f32"),
    ((64, 8, 3), (20, 8, 3), "f32"),
    ((64, 8, 3), (20, 8, 3), "bf16s"),
    ((40, 5, 4, 2), (16, 5, 4, 2), "f32"),
]


@pytest.mark.parametrize("dims,ranks,prec", ROTATED)
def test_rotation(dims, ranks, prec):
    """The rotation is FP64 whatever the stream's types. The first unfolding's singular values
    fall from 1 to 2^-8 in equal ratios, so its eigenvectors carry about
    r 2^-53 2^16 / (1 - ratio^2): 4e-10 at r = 20. Bound 1e-8, as for the other rotations."""
    print("case", dims, ranks, prec, flush=True)
    rng = np.random.default_rng(9)
    r0, rest = ranks[0], int(np.prod(ranks[1:]))
    q0, q1 = np.linalg.qr(rng.normal(size=(r0, r0)))[0], np.linalg.qr(rng.normal(size=(rest, r0)))[0]
    core = (q0 * (2.0 ** -(np.arange(r0) * min(1.0, 8.0 / r0)))) @ q1.T
    core = core.reshape(ranks)
    c, U = stream(dims, ranks, prec, core)
    _, C0, U0 = c.get_core_and_bases()
    assert np.array_equal(C0, core) and all(np.array_equal(a, b) for a, b in zip(U0, U))
    _, Cr, Ur = c.get_core_and_bases(rotate=True)
    Co, Uo = O.core_rotation(core, U)
    assert np.abs(Cr - Co).max() <= 1e-8 * np.abs(Co).max()
    for a, b in zip(Ur, Uo):
        assert np.abs(a - b).max() <= 1e-8 * np.abs(b).max()
    # the state is untouched
    _, C1, U1 = c.get_core_and_bases()
    assert np.array_equal(C0, C1) and all(np.array_equal(a, b) for a, b in zip(U0, U1))
    c.close()
