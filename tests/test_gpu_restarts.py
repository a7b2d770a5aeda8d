"""Restarts after a basis Gram that cannot be factored, on every path, in one mode and in
several at once (on the per-mode path each mode is factored by its own workgroup, which must
not depend on when the others raise the flag; a second-order stream raises the flag and
decides on it in one launch)."""
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


CASES = [
    ((40, 30), (5, 5), (0,), "plain"),
    ((40, 30), (5, 5), (0, 1), "plain"),
    ((30, 24, 20), (6, 5, 4), (0, 1, 2), "plain"),
    ((66, 50, 40), (40, 34, 20), (0, 1), "plain"),
    ((12, 20, 18, 6), (4, 6, 5, 3), (1, 2), "plain"),
    ((12, 20, 18, 6), (4, 6, 5, 3), (0, 1, 2, 3), "plain"),
    ((400, 12), (5, 5), (0,), "auto"),
    ((4000, 20), (17, 17), (1,), "auto"),
    ((300, 8), (4, 4), (0, 1), "auto"),
    ((30, 24, 8), (6, 5, 4), (1,), "fused"),
    ((130, 24, 20), (18, 5, 4), (0, 2), "fused"),
]


@pytest.mark.parametrize("dims,ranks,modes,path", CASES)
def test_dependent_basis_columns_restart(dims, ranks, modes, path):
    """Two equal columns in the bases of `modes`, and a snapshot equal to the one before, so
    that the step leaves them equal: the step ends in a restart from its snapshot, whose
    ranks lie within the caps, and the stream goes on from there."""
    from paper_2201_06958_amd import Compressor
    print("case", dims, ranks, modes, path, flush=True)
    rng = np.random.default_rng(sum(dims))
    C = rng.normal(size=ranks)
    F = [np.linalg.qr(rng.normal(size=(n, r)))[0] * np.sqrt(n) for n, r in zip(dims, ranks)]   # weights 1/N

    def field(core):
        v = core
        for n, f in enumerate(F):
            v = np.moveaxis(np.tensordot(f, v, axes=(1, n)), 0, n)
        return torch.from_numpy(np.ascontiguousarray(v)).to("cuda")

    U = [f.copy() for f in F]
    for n in modes:
        U[n][:, 1] = U[n][:, 0]
    V = field(C)
    c = Compressor(dims, 1e-2, rank_max=ranks, rank_init=ranks, data_dtype="f64", precision="f64", path=path,
                   adaptive=False)
    c.init_from_factors(V, C, U)
    c.ingest(V)
    st = c.stats()
    assert st["event"] == "numeric" and st["n_numeric"] == 1 and st["ranks"] == ranks
    # (an HOSVD at the field's own ranks reproduces it to the roundings of its sums)
    assert float((c.reconstruct() - V).abs().max()) <= 1e-11 * float(V.abs().max())
    W = field(C + 1e-3 * rng.normal(size=ranks))
    c.ingest(W)
    assert c.stats()["event"] == ""
    c.close()
