"""Snapshots and outputs off a 16-byte boundary on the routes that load several columns at a
time where the alignment allows it: n-mode products in orders 2 to 4, and third-order
streams with long third modes."""
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


def at(x, off):
    """x on the device, `off` values behind an aligned address."""
    buf = torch.empty(x.size + 4, dtype=torch.from_numpy(x).dtype, device="cuda")
    v = buf[off:off + x.size].view(x.shape)
    v.copy_(torch.from_numpy(x))
    return v


CASES = [
    ((48, 64), (7, 7), "plain"),
    ((40, 36, 16), (6, 5, 4), "plain"),
    ((96, 80, 64), (5, 6, 7), "fused"),            # enough columns for 16-byte loads
    ((33, 31, 67), (5, 6, 7), "fused"),            # rows of odd length
    ((12, 30, 26, 8), (3, 7, 6, 3), "auto"),
    ((16, 64, 48, 4), (3, 9, 8, 2), "auto"),
]


@pytest.mark.parametrize("dims,ranks,path", CASES)
@pytest.mark.parametrize("data,prec", [("f32", "f32"), ("f32", "f64"), ("f64", "f64"), ("f64", "f32")])
@pytest.mark.parametrize("offs", [(1, 2, 3), (0, 1, 0), (2, 2, 2)])
def test_steps_match_oracle(dims, ranks, path, data, prec, offs):
    from paper_2201_06958_amd import Compressor
    print("case", dims, ranks, path, data, prec, offs, flush=True)
    rng = np.random.default_rng(6)
    w = [np.full(n, 1.0 / n) for n in dims]
    tp = np.float32 if data == "f32" else np.float64
    C = rng.normal(size=ranks)
    F = [np.linalg.qr(rng.normal(size=(n, r)))[0] * np.sqrt(n) for n, r in zip(dims, ranks)]
    v = []
    for _ in range(4):
        v.append(np.ascontiguousarray(O.reconstruct(C, F), dtype=tp))
        C = C + 0.02 * rng.normal(size=ranks)
        F = [f + 0.02 * rng.normal(size=f.shape) for f in F]
    orc = O.OracleTDB(O.OracleConfig(dims=dims, weights=w, dt=1e-2, rank_max=ranks, rank_init=ranks, adaptive=False,
                                     eps_th=1.0)).init(v[0].astype(np.float64))
    c = Compressor(dims, 1e-2, rank_max=ranks, rank_init=ranks, weights=w, data_dtype=data, precision=prec,
                   path=path, adaptive=False, snapshot_mode="borrow")
    d = [at(x, o) for x, o in zip(v, (offs[0],) + offs)]
    c.init_from_factors(d[0], orc.C, orc.U)
    for k in range(1, 4):
        orc.ingest(v[k].astype(np.float64))
        c.ingest(d[k])
    out = at(np.zeros(dims, dtype=tp), offs[0])
    c.reconstruct(out)
    ref = orc.reconstruct()
    bar = 1e-9 if (data, prec) == ("f64", "f64") else 1e-6     # as the streams' other tests of these types
    assert np.abs(out.cpu().numpy().astype(np.float64) - ref).max() <= bar * np.abs(ref).max()
    c.close()
