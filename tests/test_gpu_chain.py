"""Third-order streams whose third mode is longer than 16, by tiles or by n-mode products
(single streams, as their sizes and ranks decide; batches by tiles), and the FP64 sums over
whole modes of the products."""
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


@pytest.mark.parametrize("dims", [(512, 480, 20), (500, 24, 510), (36, 512, 66), (192, 192, 192)])
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


def walk(dims, ranks, seed, steps=4, amp=0.02):
    """Random walks of core and bases around a well-conditioned start."""
    rng = np.random.default_rng(seed)
    C = rng.normal(size=ranks)
    F = [np.linalg.qr(rng.normal(size=(n, r)))[0] for n, r in zip(dims, ranks)]
    out = []
    for _ in range(steps + 1):
        out.append(O.reconstruct(C, F))
        C = C + amp * rng.normal(size=ranks)
        F = [f + amp * rng.normal(size=f.shape) / np.sqrt(f.shape[0]) for f in F]
    return out


# (sizes on both sides of the rule: the mode's length, the tiles at once, a tile's work)
ROUTES = [
    ((40, 36, 16), (6, 7, 3)), ((33, 30, 9), (4, 5, 9)), ((90, 75, 12), (12, 11, 3)),   # always tiles
    ((20, 18, 17), (6, 5, 17)), ((70, 40, 20), (9, 8, 5)), ((64, 40, 63), (5, 5, 5)),   # tiles
    ((70, 40, 20), (33, 32, 9)), ((30, 200, 40), (24, 20, 6)),                          # work above the limit
    ((20, 18, 64), (6, 5, 17)), ((33, 31, 67), (17, 16, 20)), ((66, 64, 90), (5, 64, 13)),
    ((300, 150, 18), (3, 3, 2)),                                                   # more tiles than fit at once
]


def check(c, orc, dims, prec, w):
    r, C, U = c.get_core_and_bases()
    assert r == orc.ranks
    ref, got = O.reconstruct(orc.C, orc.U), O.reconstruct(C, U)
    # FP64: amplified roundings of a few steps; FP32: as the streams' other FP32 tests
    assert np.abs(got - ref).max() <= (1e-9 if prec == "f64" else 1e-6) * np.abs(ref).max()
    for n in range(len(dims)):
        assert np.abs(U[n].T @ (U[n] * w[n][:, None]) - np.eye(r[n])).max() <= 1e-13


@pytest.mark.parametrize("dims,ranks", ROUTES)
@pytest.mark.parametrize("mode", ["copy", "borrow"])
def test_single_stream_matches_oracle(dims, ranks, mode):
    from paper_2201_06958_amd import Compressor
    print("case", dims, ranks, mode, flush=True)
    rng = np.random.default_rng(3)
    w = [v / v.sum() for v in (rng.uniform(0.5, 1.5, size=n) for n in dims)]
    v = walk(dims, ranks, 11)
    orc = O.OracleTDB(O.OracleConfig(dims=dims, weights=w, dt=1e-2, rank_max=ranks, rank_init=ranks, adaptive=False,
                                     eps_th=1.0)).init(v[0])
    c = Compressor(dims, 1e-2, rank_max=ranks, rank_init=ranks, weights=w, data_dtype="f64", precision="f64",
                   adaptive=False, snapshot_mode=mode)
    d = [torch.from_numpy(np.ascontiguousarray(x)).to("cuda") for x in v]
    c.init_from_factors(d[0], orc.C, orc.U)
    for k in range(1, 5):
        orc.ingest(v[k])
        c.ingest(d[k])
    check(c, orc, dims, "f64", w)
    c.close()


@pytest.mark.parametrize("dims,ranks,path", [((30, 200, 40), (24, 20, 6), "auto"), ((20, 18, 64), (6, 5, 17), "auto"),
                                             ((70, 40, 20), (33, 32, 9), "auto"), ((9, 20, 18, 5), (4, 7, 6, 3), "auto")])
def test_buffers_made_on_a_side_stream(dims, ranks, path):
    """The products' buffers are made by the first step that takes them, which may run on a
    stream of its own: the same as on the null stream, bit for bit."""
    from paper_2201_06958_amd import Compressor
    print("case", dims, ranks, flush=True)
    v = [torch.from_numpy(np.ascontiguousarray(x)).to("cuda") for x in walk(dims, ranks, 5)]
    got = []
    for side in (False, True):
        c = Compressor(dims, 1e-2, rank_max=ranks, rank_init=ranks, data_dtype="f64", precision="f64", path=path,
                       adaptive=False)
        c.init(v[0])
        torch.cuda.synchronize()
        s = torch.cuda.Stream() if side else torch.cuda.default_stream()
        with torch.cuda.stream(s):
            for x in v[1:]:
                c.ingest(x, stream=s)
        torch.cuda.synchronize()
        _, C, U = c.get_core_and_bases()
        got.append((C, U))
        c.close()
    assert np.array_equal(got[0][0], got[1][0]) and all(np.array_equal(a, b) for a, b in zip(got[0][1], got[1][1]))


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("shapes,ranks", [
    (((20, 18, 192), (33, 24, 192)), (5, 5, 5)),      # tiles shrunk along modes 1 and 2 to fit the LDS
    (((40, 70, 24), (17, 16, 40), (33, 9, 17)), (6, 5, 4)),
])
def test_batch_matches_oracle(shapes, ranks, prec):
    from paper_2201_06958_amd import Batch
    print("case", shapes, ranks, prec, flush=True)
    tp = np.float64 if prec == "f64" else np.float32
    runs = []
    for i, dims in enumerate(shapes):
        w = [np.full(n, 1.0 / n) for n in dims]
        v = [np.ascontiguousarray(x, dtype=tp) for x in walk(dims, ranks, 20 + i)]
        orc = O.OracleTDB(O.OracleConfig(dims=dims, weights=w, dt=1e-2, rank_max=ranks, rank_init=ranks,
                                         adaptive=False, eps_th=1.0)).init(v[0].astype(np.float64))
        runs.append((dims, w, v, orc, [torch.from_numpy(x).to("cuda") for x in v]))
    b = Batch([dict(dims=dims, dt=1e-2, rank_max=ranks, rank_init=ranks, weights=w, data_dtype=prec, precision=prec,
                    adaptive=False) for dims, w, _, _, _ in runs]).init([d[0] for *_, d in runs])
    for k in range(1, 5):
        b.ingest([d[k] for *_, d in runs])
        for _, _, v, orc, _ in runs:
            orc.ingest(v[k].astype(np.float64))
    for s, (dims, w, _, orc, _) in zip(b.streams, runs):
        check(s, orc, dims, prec, w)
    b.close()
