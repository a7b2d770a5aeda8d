"""Core and bases read to the host: states below and above the pinned buffer they go through,
what a caller leaves out, and the energetic rotation in every order and precision."""
import ctypes
import threading

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


@pytest.mark.parametrize("dims,ranks", [
    ((70, 40), (5, 3)),                    # one contracted tile, not full
    ((300, 270), (33, 18)),                # several, and rows past the last
    ((40, 36, 12), (6, 5, 4)),
    ((40, 130, 20), (20, 90, 9)),
    ((9, 20, 18, 5), (3, 7, 5, 2)),
])
@pytest.mark.parametrize("out", ["f32", "f64"])
def test_infinite_entries_stay_infinite(dims, ranks, out):
    """One infinite entry of the core, the last, and factors without zeros: every value of the
    reconstruction is an infinity of the sign that its product has."""
    from paper_2201_06958_amd.tdb import reconstruct_noalloc
    print("case", dims, ranks, out, flush=True)
    rng = np.random.default_rng(sum(dims))
    C = rng.uniform(0.5, 1.0, size=ranks)
    C[(-1,) * len(ranks)] = np.inf
    U = [rng.uniform(0.5, 1.0, size=(n, r)) * rng.choice([-1.0, 1.0], size=(n, r)) for n, r in zip(dims, ranks)]
    sign = np.sign(U[0][:, -1])
    for u in U[1:]:
        sign = sign[..., None] * np.sign(u[:, -1])
    V = torch.empty(dims, dtype=torch.float32 if out == "f32" else torch.float64, device="cuda")
    reconstruct_noalloc(torch.from_numpy(C).cuda(), [torch.from_numpy(u).cuda() for u in U], V)
    assert np.array_equal(V.cpu().numpy(), sign * np.inf)


@pytest.mark.parametrize("dims,ranks", [
    ((3, 2), (1, 1)), ((64, 512), (8, 20)), ((100, 9, 7, 5), (9, 9, 7, 1)), ((100, 60, 80), (10, 24, 20)),   # one output a thread
    ((500, 500), (40, 40)), ((501, 499), (41, 39)),                 # the last product at the limit, and above
    ((3001, 170), (21, 20)), ((45, 37, 33, 15), (9, 17, 16, 15)),   # tiles with remainders
    ((64, 60, 62, 8), (20, 24, 18, 6)), ((90, 101, 103), (22, 23, 24)),
])
@pytest.mark.parametrize("out", ["f32", "f64"])
def test_decode_matches_64_bits(dims, ranks, out):
    """Each product of r terms adds at most (r + 2) roundings of the sum of magnitudes; the
    output one more in its own type. The output may lie off a 16-byte boundary."""
    from paper_2201_06958_amd.tdb import reconstruct_noalloc
    print("case", dims, ranks, out, flush=True)
    rng = np.random.default_rng(sum(dims))
    C, U = rng.normal(size=ranks), [rng.normal(size=(n, r)) for n, r in zip(dims, ranks)]
    ref, mag = O.reconstruct(C, U), O.reconstruct(np.abs(C), [np.abs(u) for u in U])
    bound = sum(r + 3 for r in ranks) * 2.0 ** -53 * 2 * mag + (2.0 ** -24 if out == "f32" else 0.0) * np.abs(ref)
    S = int(np.prod(dims))
    for off in (0, 1):
        buf = torch.full((S + 4,), float("nan"), dtype=torch.float32 if out == "f32" else torch.float64, device="cuda")
        V = buf[off:off + S].view(dims)
        reconstruct_noalloc(torch.from_numpy(C).cuda(), [torch.from_numpy(u).cuda() for u in U], V)
        assert (np.abs(V.cpu().numpy().astype(np.float64) - ref) <= bound).all()
        assert torch.isnan(buf[:off]).all() and torch.isnan(buf[off + S:]).all()


HALF = 1 << 16     # doubles of a half of the pinned buffer


@pytest.mark.parametrize("dims,ranks", [
    (((HALF - 64) // 8 - 9, 8), (8, 8)),       # one piece, short of a half
    (((HALF - 64 - 64) // 8, 8), (8, 8)),      # exactly a half
    (((HALF - 64 - 64) // 8 + 1, 8), (8, 8)),  # the last basis ends in a second piece
    ((HALF // 8 * 3 + 5, 8), (8, 8)),          # four pieces
    ((100, 90, 80), (50, 40, 41)),             # the core alone more than a half
    ((40, 39, 38, 37), (20, 20, 17, 16)),
])
def test_read_in_pieces(dims, ranks):
    print("case", dims, ranks, flush=True)
    rng = np.random.default_rng(4)
    core = rng.normal(size=ranks)
    c, U = stream(dims, ranks, "f32", core)
    for _ in range(2):
        r, C1, U1 = c.get_core_and_bases()
        assert r == ranks and np.array_equal(C1, core) and all(np.array_equal(a, b) for a, b in zip(U1, U))
    # any of the outputs may be left out
    P = ctypes.POINTER(ctypes.c_double)
    for skip in range(-1, len(dims)):
        got = [np.full(u.shape, np.nan) for u in U]
        Cg = np.full(ranks, np.nan)
        uptr = (P * 8)()
        for n, u in enumerate(got):
            if n != skip:
                uptr[n] = u.ctypes.data_as(P)
        assert c.lib.tdb_get_core_and_bases(c.h, 0, None, None if skip < 0 else Cg.ctypes.data_as(P), uptr) == 0
        assert np.isnan(Cg).all() if skip < 0 else np.array_equal(Cg, core)
        for n, (a, b) in enumerate(zip(got, U)):
            assert np.isnan(a).all() if n == skip else np.array_equal(a, b)
    assert c.lib.tdb_get_core_and_bases(c.h, 0, None, None, None) == 0
    c.close()


def test_read_takes_no_device_memory():
    """A state of 128 MB is read without a device allocation: the free memory that another
    thread sees during the call stays what it was (within 32 MB for the runtime's own)."""
    rng = np.random.default_rng(5)
    c, U = stream((2_000_000, 8), (8, 8), "f32", np.diag(2.0 ** -np.arange(8)))
    c.get_core_and_bases()
    torch.cuda.synchronize()
    least, done = [torch.cuda.mem_get_info()[0]], threading.Event()
    before = least[0]

    def watch():
        while not done.is_set():
            least[0] = min(least[0], torch.cuda.mem_get_info()[0])

    t = threading.Thread(target=watch)
    t.start()
    for _ in range(3):
        _, C1, U1 = c.get_core_and_bases()
    done.set()
    t.join()
    assert all(np.array_equal(a, b) for a, b in zip(U1, U))
    assert before - least[0] < 32 << 20, (before, least[0])
    c.close()
