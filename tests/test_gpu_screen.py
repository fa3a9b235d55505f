"""The screened form of the FP32 encoder against the FP64 reference and the FP32 tiles.

FP32 handles leave out, by a 16-bit screen, the atoms that cannot win a step; the selection and
everything after it are FP32.  The sizes here are its edges: one atom, part and whole groups of
8 and 16 atoms, the largest M, one and two 32-angle tiles with even and odd R, every size of the
least-squares state, and launches of one patch, one tile and a remainder.  Codes are held to
the bar of the other parity tests: selected (atom, angle) sets equal on >= 99.9% (or all but one
patch of a small launch), every matched coefficient within 1e-4 relative.
"""
import numpy as np
import pytest

from oracle import rsc_oracle as orc
from paper_1806_04374_amd import workloads as wl
from tests.parity import compare_codes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MATCH = 0.999
COEF_REL = 1e-4


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04374_amd import rsc
    rsc.lib()
    return torch.device("cuda:0")


def _make(kind, N):
    from paper_1806_04374_amd import rsc
    if kind == "annular":
        return orc.build_annular_basis(N), rsc.rsc_create_annular(N)
    S = 5 if N == 11 else 7
    return orc.build_basis(N, S, S), rsc.rsc_create(N, S, S)


# (basis, N, M, R, K, P)
CASES = [
    ("grid", 11, 1, 64, 1, 1),
    ("grid", 11, 15, 1, 2, 33),        # R = 1: no rotation
    ("grid", 11, 16, 32, 2, 1000),
    ("grid", 11, 17, 31, 3, 500),      # odd R, one angle tile
    ("grid", 11, 64, 33, 4, 700),      # odd R, two tiles of the direct angle DFT
    ("grid", 11, 128, 34, 5, 500),     # the radix-2 split with 17 angle rows
    ("grid", 11, 40, 64, 8, 400),
    ("grid", 15, 7, 2, 1, 64),
    ("grid", 15, 100, 64, 1, 900),
    ("grid", 15, 128, 64, 6, 600),     # 8 waves of states just fit beside the tables
    ("grid", 15, 128, 63, 8, 300),     # they do not: 4 waves per block
    ("grid", 15, 33, 48, 3, 500),
    ("annular", 11, 1, 2, 1, 31),
    ("annular", 11, 8, 64, 2, 500),
    ("annular", 11, 9, 30, 4, 500),
    ("annular", 11, 64, 64, 4, 600),
    ("annular", 11, 128, 64, 2, 300),  # beyond the LDS: the FP32 tile
]


@pytest.mark.parametrize("case", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_screen_matches_reference(dev, case):
    from paper_1806_04374_amd import rsc
    kind, N, M, R, K, P = case
    basis, h = _make(kind, N)
    D = wl.draw_dictionary(M, basis.B, seed=900 + CASES.index(case))
    rsc.rsc_set_dictionary(h, D.astype(np.float32), R)
    used, _ = rsc.rsc_encode_info(h, K)
    assert used == ("16" if kind == "annular" and M == 128 else "auto")
    d = wl.draw_mixtures(P, N, M, min(4, M), 0.05, seed=900 + CASES.index(case))
    X = orc.synthesize(basis, D, d.atom, d.angle, d.weight, d.noise).astype(np.float32)
    print("screen", case, flush=True)
    xh = rsc.rsc_project(h, torch.from_numpy(X).to(dev))
    atom, angle, coef, r2 = [t.cpu().numpy() for t in rsc.rsc_omp_encode(h, xh, K)]
    xh_ref, code = orc.encode(basis, D, R, X.astype(np.float64), K)
    rep = compare_codes(atom, angle, coef, code, COEF_REL, xnorm=np.linalg.norm(xh_ref, axis=1))
    print(rep, flush=True)
    assert rep.matched >= P - max(1, int((1 - MATCH) * P)), str(rep)
    assert rep.coef_bad == 0, str(rep)
    h.close()


@pytest.mark.parametrize("kind,N", [("grid", 11), ("grid", 15), ("annular", 11)])
def test_every_atom_a_candidate(dev, kind, N):
    """64 atoms within 1e-4 of one another: every atom lies in the window at the first step, so the
    winner comes from the FP32 scores of all of them, in every group and both half-waves."""
    from paper_1806_04374_amd import rsc
    basis, h = _make(kind, N)
    rng = np.random.default_rng(77)
    base = wl.draw_dictionary(1, basis.B, seed=77)
    D = base + 1e-4 * rng.standard_normal((64, basis.B)) / np.sqrt(basis.B)
    D = (D / np.linalg.norm(D, axis=1, keepdims=True)).astype(np.float32).astype(np.float64)
    rsc.rsc_set_dictionary(h, D.astype(np.float32), 64)
    P = 256
    pick, w = rng.integers(0, 64, P), rng.uniform(0.5, 2.0, P)
    noise = 0.3 * rng.standard_normal((P, basis.B)) / np.sqrt(basis.B)
    xh = (w[:, None] * D[pick] + noise).astype(np.float32)
    atom, angle, coef, _ = [t.cpu().numpy() for t in rsc.rsc_omp_encode(h, torch.from_numpy(xh).to(dev), 1)]
    # scores of neighbours differ by about 1e-5 here and FP32 rounds them at about 1e-7: at most a
    # percent or so of the patches tie, and there the chosen score is as large
    A = orc.augmented_dictionary_basis(basis, D, 64)                   # row r M + m
    score = np.abs(xh.astype(np.float64) @ A.T)
    chosen = score[np.arange(P), angle[:, 0].astype(np.int64) * 64 + atom[:, 0]]
    assert (chosen >= score.max(axis=1) * (1 - 2e-6)).all()
    assert len(np.unique(atom[:, 0])) > 16
    h.close()


@pytest.mark.parametrize("kind,N", [("grid", 11), ("grid", 15), ("annular", 11)])
@pytest.mark.parametrize("power", [-61, -40, 50])
def test_scaled_coordinates(dev, kind, N, power):
    """Coordinates scaled by a power of two give the same selections and scaled coefficients: the
    screen's own scaling covers the range, and below a squared norm of 1e-30 (2^-61) every atom is
    a candidate."""
    from paper_1806_04374_amd import rsc
    basis, h = _make(kind, N)
    D = wl.draw_dictionary(48, basis.B, seed=5)
    rsc.rsc_set_dictionary(h, D.astype(np.float32), 64)
    rng = np.random.default_rng(6)
    xh = torch.from_numpy(rng.standard_normal((333, basis.B)).astype(np.float32)).to(dev)
    a0, r0, c0, _ = rsc.rsc_omp_encode(h, xh, 3)
    a1, r1, c1, _ = rsc.rsc_omp_encode(h, xh * 2.0 ** power, 3)
    assert torch.equal(a0, a1) and torch.equal(r0, r1)
    assert torch.equal(c0 * 2.0 ** power, c1)
    h.close()


@pytest.mark.parametrize("kind,N,M,R,K,tile", [("grid", 11, 64, 64, 4, "32"), ("grid", 15, 100, 64, 6, "16"),
                                               ("annular", 11, 64, 64, 4, "16")])
def test_screen_agrees_with_fp32_tile(dev, kind, N, M, R, K, tile):
    """The same coordinates through the screen and through the FP32 tile that scores every atom:
    the same codes."""
    from paper_1806_04374_amd import rsc
    basis, h = _make(kind, N)
    D = wl.draw_dictionary(M, basis.B, seed=8)
    rsc.rsc_set_dictionary(h, D.astype(np.float32), R)
    g = torch.Generator(device=dev).manual_seed(3)
    xh = torch.randn((20000, basis.B), generator=g, device=dev)
    a = [t.clone() for t in rsc.rsc_omp_encode(h, xh, K)]
    rsc.rsc_set_tile(h, tile)
    b = rsc.rsc_omp_encode(h, xh, K)
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    h.close()


def test_autotune_refuses_annular_beyond_four(dev):
    """No form of the pursuit on the annular basis is compiled for K > 4: refused before any launch."""
    from paper_1806_04374_amd import rsc
    h = rsc.rsc_create_annular(11)
    d = np.random.default_rng(1).standard_normal((8, h.B)).astype(np.float32)
    rsc.rsc_set_dictionary(h, d / np.linalg.norm(d, axis=1, keepdims=True), 32)
    x = torch.randn((100, h.B), device=dev)
    with pytest.raises(rsc.RscError):
        rsc.rsc_autotune_encode(h, x, 5)


@pytest.mark.parametrize("kind,N,prec,R,K,tiles", [("grid", 11, "fp32", 64, 4, ["auto", "32"]), ("grid", 11, "fp32", 30, 4, ["auto", "16"]),
                                                  ("grid", 15, "fp32", 64, 2, ["auto", "16"]), ("annular", 11, "fp32", 64, 2, ["auto", "16"]),
                                                  ("annular", 15, "fp32", 64, 2, ["16"]), ("grid", 11, "bf16", 64, 4, ["32"])])
def test_autotune_times_both_forms(dev, kind, N, prec, R, K, tiles):
    """Where the library has a screened form the autotuner times it against the full form with the
    same codes, so whichever it keeps, the codes are the same."""
    from paper_1806_04374_amd import rsc
    basis, h = _make(kind, N)
    if prec != "fp32":
        h = rsc.rsc_create(N, basis.S, basis.T, prec=prec)
    d = np.random.default_rng(2).standard_normal((24, basis.B)).astype(np.float32)
    rsc.rsc_set_dictionary(h, d / np.linalg.norm(d, axis=1, keepdims=True), R)
    x = torch.randn((3000, basis.B), generator=torch.Generator(device=dev).manual_seed(1), device=dev)
    before = [t.clone() for t in rsc.rsc_omp_encode(h, x, K)]
    rows = rsc.rsc_autotune_encode(h, x, K, reps=1)
    assert [r[0] for r in rows] == [t for t in tiles for _ in range(4)]
    assert rsc.rsc_get_launch(h)[0] in tiles
    for t in tiles:
        rsc.rsc_set_launch(h, t, 1)
        for a, b in zip(before, rsc.rsc_omp_encode(h, x, K)):
            assert torch.equal(a, b)
    h.close()


def test_autotune_keeps_the_full_form_for_low_contrast(dev):
    """Windows whose contrast is 0.01 of their mean, coded with atoms of no mean: nearly every atom is a
    candidate of the screen, and the full form is more than three times as fast."""
    from paper_1806_04374_amd import rsc
    basis, h = _make("grid", 15)
    const = basis.pinv.sum(axis=1)
    const /= np.linalg.norm(const)
    d = np.random.default_rng(1).standard_normal((128, basis.B))
    d -= (d @ const)[:, None] * const
    rsc.rsc_set_dictionary(h, (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32), 64)
    x = torch.randn((60000, basis.B), generator=torch.Generator(device=dev).manual_seed(1), device=dev)
    x = x / x.norm(dim=1, keepdim=True) * 0.01 + torch.from_numpy(const).to(dev).float()
    rsc.rsc_autotune_encode(h, x, 4, reps=3)
    assert rsc.rsc_get_launch(h)[0] == "16"
    h.close()


@pytest.mark.parametrize("kind,N,K,P,M", [("grid", 15, 1, 1, 20), ("grid", 15, 2, 33, 20), ("grid", 11, 1, 5003, 20),
                                          ("annular", 11, 1, 700, 20), ("grid", 15, 1, 3001, 97), ("grid", 11, 4, 999, 60)])
def test_classify_takes_the_smallest_error(dev, kind, N, K, P, M):
    """Labels and errors that the screened encoder writes itself are those of one pursuit per class:
    the smallest squared residual norm, the first class on equal ones (the first two share a
    dictionary), bit for bit."""
    from paper_1806_04374_amd import rsc
    basis, _ = _make(kind, N)
    rng = np.random.default_rng([N, K, P])
    hs = []
    for c in range(4):
        if c != 1:
            d = rng.standard_normal((M + c, basis.B)).astype(np.float32)
        h = _make(kind, N)[1] if c < 3 or kind == "annular" else rsc.rsc_create(N, basis.S, basis.T, prec="bf16")
        rsc.rsc_set_dictionary(h, d / np.linalg.norm(d, axis=1, keepdims=True), 48)
        hs.append(h)
    x = torch.randn((P, basis.B), generator=torch.Generator(device=dev).manual_seed(P), device=dev)
    label, sse = rsc.rsc_classify(hs, x, K)
    r2 = torch.stack([rsc.rsc_omp_encode(h, x, K)[3].clone() for h in hs])
    want, at = r2.min(0)
    at = (r2 == want).to(torch.int32).argmax(0)
    assert torch.equal(sse, want) and torch.equal(label.long(), at.long())
