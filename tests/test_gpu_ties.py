"""Ties in the screened FP32 encoder: every output is the full form's, bit for bit.

The screened form sums scores, coefficients and residuals in the full form's order, and where two
atoms come within the rounding of these sums it compares them in the order of the full form's
first pass.  So nothing may differ from the tile that "auto" would take without a screen, least of
all where a selection is decided by rounding:

  tied        w (a + b) with unit atoms a and b at angles of the grid scores w (1 + <a, b>) with both
  contrast    K atoms and noise of 1e-2 to 1e-5 of the patch: late residuals are mostly inherited rounding
  halfturn    odd harmonics at rounding level: every atom ties at angles half a turn apart
  flat        harmonics above 0 at rounding level: every atom ties at all its angles
  duplicates  each atom twice in the dictionary, the copy turned by a step of the grid
  tiny        noise scaled by 2^-61: squared norms below 1e-30, every atom a candidate
  noise       no ties

Launches cover one patch, a tile and a remainder, ties in every patch and in one of 97, more
tiles than waves, every layout and split of the angles, and M K from 1 up.
"""
import pytest

from oracle import rsc_oracle as orc

torch = pytest.importorskip("torch")
np = pytest.importorskip("numpy")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04374_amd import rsc
    rsc.lib()
    return torch.device("cuda:0")


# (basis, N, M, R, K, P, one tied patch in, the full form under "auto")
CASES = [
    ("grid", 11, 1, 64, 1, 1, 1, "32"),
    ("grid", 11, 64, 64, 4, 1, 1, "32"),
    ("grid", 11, 64, 64, 4, 33, 1, "32"),
    ("grid", 11, 64, 64, 4, 400003, 97, "32"),
    ("grid", 11, 20, 34, 2, 7001, 1, "32"),
    ("grid", 11, 128, 64, 2, 3001, 1, "16"),   # beyond the 32x32 tile's LDS
    ("grid", 11, 128, 45, 4, 3001, 2, "16"),
    ("grid", 11, 16, 32, 8, 70001, 1, "16"),
    ("grid", 11, 9, 2, 3, 501, 1, "16"),
    ("grid", 11, 33, 64, 6, 2003, 1, "16"),
    ("grid", 15, 128, 64, 6, 40009, 97, "16"),
    ("grid", 15, 22, 33, 6, 517, 1, "16"),
    ("grid", 15, 100, 64, 1, 3001, 1, "16"),
    ("grid", 15, 60, 31, 3, 999, 1, "16"),
    ("grid", 15, 40, 30, 8, 999, 1, "16"),
    ("annular", 11, 64, 64, 4, 5003, 3, "16"),
    ("annular", 11, 10, 30, 2, 777, 1, "16"),
]
KINDS = ["tied", "contrast", "halfturn", "flat", "duplicates", "tiny", "noise"]


def _handle(basis, N):
    from paper_1806_04374_amd import rsc
    S = 5 if N == 11 else 7
    if basis == "annular":
        return orc.build_annular_basis(N), rsc.rsc_create_annular(N)
    return orc.build_basis(N, S, S), rsc.rsc_create(N, S, S)


def _harmonics(h, b, dev):
    """Harmonic of each packed coordinate: steering by half a turn flips the odd ones, and so on."""
    from paper_1806_04374_amd import rsc
    one = torch.ones((1, b.B), device=dev)
    flips = rsc.rsc_steer(h, one, theta=torch.full((1,), np.pi, device=dev))[0] < 0
    moved = (rsc.rsc_steer(h, one, theta=torch.full((1,), 0.1, device=dev))[0] - 1).abs() > 1e-4
    return flips, moved                                   # odd; not harmonic 0


def _full_form_bits(h, x, K, full):
    from paper_1806_04374_amd import rsc
    rsc.rsc_set_launch(h, "auto", 0)
    assert rsc.rsc_encode_info(h, K)[0] == "auto"
    rsc.rsc_precision_stats(h, reset=True)
    got = [t.clone() for t in rsc.rsc_omp_encode(h, x, K)]
    n64 = rsc.rsc_precision_stats(h, reset=True)
    rsc.rsc_set_launch(h, full, 0)
    want = rsc.rsc_omp_encode(h, x, K)
    for name, a, b in zip(("atom", "angle", "coef", "resid2"), got, want):
        differ = (a != b).reshape(a.shape[0], -1).any(1)
        assert not bool(differ.any()), f"{name}: {int(differ.sum())} of {a.shape[0]} patches, first {int(differ.nonzero()[0])}"
    assert rsc.rsc_precision_stats(h, reset=True) == n64
    return got


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("basis,N,M,R,K,P,every,full", CASES)
def test_ties_as_full_form(dev, basis, N, M, R, K, P, every, full, kind):
    from paper_1806_04374_amd import rsc
    b, h = _handle(basis, N)
    rng = np.random.default_rng([N, M, R, P])
    d = rng.standard_normal((M, b.B))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    g = torch.Generator(device=dev).manual_seed(P)
    D = torch.from_numpy(d).to(dev)
    if kind == "duplicates" and M > 1:
        turns = torch.randint(0, 2, (M // 2,), generator=g, device=dev) * (2 * np.pi / R)
        D[M - M // 2:] = rsc.rsc_steer(h, D[:M // 2].contiguous(), theta=turns.float())
        d = D.cpu().numpy()
    rsc.rsc_set_dictionary(h, d, R)
    turn = lambda a: rsc.rsc_steer(h, a.contiguous(), theta=(   # noqa: E731
        torch.randint(0, R, (P,), generator=g, device=dev) * (2 * np.pi / R)).float())
    noise = torch.randn((P, b.B), generator=g, device=dev)
    atoms = torch.randint(0, M, (P, max(K, 2)), generator=g, device=dev)
    weights = 0.5 + torch.rand((P, max(K, 2)), generator=g, device=dev)
    odd, moved = _harmonics(h, b, dev)
    if kind == "tied":
        x = weights[:, :1] * (turn(D[atoms[:, 0]]) + turn(D[atoms[:, 1]]))
    elif kind in ("contrast", "duplicates"):
        x = sum(weights[:, j:j + 1] * turn(D[atoms[:, j]]) for j in range(K))
        x += 10 ** -(2 + 3 * torch.rand((P, 1), generator=g, device=dev)) * noise / b.B ** 0.5
    elif kind == "halfturn":
        x = torch.where(odd, 1e-7 * noise, noise)
    elif kind == "flat":
        x = torch.where(moved, 1e-8 * noise, noise)
    else:
        x = noise * (2.0 ** -61 if kind == "tiny" else 1.0)
    free = torch.arange(P, device=dev) % every != 0
    if kind != "tiny":
        x[free] = torch.randn((int(free.sum()), b.B), generator=g, device=dev)
    print("ties", kind, basis, N, M, R, K, P, flush=True)
    _full_form_bits(h, x.contiguous(), K, full)
    h.close()


def test_symmetric_atoms_take_the_first_angle(dev):
    """An atom that rotation leaves alone, or half a turn, has equal scores at all its angles: the
    first angle is selected, as in the full form."""
    from paper_1806_04374_amd import rsc
    b, h = _handle("grid", 11)
    rng = np.random.default_rng(4)
    d = rng.standard_normal((64, b.B))
    harm = np.concatenate([[0] * 5] + [[k] * 10 for k in range(1, 6)])
    d[0, harm > 0] = 0.0
    d[1, harm % 2 == 1] = 0.0
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    rsc.rsc_set_dictionary(h, d, 64)
    g = torch.Generator(device=dev).manual_seed(3)
    D = torch.from_numpy(d).to(dev)
    x = 3 * D[torch.arange(5000, device=dev) % 2] + 0.1 * torch.randn((5000, b.B), generator=g, device=dev)
    got = _full_form_bits(h, x, 4, "32")
    assert int((got[1][:, 0] >= 32).sum()) == 0
    h.close()
