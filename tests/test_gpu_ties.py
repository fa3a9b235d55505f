"""Ties in the screened FP32 encoder: patches whose selection FP32 rounding decides are coded as the
full encoder codes them.

A patch that is the sum of two atoms at angles of the grid, w (a + b) with unit a and b, scores
w (1 + <a, b>) with both, a tie that only the order of the sums breaks, so every output of such a
patch has to be the full form's bit for bit.  The launches cover one patch, a tile and a
remainder, ties in every patch and in one of 97, and more tiles than waves.
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
    ("grid", 11, 64, 64, 4, 1, 1, "32"),
    ("grid", 11, 64, 64, 4, 33, 1, "32"),
    ("grid", 11, 64, 64, 4, 400003, 97, "32"),
    ("grid", 11, 128, 45, 4, 3001, 2, "16"),
    ("grid", 11, 16, 32, 8, 70001, 1, "16"),
    ("grid", 15, 128, 64, 6, 40009, 97, "16"),
    ("grid", 15, 22, 33, 6, 517, 1, "16"),
    ("annular", 11, 64, 64, 4, 5003, 3, "16"),
]


@pytest.mark.parametrize("basis,N,M,R,K,P,every,full", CASES)
def test_ties_as_full_form(dev, basis, N, M, R, K, P, every, full):
    from paper_1806_04374_amd import rsc
    S = 5 if N == 11 else 7
    h = rsc.rsc_create_annular(N) if basis == "annular" else rsc.rsc_create(N, S, S)
    b = orc.build_annular_basis(N) if basis == "annular" else orc.build_basis(N, S, S)
    rng = np.random.default_rng([N, M, R, P])
    d = rng.standard_normal((M, b.B))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    rsc.rsc_set_dictionary(h, d, R)
    g = torch.Generator(device=dev).manual_seed(P)
    D = torch.from_numpy(d).to(dev)
    atoms = torch.stack([torch.randperm(M, generator=g, device=dev)[:2] for _ in range(64)])[
        torch.randint(0, 64, (P,), generator=g, device=dev)]
    w = 0.5 + torch.rand((P, 1), generator=g, device=dev)
    turn = lambda a: rsc.rsc_steer(h, a.contiguous(), theta=(   # noqa: E731
        torch.randint(0, R, (P,), generator=g, device=dev) * (2 * np.pi / R)).float())
    x = w * (turn(D[atoms[:, 0]]) + turn(D[atoms[:, 1]]))
    free = torch.arange(P, device=dev) % every != 0
    x[free] = torch.randn((int(free.sum()), b.B), generator=g, device=dev)
    got = [t.clone() for t in rsc.rsc_omp_encode(h, x, K)]
    assert int(got[0].min()) >= -1
    rsc.rsc_set_launch(h, full, 0)
    want = rsc.rsc_omp_encode(h, x, K)
    sel = (got[0] == want[0]).all(1) & (got[1] == want[1]).all(1)
    assert bool(sel.all()), f"{int((~sel).sum())} of {P} selections differ"
    tied = ~free
    same = sel & (got[2] == want[2]).all(1) & (got[3] == want[3])
    # sums of rounded rows tie to within the window in nearly every patch; a third atom may beat both
    assert float(same[tied].float().mean()) > 0.5
    assert torch.allclose(got[2], want[2], rtol=1e-4, atol=1e-4)


def test_symmetric_atoms_stay_screened(dev):
    """An atom that rotation leaves alone, or half a turn, ties at all its angles by itself: the first
    angle is selected, as in the full form."""
    from paper_1806_04374_amd import rsc
    b = orc.build_basis(11, 5, 5)
    h = rsc.rsc_create(11, 5, 5)
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
    got = [t.clone() for t in rsc.rsc_omp_encode(h, x, 4)]
    rsc.rsc_set_launch(h, "32", 0)
    want = rsc.rsc_omp_encode(h, x, 4)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert int((got[1][:, 0] >= 32).sum()) == 0
