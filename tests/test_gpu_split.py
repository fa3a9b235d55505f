"""The 15x15 patch projection and the synthesis in three BF16 parts, against the FP64 basis.

Error: the parts hold 24 significant bits, the dropped products add up to at most 2^-22 of |a||x| (a
twentieth of that on average, with either sign) and the sum is rounded at its full size once per 16
terms, so a coordinate is within a few 2^-24 of sum |a||x| on average; sqrt-summed over the terms that is below 3e-7 of the 2-norm here (FP32 products in
a chain: 2.5e-7 measured, these: 0.9e-7), asserted at 3e-7.  Wide ranges, whole and part chunks,
and chunks that hold an infinite value, which take FP32 products."""
import numpy as np
import pytest

from oracle import rsc_oracle as orc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
REL = 3e-7


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
        basis, h = orc.build_annular_basis(N), rsc.rsc_create_annular(N)
    else:
        S = 7 if N == 15 else 5
        basis, h = orc.build_basis(N, S, S), rsc.rsc_create(N, S, S)
    return basis, h, basis.mask.reshape(-1)


def _rel(a, ref):
    return np.linalg.norm(a - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("kind", ["grid", "annular"])
@pytest.mark.parametrize("P", [1, 31, 32, 33, 500])
def test_project(dev, kind, P):
    from paper_1806_04374_amd import rsc
    basis, h, disk = _make(kind, 15)
    rng = np.random.default_rng(P)
    x = (rng.standard_normal((P, 15, 15)) * 10.0 ** rng.uniform(-6, 6, (P, 1, 1))).astype(np.float32)
    out = rsc.rsc_project(h, torch.from_numpy(x).to(dev)).cpu().numpy()
    ref = x.reshape(P, -1)[:, disk].astype(np.float64) @ basis.pinv.T
    for p in range(P):
        assert _rel(out[p], ref[p]) <= 2 * REL, p
    h.close()


@pytest.mark.parametrize("kind,N", [("grid", 15), ("annular", 15), ("annular", 11)])
@pytest.mark.parametrize("P", [1, 32, 33, 300])
def test_synthesize_hat(dev, kind, N, P):
    from paper_1806_04374_amd import rsc
    basis, h, disk = _make(kind, N)
    xh = np.random.default_rng(P).standard_normal((P, basis.B)).astype(np.float32)
    out = rsc.rsc_synthesize_hat(h, torch.from_numpy(xh).to(dev)).cpu().numpy().reshape(P, -1)
    assert _rel(out[:, disk], xh.astype(np.float64) @ basis.phi.T) <= REL
    assert not out[:, ~disk].any()
    h.close()


def test_infinite_values_as_in_fp32(dev):
    """An infinite pixel or coordinate gives what FP32 products give: infinities of the sign of its
    factor (not NaN from a remainder), and its neighbours in the chunk stay finite."""
    from paper_1806_04374_amd import rsc
    basis, h, disk = _make("grid", 15)
    rng = np.random.default_rng(9)
    x = rng.standard_normal((70, 15, 15)).astype(np.float32)
    x[40, 7, 6] = np.inf
    out = rsc.rsc_project(h, torch.from_numpy(x).to(dev)).cpu().numpy()
    col = np.flatnonzero(disk).tolist().index(7 * 15 + 6)
    w = basis.pinv[:, col].astype(np.float32)
    big = np.abs(w) > 1e-6
    assert np.array_equal(out[40][big], np.where(w[big] > 0, np.inf, -np.inf))
    rest = np.delete(np.arange(70), 40)
    ref = x[rest].reshape(69, -1)[:, disk].astype(np.float64) @ basis.pinv.T
    assert _rel(out[rest], ref) <= 4e-7
    xh = rng.standard_normal((70, basis.B)).astype(np.float32)
    xh[3, 20] = -np.inf
    px = rsc.rsc_synthesize_hat(h, torch.from_numpy(xh).to(dev)).cpu().numpy().reshape(70, -1)
    f = basis.phi[:, 20].astype(np.float32)
    big = np.abs(f) > 1e-6
    assert np.array_equal(px[3][disk][big], np.where(f[big] > 0, -np.inf, np.inf))
    assert np.isfinite(np.delete(px, 3, axis=0)).all()
    h.close()


@pytest.mark.parametrize("kind,N", [("grid", 15), ("annular", 15), ("annular", 11)])
@pytest.mark.parametrize("power", [-115, -105, -95, 100])
def test_small_and_large_patches(dev, kind, N, power):
    """Patches whose values are too small for three whole BF16 parts (their last part would be below the
    normal numbers) keep the accuracy of the others, alone in a chunk of ordinary ones and in whole
    chunks; scaling by a power of two changes nothing above that range."""
    from paper_1806_04374_amd import rsc
    basis, h, disk = _make(kind, N)
    rng = np.random.default_rng(N)
    scale = np.ldexp(1.0, np.where((np.arange(100) == 5) | (np.arange(100) >= 40), power, 0)).astype(np.float32)
    xh = rng.standard_normal((100, basis.B)).astype(np.float32) * scale[:, None]
    px = rsc.rsc_synthesize_hat(h, torch.from_numpy(xh).to(dev)).cpu().numpy().reshape(100, -1)[:, disk]
    want = xh.astype(np.float64) @ basis.phi.T
    for p in range(100):
        assert _rel(px[p], want[p]) <= 2 * REL, p
    if N == 15:
        x = rng.standard_normal((100, 15, 15)).astype(np.float32) * scale[:, None, None]
        out = rsc.rsc_project(h, torch.from_numpy(x).to(dev)).cpu().numpy()
        want = x.reshape(100, -1)[:, disk].astype(np.float64) @ basis.pinv.T
        for p in range(100):
            assert _rel(out[p], want[p]) <= 2 * REL, p
    h.close()
