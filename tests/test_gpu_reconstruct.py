"""Codes back to pixels against the FP64 reference on every layout the pursuit is compiled for:
part and whole 32-patch chunks, one slot to sixteen (the slots go by 1 or 2 at a time), empty and
out-of-range slots, and an output that is not 16-byte aligned.

Tolerance: a pixel is a sum of B <= 153 products of FP32 values, and each coordinate of K <= 16
terms; sqrt(B + 16) roundings of 2^-24 each are 8e-7 of the 2-norm, asserted at 2e-6."""
import numpy as np
import pytest

from oracle import rsc_oracle as orc
from paper_1806_04374_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04374_amd import rsc
    rsc.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("kind,N,M,R", [("grid", 11, 64, 64), ("grid", 15, 100, 33), ("annular", 11, 20, 30),
                                        ("annular", 15, 9, 64), ("grid", 13, 8, 16)])
@pytest.mark.parametrize("P,K", [(1, 1), (31, 2), (33, 3), (32, 4), (500, 5), (64, 16)])
def test_reconstruct_matches_reference(dev, kind, N, M, R, P, K):
    from paper_1806_04374_amd import rsc
    if kind == "annular":
        basis, h = orc.build_annular_basis(N), rsc.rsc_create_annular(N)
    else:
        S = 7 if N == 15 else 5
        basis, h = orc.build_basis(N, S, S), rsc.rsc_create(N, S, S)
    D = wl.draw_dictionary(M, basis.B, seed=3)
    rsc.rsc_set_dictionary(h, D.astype(np.float32), R)
    rng = np.random.default_rng(P * 100 + K)
    atom, angle = rng.integers(0, M, (P, K)), rng.integers(0, R, (P, K))
    coef = rng.standard_normal((P, K)).astype(np.float32)
    skip = rng.random((P, K)) < 0.2            # empty, then slots with an atom or an angle out of range
    atom[skip] = rng.choice([-1, M, 1 << 20], skip.sum())
    wrong = rng.random((P, K)) < 0.1
    angle[wrong] = rng.choice([-1, R], wrong.sum())
    hat = np.zeros((P, basis.B))
    d32 = D.astype(np.float32).astype(np.float64)
    for j in range(K):
        for p in range(P):
            if not (skip[p, j] or wrong[p, j]):
                hat[p] += coef[p, j] * orc.steer_basis(basis, d32[atom[p, j]:atom[p, j] + 1], 2 * np.pi * angle[p, j] / R)[0]
    ref = orc.to_pixels(basis, hat) if kind == "grid" else None
    if ref is None:
        ref = np.zeros((P, N * N))
        ref[:, basis.mask.reshape(-1)] = hat @ basis.phi.T
    ref = ref.reshape(P, N, N)
    args = [torch.from_numpy(x).to(dev) for x in (atom.astype(np.int32), angle.astype(np.int32), coef)]
    print("reconstruct", kind, N, P, K, flush=True)
    out = rsc.rsc_reconstruct(h, *args).cpu().numpy()
    assert np.linalg.norm(out - ref) <= 2e-6 * max(np.linalg.norm(ref), 1e-30)
    off = torch.empty(P * N * N + 1, device=dev)[1:].view(P, N, N)
    assert np.array_equal(rsc.rsc_reconstruct(h, *args, out=off).cpu().numpy(), out)
    h.close()
