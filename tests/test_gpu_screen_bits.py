"""The screened encoder's arithmetic against the full FP32 forms, bit for bit.

16-bit handles score and select in FP32 among the screen's candidates, in the order of sums of the
32x32 tile's second pass, and update coefficients and residual as it does, so wherever the two
select the same columns and both stay in FP32 every output bit is the same.
"""
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


def _condition_bound(basis, D, R, atom, angle):
    """k ||L^-1||_F^2 of the Gram matrix of each patch's k selected columns, in 64 bits (the bound
    beyond which a handle's least squares go to FP64: 1e3 on FP32 handles, 1e6 on 16-bit ones).  It
    grows with k, so the last step's covers the earlier ones."""
    A = torch.from_numpy(orc.augmented_dictionary_basis(basis, D, R)).to(atom.device)   # row r M + m
    M = D.shape[0]
    G = A[(angle.long() * M + atom.long()).clamp(min=0)]                                # [P, K, B]
    gram = torch.stack([(G[:, i, None, :] * G).sum(-1) for i in range(G.shape[1])], 1)
    tr = torch.linalg.inv(gram).diagonal(dim1=1, dim2=2).sum(1)                         # ||L^-1||_F^2
    return G.shape[1] * tr


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("M,R,K,P", [(1, 64, 1, 1), (16, 34, 2, 33), (64, 64, 4, 20011), (112, 48, 3, 5000)])
def test_16bit_handles_as_the_32_tile(dev, prec, M, R, K, P):
    from paper_1806_04374_amd import rsc
    basis = orc.build_basis(11, 5, 5)
    D = wl.draw_dictionary(M, basis.B, seed=M).astype(np.float32)
    d = wl.draw_mixtures(P, 11, M, min(4, M), 0.05, seed=M + 1)
    X = orc.synthesize(basis, D.astype(np.float64), d.atom, d.angle, d.weight, d.noise)
    x = torch.from_numpy((X.reshape(P, -1)[:, basis.mask.reshape(-1)] @ basis.pinv.T).astype(np.float32)).to(dev)
    h, f = rsc.rsc_create(11, 5, 5, prec=prec), rsc.rsc_create(11, 5, 5)
    for q in (h, f):
        rsc.rsc_set_dictionary(q, D, R)
    rsc.rsc_set_tile(f, "32")
    print("bits", prec, M, R, K, P, flush=True)
    got, want = rsc.rsc_omp_encode(h, x, K), rsc.rsc_omp_encode(f, x, K)
    same = (got[0] == want[0]).all(1) & (got[1] == want[1]).all(1)
    # the tile's first pass sums the scores that choose the atom in another order: patches whose two
    # best atoms tie to about 1e-7 of the residual may differ, about one step in 1e6
    assert int((~same).sum()) <= 1
    well = same & (want[0] >= 0).all(1) & (_condition_bound(basis, D.astype(np.float64), R, want[0], want[1]) < 500)
    assert int(well.sum()) >= 0.8 * P
    assert torch.equal(got[2][well], want[2][well]) and torch.equal(got[3][well], want[3][well])
    h.close()
    f.close()
