"""Equal columns within a block of 32 leave the device's Cholesky factor a pivot of zero:
refused, the later column named, the block of vectors as it was.  In the first block of
columns, in later ones (whose pivots come out of the block steps), in a ragged last one."""
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,pair", [(2, (0, 1)), (40, (3, 31)), (40, (33, 38)), (64, (32, 63)), (96, (70, 95)),
                                    (130, (128, 129)), (200, (64, 90))])
def test_equal_columns_are_refused(n, pair):
    from paper_2410_02754_amd import ChfsiError, Operator
    op = Operator((4, 3, 3), (4.4, 3.3, 3.3), 3, "gll", 4)
    X = torch.tensor(synth.random_block(9, op.n_dof, n), device="cuda")
    X[:, pair[1]] = X[:, pair[0]]
    Y = X.clone()
    with pytest.raises(ChfsiError) as e:
        op.chol_gs(X)
    assert e.value.code == -4 and e.value.bad_col == pair[1]
    assert torch.equal(X, Y)
    op.close()
