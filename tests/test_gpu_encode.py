"""psdf_encode_padded at the edges of its one-launch form (up to 4096 rows, 64
slots a row and 16384 entries; 1024 lanes) and just past them, against the
same selection in numpy.  Entries are moved, never computed on: bytes equal."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Mbar,mbar", [(1, 1), (1, 64), (1, 65), (63, 3), (1023, 5), (1024, 16),
                                       (1025, 7), (2049, 7), (256, 64), (257, 64), (4096, 4),
                                       (4096, 5), (4097, 1)])
@pytest.mark.parametrize("fill", [0.0, 0.5, 1.0])
def test_encode_edges(Mbar, mbar, fill):
    import paper_2607_04310_amd.api as api
    rng = np.random.default_rng([Mbar, mbar])
    A = rng.normal(size=(Mbar, mbar, 2)).astype(np.float32)
    B = rng.normal(size=(Mbar, mbar, 2)).astype(np.float32)
    S = rng.random((Mbar, mbar)) < fill
    A[0, 0] = np.nan, -np.inf
    for mask in (torch.tensor(S), torch.tensor(S.astype(np.uint8) * 200)):
        es = api.psdf_encode_padded(torch.tensor(A).cuda(), torch.tensor(B).cuda(), mask.cuda())
        off = np.concatenate([[0], np.cumsum(S.sum(1))]).astype(np.int32)
        assert np.array_equal(es.obst_off.cpu().numpy(), off)
        for got, want in ((es.ax, A[S][:, 0]), (es.ay, A[S][:, 1]), (es.bx, B[S][:, 0]),
                          (es.by, B[S][:, 1])):
            assert got.cpu().numpy().tobytes() == want.tobytes()
