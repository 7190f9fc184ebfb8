"""GPU parity of the complex QR's persistent panel, whose columns are handed on word by word, in the
default form of every precision: rows one less, as many and one more than a workgroup's threads
(where double changes form) and than the tallest column, a panel of 256 workgroups; and an input
that holds the very word that marks what is not yet there."""
import numpy as np
import pytest

import mdgen
from test_gpu_complex import check_csolve, to_gpu

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2110_08375_amd

    return paper_2110_08375_amd


@pytest.mark.parametrize("P,m,n,tile", [
    (2, 9, 8, 8), (2, 255, 32, 16), (2, 256, 32, 32), (2, 257, 24, 8), (2, 2048, 16, 8), (2, 2052, 16, 8),
    (2, 256, 256, 256), (1, 256, 64, 32), (1, 257, 64, 32), (1, 257, 32, 16), (1, 4100, 16, 8), (4, 1024, 16, 8), (4, 257, 16, 16),
    (8, 512, 8, 8),
])
def test_cpanel_edges(M, orc, P, m, n, tile):
    check_csolve(M, orc, P, m, n, tile)


@pytest.mark.parametrize("P", (2, 4, 8))
def test_cpanel_empty_word_in_the_input(M, P):
    """That signalling NaN in the first column, which is published as it came: NaN in x, no time-out."""
    m, n, tile = 70, 32, 16
    print("case cpanel empty word P=%d m=%d n=%d tile=%d" % (P, m, n, tile), flush=True)
    A, _ = mdgen.cls_problem(P, m, n, 4100 + P)
    b = mdgen.cmd_vector(P, m, 4100 + P, mdgen.STREAM_B)
    A.view(np.uint64)[0, 0, 0, 40] = 0x7FF4000000007153
    x, info = M.csolve(P, to_gpu(A), to_gpu(b), tile)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    assert np.isnan(x.cpu().numpy()).any()


@pytest.mark.parametrize("P,m,n,tile", [(2, 40, 12, 1), (2, 40, 12, 2), (2, 40, 12, 3), (4, 40, 9, 1), (8, 24, 5, 1), (4, 40, 9, 3),
                                        (1, 40, 12, 1)])
def test_cpanel_narrow_tiles(M, orc, P, m, n, tile):
    """Tiles of one column, which hand nothing on, and of the few from which dd takes the persistent panel."""
    check_csolve(M, orc, P, m, n, tile)
