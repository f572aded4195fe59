"""GPU parity of the packed backward at the edges of its two tilings: the key-split kernels
(16- or 32-row workgroups, 32-row blocks over eight waves; the small launches of
test_gpu_backward run them too) and the 256-row kernels on the smallest launches that are
left to them.  Oracle and bars of test_gpu_backward."""
import pytest
import torch

from paper_2609_32540_amd import ff

from gpu_util import last_launch
from test_gpu_backward import TABLE6, run_case

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ff.lib()


# chunk and frame tokens around one 16-row tile and one 32-row block; streams of 1 to 3
# chunks leave most of the eight waves without a block, and a run of three 33-token chunks
# ends inside its fourth block
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("Nq,G", [(15, 5), (16, 16), (17, 1), (33, 31)])
def test_split_edges(d, Nq, G):
    run_case(4, Nq, G, 3, [[0, 2], [], [1], [0, 1, 2]], 2, 3, d, seed=31)
    # (dK and dV of such short streams run the 256-row kernel at d = 128)
    assert last_launch()[2:] == ((1, 0) if d == 128 else (2, 1))


# the same edges with streams of 720 to 816 rows: one 16-row tile per workgroup in both passes
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("Nq,G,n", [(15, 5, 48), (16, 16, 48), (17, 1, 48), (33, 31, 24)])
def test_split_edges_of_long_streams(d, Nq, G, n):
    table = [[[0, 2], [], [1], [0, 1, 2]][4 * c // n] for c in range(n)]
    run_case(n, Nq, G, 3, table, n, 2, d, seed=32)
    assert last_launch()[2:] == (1, 1)


@pytest.mark.parametrize("d", [128, 64])
def test_split_two_tiles(d):
    # 12 heads x 6 chunks of 198 tokens: two 16-row tiles per workgroup, the last one ragged
    # (13 tiles a chunk), and three anchor frames of 66
    run_case(6, 198, 66, 3, TABLE6, 2, 12, d, seed=33)
    assert last_launch()[2:] == (2, 2 if d == 64 else 1)   # (dK and dV take one at d = 128)


@pytest.mark.parametrize("d", [128, 64])
def test_256_row_kernels_on_a_partial_tile(d):
    # 40 heads x 4 chunks of 250 tokens: 160 query units fill the GPU, one ragged 256-row
    # tile a chunk, 70-token frames
    run_case(4, 250, 70, 2, [[], [0], [1], [0, 1]], 1, 40, d, seed=35)
    assert last_launch()[2:] == (0, 0)
