"""GPU parity of RoPE over the block shapes of its kernel: 2 to 4 tokens a block, blocks of
less than one, of exactly five and of more than five 16-byte vectors a thread, Q alone, K
alone, both.  Bar: 1 bf16 unit in the last place of the rounded float64 value, 1e-5 for
float32 (as test_gpu_parity)."""
import numpy as np
import pytest
import torch

from paper_2609_32540_amd import ff

from gpu_util import bf16_ordered, exact, make_cache, oracle_rope, to_dev
from test_gpu_parity import small

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True, scope="module")
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ff.lib()


# vectors of a token at bf16: 16 heads (4 tokens a block: a small token), 5 and 12 heads (2
# tokens; 12 with 4680 tokens: 4 tokens, 3 steps), 40 heads (2 tokens = 5 steps of 256
# lanes), 41 heads (a sixth, partial step), 81 heads (a second full round of five)
@pytest.mark.parametrize("heads,head_dim,grid", [(1, 64, (1, 1)), (1, 128, (3, 5)), (5, 128, (4, 5)),
                                                 (12, 128, (30, 52)), (40, 128, (3, 3)), (41, 128, (3, 3)),
                                                 (81, 128, (1, 3))])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_block_shapes(heads, head_dim, grid, dtype):
    w = small(dtype, head_dim, heads=heads, grid_h=grid[0], grid_w=grid[1], stages=1, layers=1)
    cache = make_cache(w, 1, 1)
    frames = [7, 0, 19]
    g = torch.Generator().manual_seed(5)
    x, y = (torch.randn((w.chunk_tokens, heads, head_dim), generator=g).to(w.torch_dtype) for _ in range(2))
    refs = [oracle_rope(w, t, frames) for t in (x, y)]
    for use in ((0, 1), (0, None), (None, 1)):
        q = to_dev(x) if use[0] is not None else None
        k = to_dev(y) if use[1] is not None else None
        cache.rope3d(q, k, frames)
        for t, ref in ((q, refs[0]), (k, refs[1])):
            if t is None:
                continue
            if dtype == "bf16":
                want = bf16_ordered(torch.from_numpy(ref).to(torch.bfloat16))
                assert np.abs(bf16_ordered(t) - want).max() <= 1
            else:
                assert np.abs(exact(t) - ref).max() <= 1e-5
