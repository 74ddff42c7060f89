"""1 to 4 replicas, wavefronts with none to six tiles of 512 parameters each: up to 3 replicas two sets of registers take the tiles in
turn.  (2047 workgroups of four wavefronts share a set of this size.)

Reference: exact sums.  An entry's products go through fewer than 128 fp64 additions one after the other: 48 in a lane, 6 over the lanes, 2 over the
wavefronts, up to 46 for the partial matrices."""
import pytest
import torch

import paper_2501_18512_amd as sdl
from gpu_util import exact_gram, gram_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [0, 1, 2, 3, 5])
@pytest.mark.parametrize("M,shift", [(1, 0), (2, 0), (2, 3), (3, 0), (4, 0)])
def test_tiles_in_turn(M, shift, tiles):
    n = 4 * 2047 * 512 * tiles + 512 * 700 + 37      # some wavefronts have one tile more
    gen = torch.Generator("cuda").manual_seed(tiles)
    g = torch.randn(n + shift, device="cuda", generator=gen)[shift:]
    w = [(g - torch.randn(n, device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(M)]
    w = [torch.cat([x[:shift], x])[shift:] for x in w]
    result, workspace = sdl.alloc_cosine(M)
    sdl.sdl_outer_grad_cosine(g, w, n, result[0], workspace)
    assert gram_error(sdl.split_cosine_result(result[0], M)[0], *exact_gram(g, w)) <= 128
