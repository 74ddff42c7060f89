"""1 to 4 replicas, workgroups with none to five tiles of 512 parameters each: up to 3 replicas two sets of registers take the tiles in
turn.  (8192 workgroups share a set of this size.)"""
import numpy as np
import pytest
import torch

import paper_2501_18512_amd as sdl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [0, 1, 2, 3, 5])
@pytest.mark.parametrize("M,shift", [(1, 0), (2, 0), (2, 3), (3, 0), (4, 0)])
def test_tiles_in_turn(M, shift, tiles):
    n = 8192 * 512 * tiles + 512 * 700 + 37          # some workgroups have one tile more
    gen = torch.Generator("cuda").manual_seed(tiles)
    g = torch.randn(n + shift, device="cuda", generator=gen)[shift:]
    w = [(g - torch.randn(n, device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(M)]
    w = [torch.cat([x[:shift], x])[shift:] for x in w]
    result, workspace = sdl.alloc_cosine(M)
    sdl.sdl_outer_grad_cosine(g, w, n, result[0], workspace)
    G = sdl.split_cosine_result(result[0], M)[0].cpu().numpy()
    d = torch.stack([torch.nn.functional.pad((g - x.float()).double(), (0, -n % 2048)) for x in w])
    want = torch.bmm(d.view(M, -1, 2048).transpose(0, 1).contiguous(), d.view(M, -1, 2048).permute(1, 2, 0).contiguous()).sum(0).cpu().numpy()
    norm = np.sqrt(np.diag(want))
    # sums of at most 2^15 terms one after the other on either side, a term 2^-53 off at most
    assert np.abs(G - want).max() <= 2.0 ** -37 * np.outer(norm, norm).max()
