"""The fused step at a measured pace (two to four quads a lane, one after the other): launches on both sides of the sizes where its
kernels change, ragged last tiles, the elements around a tensor's body and lists with tensors that have none."""
import numpy as np
import pytest
import torch

import paper_2104_07857_amd as zi
import zi_synth
from gpu_util import NormBuffers, zi_cfg
from test_gpu_fine_tiles import ONE_ROUND, SHORT, TILE, pieces, random_state, step_with_oracle

pytestmark = pytest.mark.gpu
EIGHT, STORES, MOST = 1 << 11, 15 << 8, 7 << 10                         # workgroups on a compute unit, kPacedStoresOne, kMostPacedTiles


@pytest.mark.parametrize("tiles", [SHORT, EIGHT, STORES, ONE_ROUND, 3 << 11, MOST])
@pytest.mark.parametrize("beyond,offset", [(0, 0), (1, 0), (4, 0), (259, 0), (66, 1)])
def test_one_tensor_around_the_lines(tiles, beyond, offset):
    n = tiles * TILE + beyond
    step_with_oracle(zi.ZI_FP16 if beyond % 2 else zi.ZI_BF16, n, (offset,) * 5, mode=1 if beyond == 4 else 0, copy=beyond != 1,
                     clip=0.7 if offset else 0.0)


def test_arrays_that_start_anywhere():
    step_with_oracle(zi.ZI_BF16, 3300 * TILE + 77, (3, 1, 0, 2, 61))


# Cuts around a few elements leave tensors without a body among the others.
@pytest.mark.parametrize("copies", [True, False])
@pytest.mark.parametrize("count", [2, 20, 50, 200])
@pytest.mark.parametrize("tiles", [SHORT, 2700, ONE_ROUND - 60])
def test_lists_give_the_bits_of_short_launches(tiles, count, copies):
    n = tiles * TILE + 65
    state = random_state(n, n + count)
    keep = state if copies else state[:4]
    whole = [x.clone() for x in state]
    r = np.random.default_rng(count)
    cuts = [0, 1, 4] + sorted(int(x) for x in r.integers(4, n, count - 1)) + [n]
    cuts = sorted(cuts + [c + 2 for c in cuts[3:-1:5]])
    for flat in (True, False):
        tensors = pieces(keep, cuts)
        if not flat:
            tensors = [tuple(x.clone() if torch.is_tensor(x) else x for x in t) for t in tensors]
        zi.zi_adamw_step(tensors, zi.ZI_BF16, zi_cfg(zi_synth.workload("c1")))
        if flat:
            got = [x.clone() for x in keep]
            for a, b in zip(keep, whole):
                a.copy_(b)
        else:
            again = [torch.cat([t[w] for t in tensors]) for w in range(len(keep))]
    part = whole if copies else whole[:4]
    for piece in pieces(part, list(range(0, n, 800_000)) + [n]):
        zi.zi_adamw_step([piece], zi.ZI_BF16, zi_cfg(zi_synth.workload("c1")))
    torch.cuda.synchronize()
    for w, (a, b, c) in enumerate(zip(got, again, part)):
        assert torch.equal(a, c) and torch.equal(b, c), "p m v g lp".split()[w]


@pytest.mark.parametrize("n,count", [(1_600_000, 1), (2_500_000, 1), (3_500_000, 1), (1_600_000, 20), (1_600_000, 70)])
def test_overflow_skips_paced_tiles(n, count):
    state = random_state(n, count)
    state[3][n - 1] = 0x7F80                                            # +inf
    before = [x.clone() for x in state]
    nb = NormBuffers()
    cuts = [n * i // count for i in range(count + 1)]
    zi.zi_grad_norm(pieces(state, cuts), zi.ZI_BF16, 1.0, nb.out, nb.ws)
    zi.zi_adamw_step(pieces(state, cuts), zi.ZI_BF16, zi_cfg(zi_synth.workload("c4")), nb.out)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(state, before))
