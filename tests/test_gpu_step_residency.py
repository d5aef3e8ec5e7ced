"""Step launches on both sides of the sizes where the number of resident workgroups changes, or whether a list's tiles are whole."""
import numpy as np
import pytest
import torch

import oracle
import paper_2104_07857_amd as zi
import zi_synth
from gpu_util import NormBuffers, compare_state, gen_numpy, to_dev, to_np, zi_cfg

pytestmark = pytest.mark.gpu
TILE = 512
RUN, LIST, BARE, MOST_BARE, FEW = 1 << 15, 1 << 16, 1 << 15, 3 << 15, 9     # kFineRunTiles, kFineListTiles, kBareListTiles, kBareListMostTiles, kFewTiles


@pytest.mark.parametrize("dt", [zi.ZI_BF16, zi.ZI_FP16])
@pytest.mark.parametrize("n", [RUN * TILE, RUN * TILE + 4])
def test_one_tensor_around_the_limit(n, dt):
    hp, hm, hv, hg = gen_numpy(zi_synth.StateSpec(n + dt, dt), n)
    dev = [to_dev(a.copy()) for a in (hp, hm, hv, hg)] + [torch.zeros(n, dtype=torch.int16, device="cuda:0")]
    zi.zi_adamw_step([tuple(dev) + (n,)], dt, zi_cfg(zi_synth.workload("c1")))
    torch.cuda.synchronize()
    lp = np.zeros(n, np.uint16)
    oracle.adamw(hp, hm, hv, hg, lp, dt, oracle.config(step=10), 0.0, 0)
    compare_state((hp, hm, hv, lp), [to_np(dev[i]) for i in (0, 1, 2, 4)], dt)


def test_one_short_tensor_replays_from_a_captured_graph():
    dt, n = zi.ZI_BF16, 3000
    host = gen_numpy(zi_synth.StateSpec(8, dt), n)
    cfg = zi_cfg(zi_synth.workload("c4"))
    sides = []
    for _ in range(2):
        bufs = [to_dev(a.copy()) for a in host] + [torch.zeros(n, dtype=torch.int16, device="cuda:0")]
        sides.append((zi.make_tensors([tuple(bufs) + (n,)]), NormBuffers(), bufs))
    (tl, nb, graphed), (tl_e, nb_e, eager) = sides
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        graph.capture_begin()
        zi.zi_grad_norm(tl, dt, 1.0, nb.out, nb.ws, stream=stream)
        zi.zi_adamw_step(tl, dt, cfg, nb.out, stream)
        graph.capture_end()
    for _ in range(4):
        graph.replay()
        zi.zi_grad_norm(tl_e, dt, 1.0, nb_e.out, nb_e.ws)
        zi.zi_adamw_step(tl_e, dt, cfg, nb_e.out)
        torch.cuda.synchronize()
        for a, b in zip(graphed, eager):
            assert torch.equal(a, b)
            a[:3] += 0                               # eager work between the replays
        assert nb.read() == nb_e.read()


@pytest.mark.parametrize("tiles,count,shuffled,copies", [
    (LIST, 64, True, True), (LIST, 64, True, False), (LIST, 256, False, True), (LIST, 256, False, False),
    (BARE, 64, True, False), (MOST_BARE, 64, True, False), (FEW * 150, 150, False, True), (FEW * 150, 150, False, False)])
@pytest.mark.parametrize("beyond", [-TILE, 0, TILE])
def test_lists_around_the_limits_equal_one_tensor(tiles, count, shuffled, copies, beyond):
    """Lists whose (first) launch is one of so many tiles, or a tile a tensor on either side of that, give the bits of one flat
    tensor.  Shuffled gradients keep a list from being views at the same places of five buffers."""
    each = tiles // count * TILE + beyond
    count += 1 if shuffled else 0                    # such lists take the way of more than 64 tensors
    dt, n = zi.ZI_BF16, count * each
    gen = torch.Generator(device="cuda:0").manual_seed(each)
    rand = lambda std: torch.empty(n, device="cuda:0").normal_(0.0, std, generator=gen)      # noqa: E731
    state = [rand(0.02), rand(1e-4), rand(1e-6).abs_(), rand(1e-3).bfloat16().view(torch.int16),
             torch.zeros(n, dtype=torch.int16, device="cuda:0")]
    whole = [x.clone() for x in state]
    if shuffled:                                     # the gradients' pieces stand in reverse order
        state[3] = state[3].view(count, each).flip(0).reshape(-1)
        place = lambda w, i: (count - 1 - i if w == 3 else i) * each                         # noqa: E731
    else:
        place = lambda w, i: i * each                                                        # noqa: E731
    pick = lambda x, at, k: None if x is None else x[at:at + k]                              # noqa: E731
    arrays = state if copies else state[:4] + [None]
    cfg = zi_cfg(zi_synth.workload("c1"))
    zi.zi_adamw_step([tuple(pick(x, place(w, i), each) for w, x in enumerate(arrays)) + (each,) for i in range(count)], dt, cfg)
    zi.zi_adamw_step([tuple(whole if copies else whole[:4] + [None]) + (n,)], dt, cfg)
    torch.cuda.synchronize()
    if shuffled:
        state[3] = state[3].view(count, each).flip(0).reshape(-1)
    for w, (a, b) in enumerate(zip(state, whole)):
        assert torch.equal(a, b), "p m v g lp".split()[w]
