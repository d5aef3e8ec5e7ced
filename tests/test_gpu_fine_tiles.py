"""The fused step in fine tiles (one quad a lane): launches on both sides of the sizes where whole and fine tiles, runs of
XCDs and plain order, and the number of resident workgroups change, and the elements around a tensor's body."""
import numpy as np
import pytest
import torch

import oracle
import paper_2104_07857_amd as zi
import zi_synth
from gpu_util import NormBuffers, compare_state, gen_numpy, to_dev, to_np, zi_cfg

pytestmark = pytest.mark.gpu
TILE, SHORT, ONE_ROUND, RUNS, LONG = 512, 7 << 8, 1 << 12, 1 << 15, 1 << 16      # kFineShortTiles, kOneRoundTiles, kFine{Run,List}Tiles


def step_with_oracle(dt, n, offsets, mode=0, copy=True, clip=0.0, scale=1.0):
    """Steps one tensor whose five arrays start `offsets` elements into their buffers; every element against the oracle, the
    buffers' ends unchanged."""
    host = list(gen_numpy(zi_synth.StateSpec(n + dt + 5, dt), n)) + [np.zeros(n, np.uint16)]
    pad = 70
    bufs = []
    for a, o in zip(host, offsets):
        b = np.full(n + pad, 7, a.dtype)
        b[o:o + n] = a
        bufs.append(to_dev(b))
    views = [b[o:o + n] for b, o in zip(bufs, offsets)]
    if not copy:
        views[4] = None
    nb = NormBuffers()
    tensors = [tuple(views) + (n,)]
    cfg = zi.make_config(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, step=10, loss_scale=scale,
                         max_grad_norm=clip, mode=mode)
    zi.zi_grad_norm(tensors, dt, scale, nb.out, nb.ws)
    zi.zi_adamw_step(tensors, dt, cfg, nb.out)
    torch.cuda.synchronize()
    p, m, v, g, lp = host
    sumsq, flag = oracle.grad_sumsq([g], dt)
    oracle.adamw(p, m, v, g, lp if copy else None, dt,
                 oracle.config(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, step=10, loss_scale=scale,
                               max_grad_norm=clip, mode=mode), sumsq, flag)
    got = [to_np(b) for b in bufs]
    for w, (a, o) in enumerate(zip(got, offsets)):
        edge = np.concatenate([a[:o], a[o + n:]])
        assert (edge == 7).all(), "p m v g lp".split()[w]
    keep = [got[w][offsets[w]:offsets[w] + n] for w in (0, 1, 2, 4)]
    if not copy:
        keep[3] = lp
    compare_state((p, m, v, lp), keep, dt)


# Heads of 0, 1 and 63 elements, tails of 0 to 3, head and tail together more than a wavefront, no body at all.
@pytest.mark.parametrize("dt", [zi.ZI_BF16, zi.ZI_FP16])
@pytest.mark.parametrize("n,offset", [(1, 0), (3, 5), (62, 1), (63, 1), (64, 1), (65, 1), (66, 1), (67, 1), (70, 1), (255, 0),
                                      (256, 0), (257, 0), (259, 63), (511, 1), (512, 1), (513, 1), (1003, 0), (1027, 37)])
def test_ends_of_short_tensors(dt, n, offset):
    step_with_oracle(dt, n, [offset] * 5, mode=n % 2, copy=n % 3 != 0, clip=1.0 if n % 2 else 0.7, scale=1.0 if n % 5 else 1000.0)


@pytest.mark.parametrize("dt", [zi.ZI_BF16, zi.ZI_FP16])
def test_arrays_that_start_anywhere(dt):
    for n, offsets in ((777, (1, 2, 3, 4, 5)), (70_001, (0, 7, 63, 33, 1)), (ONE_ROUND * TILE + 700, (3, 1, 0, 2, 61))):
        step_with_oracle(dt, n, offsets, copy=n != 777)


@pytest.mark.parametrize("n", [SHORT * TILE, SHORT * TILE + 4, ONE_ROUND * TILE, ONE_ROUND * TILE + 4, 8 * 1024 * 256 + 256,
                               2 * 8 * 1024 * 256 - 4])
def test_one_tensor_around_the_lines(n):
    step_with_oracle(zi.ZI_BF16 if n % 8 else zi.ZI_FP16, n, (0,) * 5, mode=1 if n % 8 else 0)


def random_state(n, seed):
    gen = torch.Generator(device="cuda:0").manual_seed(seed)
    rand = lambda std: torch.empty(n, device="cuda:0").normal_(0.0, std, generator=gen)      # noqa: E731
    return [rand(0.02), rand(1e-4), rand(1e-6).abs_(), rand(1e-3).bfloat16().view(torch.int16),
            torch.zeros(n, dtype=torch.int16, device="cuda:0")]


def pieces(state, cuts):
    lp = [] if len(state) == 5 else [None]
    return [tuple([x[a:b] for x in state] + lp + [b - a]) for a, b in zip(cuts[:-1], cuts[1:]) if b > a]


# The update is per element, so any cut gives the bits of whole launches of one round (1.5e6 elements each).
@pytest.mark.parametrize("copies", [True, False])
@pytest.mark.parametrize("n,count", [(RUNS * TILE, 1), (RUNS * TILE + 260, 1), (LONG * TILE + 1, 7), (LONG * TILE - 5, 40),
                                     (ONE_ROUND * TILE + 9, 3), (ONE_ROUND * TILE - 3, 5), (SHORT * TILE + 65, 30),
                                     (6_000_000, 300), (5_000_000, 33), (9_000_000, 2), (18_000_000, 40)])
def test_any_cut_gives_the_same_bits(n, count, copies):
    state = random_state(n, n + count)
    keep = state if copies else state[:4]
    whole = [x.clone() for x in state]
    r = np.random.default_rng(count)
    cuts = [0] + sorted(int(x) for x in r.integers(0, n, count - 1)) + [n]
    cfg = zi_cfg(zi_synth.workload("c1"))
    zi.zi_adamw_step(pieces(keep, cuts), zi.ZI_BF16, cfg)
    for part in pieces(whole if copies else whole[:4], list(range(0, n, 1_500_000)) + [n]):
        zi.zi_adamw_step([part], zi.ZI_BF16, cfg)
    torch.cuda.synchronize()
    for w, (a, b) in enumerate(zip(state, whole)):
        assert torch.equal(a, b), "p m v g lp".split()[w]


@pytest.mark.parametrize("n,count", [(3_000_000, 1), (3_000_000, 20), (3_000_000, 100)])
def test_overflow_skips_fine_tiles(n, count):
    state = random_state(n, count)
    state[3][n - 1] = 0x7F80                                            # +inf
    before = [x.clone() for x in state]
    nb = NormBuffers()
    cuts = [n * i // count for i in range(count + 1)]
    zi.zi_grad_norm(pieces(state, cuts), zi.ZI_BF16, 1.0, nb.out, nb.ws)
    zi.zi_adamw_step(pieces(state, cuts), zi.ZI_BF16, zi_cfg(zi_synth.workload("c4")), nb.out)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(state, before))


# Arrays of their own are dealt out in runs of XCDs: tensors with no run, one and several, at any place of the launch.
@pytest.mark.parametrize("lengths", [[4_000_000, 1_100_001, 3_000_000], [5, 2_200_003, 70, 9_000_001, 1]])
def test_arrays_of_their_own_give_the_bits_of_views(lengths):
    n = sum(lengths)
    state = random_state(n, n)
    cuts = [0] + np.cumsum(lengths).tolist()
    own = [tuple(x.clone() if torch.is_tensor(x) else x for x in t) for t in pieces(state, cuts)]
    cfg = zi_cfg(zi_synth.workload("c1"))
    zi.zi_adamw_step(own, zi.ZI_BF16, cfg)
    for part in pieces(state, list(range(0, n, 800_000)) + [n]):
        zi.zi_adamw_step([part], zi.ZI_BF16, cfg)
    torch.cuda.synchronize()
    for w, whole in enumerate(state):
        assert torch.equal(torch.cat([t[w] for t in own]), whole), "p m v g lp".split()[w]


# More than 64 flat tensors of up to 2^20 elements on average go 256 to a launch.
@pytest.mark.parametrize("lengths", [[400_000] * 64, [400_000] * 66, [5, 800_003] * 33])
def test_shared_launches_give_the_bits_of_single_ones(lengths):
    n = sum(lengths)
    state = random_state(n, len(lengths))
    whole = [x.clone() for x in state]
    cfg = zi_cfg(zi_synth.workload("c1"))
    zi.zi_adamw_step(pieces(state, [0] + np.cumsum(lengths).tolist()), zi.ZI_BF16, cfg)
    for part in pieces(whole, list(range(0, n, 800_000)) + [n]):
        zi.zi_adamw_step([part], zi.ZI_BF16, cfg)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(state, whole))
