"""Lists of more than 64 tensors: how they share launches (no GPU), and that a list gives every tensor the bits
that a call of its own gives it, where the lookup of the tensor and the overlap of the launches could go wrong."""
import gc

import numpy as np
import pytest
import torch

import paper_2104_07857_amd as zi
import zi_synth

TILE = 512


@pytest.fixture(scope="module", autouse=True)
def _leave_no_garbage():
    """Tensors that the tests so far left in reference cycles (raised errors hold frames) are freed here, not at some
    moment of a later test that compares the allocator's figures before and after a call."""
    yield
    gc.collect()


@pytest.mark.parametrize("count,per_launch", [(64, [32, 31, 1]), (65, [64, 1]), (129, [64, 64, 1])])
def test_long_lists_share_launches_of_64(count, per_launch):
    base, gap = 0x7F00_0000_0000, 1 << 36
    lens = [100 + 600 * (i % 7) for i in range(count)]
    lens[10] = 1 << 22                                             # launched alone only in the short list
    items, launches = zi.zi_plan_step([tuple(base + (5 * i + k) * gap for k in range(5)) + (n,) for i, n in enumerate(lens)])
    assert launches == len(per_launch)
    groups = {}
    for it in items:
        groups.setdefault(it.launch, []).append(it)
    assert sorted(len(g) for g in groups.values()) == sorted(per_launch)
    for g in groups.values():                                      # tiles of a launch are numbered densely, in order
        nxt = 0
        for it in g:
            assert it.first_tile == nxt and it.n_tiles == max(1, -(-((lens[it.tensor] - it.head) // 4) // (TILE // 4)))
            nxt += it.n_tiles


def test_flat_lists_share_launches_of_256():
    """Tensors at the same places of five buffers; one array out of step, or a copy missing, and it is 64 again."""
    base, gap, n = 0x7F00_0000_0000, 1 << 36, 300

    def plan(shift=0, missing=-1):
        t = [[base + k * gap + 1001 * i * (4 if k < 3 else 2) for k in range(5)] + [1000] for i in range(n)]
        t[n - 1][3] += 2 * shift
        if missing >= 0:
            t[missing][4] = None
        items, launches = zi.zi_plan_step([tuple(x) for x in t])
        assert len(items) == n and [it.tensor for it in items] == list(range(n))
        return launches

    assert plan() == 2 and plan(shift=1) == 5 and plan(missing=7) == 5


@pytest.mark.gpu
@pytest.mark.parametrize("flat", [True, False])
@pytest.mark.parametrize("clip,scale,norm_scale", [(0.0, 1.0, 1.0), (0.5, 2.0, 2.0), (0.7, 2.0, 2.0), (0.5, 3.0, 3.0), (0.5, 2.0, 4.0),
                                                   (1e9, 1.0, 1.0)])
@pytest.mark.parametrize("count,l2,dt", [(63, False, zi.ZI_BF16), (64, True, zi.ZI_FP16), (270, False, zi.ZI_FP16), (700, False, zi.ZI_BF16)])
def test_a_list_equals_its_tensors_one_by_one(count, l2, dt, clip, scale, norm_scale, flat):
    """Ragged tensors at odd offsets of flat buffers (some a tile or less, one longer than an XCD run of tiles, one
    of 2^22 elements in the middle), with a norm that clips or not, stepped twice in a row as a list and tensor by tensor; the copies at the
    same places as the other arrays or at others."""
    rng = np.random.default_rng(count)
    sizes = [int(x) for x in rng.integers(1, 4000, count)]
    sizes[3], sizes[7], sizes[20], sizes[count - 1] = 1, TILE, 1030 * TILE + 5, 2 * TILE + 3
    sizes.insert(30, (1 << 22) + 77)
    starts = np.cumsum([3] + [n + int(x) for n, x in zip(sizes, rng.integers(0, 9, len(sizes)))])[:-1]
    total = int(starts[-1]) + sizes[-1] + 4
    spec = zi_synth.StateSpec(11, dt, g_std=2e-3)
    host = [np.empty(total, np.float32) for _ in range(3)] + [np.empty(total, np.uint16)]
    for fill, a in zip((spec.fill_p, spec.fill_m, spec.fill_v, spec.fill_g), host):
        fill(a, total)

    def state():
        bufs = [torch.from_numpy(a.copy().view(np.int16) if a.dtype == np.uint16 else a.copy()).cuda() for a in host]
        skew = 0 if flat else 3
        bufs.append(torch.full((total + skew * len(sizes),), 7, dtype=torch.int16, device="cuda:0"))
        return bufs, [tuple(b[s:s + n] for b in bufs[:4]) + (bufs[4][s + skew * i:s + skew * i + n], n)
                      for i, (s, n) in enumerate(zip(starts.tolist(), sizes))]

    cfg = zi.make_config(step=10, loss_scale=scale, max_grad_norm=clip, mode=zi.ZI_MODE_ADAM_L2 if l2 else zi.ZI_MODE_ADAMW)
    (a, ta), (b, tb) = state(), state()
    norm = torch.zeros(4, dtype=torch.float64, device="cuda:0")
    for _ in range(2):
        zi.zi_grad_norm_noalloc(ta, dt, norm_scale, norm)
        zi.zi_adamw_step(ta, dt, cfg, norm)
    for _ in range(2):
        for t in tb:
            zi.zi_adamw_step([t], dt, cfg, norm)
    torch.cuda.synchronize()
    assert float(norm[1]) * norm_scale / scale > 0.7 or clip == 1e9      # the thresholds do clip
    for x, y in zip(a, b):                                          # what lies between the tensors included
        assert torch.equal(x.view(torch.int32 if x.dtype == torch.float32 else torch.int16),
                           y.view(torch.int32 if y.dtype == torch.float32 else torch.int16))


@pytest.mark.gpu
def test_an_overflow_skips_a_long_list():
    tl, bufs = [], []
    for i in range(70):
        b = [torch.full((1000 + i,), 0.5, device="cuda:0") for _ in range(3)]
        b += [torch.ones(1000 + i, dtype=torch.bfloat16, device="cuda:0"), torch.full((1000 + i,), 7, dtype=torch.int16, device="cuda:0")]
        bufs.append(b)
        tl.append(tuple(b) + (1000 + i,))
    bufs[69][3][-1] = float("inf")
    norm = torch.zeros(4, dtype=torch.float64, device="cuda:0")
    zi.zi_grad_norm_noalloc(tl, zi.ZI_BF16, 1.0, norm)
    zi.zi_adamw_step(tl, zi.ZI_BF16, zi.make_config(step=1, max_grad_norm=1.0), norm)
    torch.cuda.synchronize()
    for p, m, v, _, lp in bufs:
        assert bool((p == 0.5).all()) and bool((m == 0.5).all()) and bool((v == 0.5).all()) and bool((lp == 7).all())
