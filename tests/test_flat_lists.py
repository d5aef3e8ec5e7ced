"""Lists of 33 to 64 short tensors that are views at the same places of five flat buffers: one launch."""
import numpy as np
import pytest
import torch

import paper_2104_07857_amd as zi

BASE, GAP = 0x7F00_0000_0000, 1 << 36
LIMIT = 5 << 16                       # average length up to which such tensors count as short


def _launches(count, length, shift=0):
    t = [[BASE + k * GAP + (length + 3) * i * (4 if k < 3 else 2) for k in range(5)] + [length] for i in range(count)]
    t[-1][4] += 2 * shift
    items, launches = zi.zi_plan_step([tuple(x) for x in t])
    assert [it.tensor for it in items] == list(range(count))
    return launches


@pytest.mark.parametrize("count", [32, 33, 64])
def test_which_lists_are_one_launch(count):
    two = 1 if count == 32 else 2
    assert _launches(count, 1000) == _launches(count, LIMIT) == 1
    assert _launches(count, LIMIT + 1) == two and _launches(count, 1000, shift=1) == two


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [zi.ZI_BF16, zi.ZI_FP16])
@pytest.mark.parametrize("count,most", [(2, 0), (2, 1), (16, 0), (17, 0), (32, 0), (32, 1), (33, 0), (64, 0)])
def test_every_tensor_as_by_itself(count, most, dt):
    """Up to 32 tensors with 2^21 elements in all have arguments of their own; most: one element more."""
    rng = np.random.default_rng(count)
    sizes = [int(x) for x in rng.integers(1, 3000, count)]
    sizes[min(5, count - 2)], sizes[-1] = 1030 * 512 + 5, 1
    if count <= 32:
        sizes[0] += (1 << 21) + most - sum(sizes)
    starts = np.cumsum([7] + [n + int(x) for n, x in zip(sizes, rng.integers(0, 9, count))])[:-1].tolist()
    total = starts[-1] + sizes[-1] + 3
    gen = torch.Generator(device="cuda:0").manual_seed(count)
    a = [torch.empty(total, device="cuda:0").normal_(0.0, s, generator=gen) for s in (0.02, 1e-4, 1e-6, 1e-3)]
    a[2].abs_()
    a[3] = a[3].to(torch.bfloat16 if dt == zi.ZI_BF16 else torch.float16)
    a.append(torch.full((total,), 7.0, dtype=a[3].dtype, device="cuda:0"))
    b = [x.clone() for x in a]
    views = lambda bufs: [tuple(x[s:s + n] for x in bufs) + (n,) for s, n in zip(starts, sizes)]      # noqa: E731
    norm, cfg = torch.zeros(4, dtype=torch.float64, device="cuda:0"), zi.make_config(step=3, max_grad_norm=0.5)
    zi.zi_grad_norm_noalloc(views(a), dt, 1.0, norm)
    zi.zi_adamw_step(views(a), dt, cfg, norm)
    for t in views(b):
        zi.zi_adamw_step([t], dt, cfg, norm)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)
