"""Sums of squares that every order of adding gives exactly: gradients that are whole numbers of up to eight bits.  A lane
whose share is lost or counted twice on the way through a wavefront, a workgroup or the partials changes the result."""
import numpy as np
import pytest
import torch

import paper_2104_07857_amd as zi
from gpu_util import NormBuffers

pytestmark = pytest.mark.gpu


def gradients(numels, dt, seed, offset):
    """Views into one buffer, and the sum of their squares."""
    r = np.random.default_rng(seed)
    host = r.integers(-127, 128, offset + sum(numels) + 8)
    flat = torch.from_numpy(host.astype(np.float32)).to(torch.bfloat16 if dt == zi.ZI_BF16 else torch.float16).to("cuda:0")
    at, tensors, total = offset, [], 0
    for n in numels:
        tensors.append((None, None, None, flat[at:at + n], None, n))
        total += int((host[at:at + n].astype(np.int64) ** 2).sum())
        at += n
    return flat, tensors, total


@pytest.mark.parametrize("dt", [zi.ZI_BF16, zi.ZI_FP16])
@pytest.mark.parametrize("numels", [[1], [63], [64], [65], [513], [4095], [4096], [4097], [4104, 1], [16_384], [16_385], [70_001],
                                    [1 << 20], [(1 << 20) + 1], [1 << 19, (1 << 19) + 8], [(1 << 21) + 3], [3_000_001], [8, 4096, 9, 1, 16_384, 77], [1000] * 32, [5000] * 33,
                                    [20_000] * 100, [3270] * 320, [3270] * 321, [7] * 700])
def test_whole_numbers_sum_exactly(numels, dt):
    for offset in (0, 3):
        flat, tensors, total = gradients(numels, dt, len(numels) + numels[0], offset)
        nb = NormBuffers()
        zi.zi_grad_norm(tensors, dt, 1.0, nb.out, nb.ws)
        assert float(nb.out[0].item()) == float(total)
        zi.zi_grad_norm_noalloc(tensors, dt, 1.0, nb.out)
        assert float(nb.out[0].item()) == float(total)
