"""Page-locked lists of more than 48 short tensors at the same places of five flat buffers: 256 to a launch of the step
over the link, with the bits of the chunk pipeline."""
import numpy as np
import pytest
import torch

import paper_2104_07857_amd as zi

pytestmark = pytest.mark.gpu
PER_LAUNCH = 256


def _step(eng, base, spans, dt, cfg, norm, lp, g_host, pacing):
    zi.zi_engine_set_option(eng, zi.ZI_OPT_MAX_INFLIGHT, pacing)
    bufs = []
    for w, x in enumerate(base):
        host = w < 3 or (g_host if w == 3 else lp == "host")
        if w == 4 and lp is None:
            bufs.append(None)
        elif host:
            y = torch.empty(x.shape, dtype=x.dtype, pin_memory=True)
            y.copy_(x)
            bufs.append(y)
        else:
            bufs.append(x.cuda())
    views = [tuple(None if x is None else x[s:s + n] for x in bufs) + (n,) for s, n in spans]
    status = zi.zi_adamw_step_streamed(eng, views, dt, cfg, norm)
    torch.cuda.synchronize()
    return status, zi.zi_engine_last_stats(eng), [None if x is None else x.cpu() for x in bufs]


@pytest.mark.parametrize("lp,g_host", [("device", False), ("host", True), (None, False)])
@pytest.mark.parametrize("count,l2,dt", [(48, False, zi.ZI_BF16), (49, True, zi.ZI_FP16), (256, False, zi.ZI_BF16), (257, False, zi.ZI_FP16),
                                         (700, True, zi.ZI_BF16)])
def test_flat_lists_equal_the_chunk_pipeline(count, l2, dt, lp, g_host):
    rng = np.random.default_rng(count)
    lens = [int(x) for x in rng.integers(1, 200, count)]
    lens[3], lens[17], lens[count - 1] = 512 * 97 * 3 + 5, 512, 1
    starts = np.cumsum([9] + [n + int(x) for n, x in zip(lens, rng.integers(0, 70, count))])[:-1].tolist()
    total = starts[-1] + lens[-1] + 5
    gen = torch.Generator().manual_seed(count)
    base = [torch.empty(total).normal_(0.0, s, generator=gen) for s in (0.02, 1e-4, 1e-6, 1e-3)]
    base[2].abs_()
    base[3] = base[3].to(torch.bfloat16 if dt == zi.ZI_BF16 else torch.float16)
    base.append(torch.full((total,), 7.0, dtype=base[3].dtype))
    norm, g = torch.zeros(4, dtype=torch.float64, device="cuda:0"), base[3].cuda()
    spans = list(zip(starts, lens))
    zi.zi_grad_norm_noalloc([(None, None, None, g[s:s + n], None, n) for s, n in spans], dt, 1.0, norm)
    cfg = zi.make_config(step=7, max_grad_norm=0.05, mode=zi.ZI_MODE_ADAM_L2 if l2 else zi.ZI_MODE_ADAMW)
    eng = zi.zi_engine_create(0, 64 * 1024, 3)
    try:
        s1, st1, a = _step(eng, base, spans, dt, cfg, norm, lp, g_host, 0)
        s2, st2, b = _step(eng, base, spans, dt, cfg, norm, lp, g_host, 2)
        assert s1 == s2 == zi.ZI_OK and st1.n_copies == 0 and st2.n_copies > 0
        assert st1.n_kernels == (1 if count <= 48 else -(-count // PER_LAUNCH))
        assert (st1.bytes_h2d, st1.bytes_d2h, st1.n_slot_uses) == (st2.bytes_h2d, st2.bytes_d2h, st2.n_slot_uses)
        for x, y, z in zip(a, b, base):
            assert (x is None) == (y is None) and (x is None or torch.equal(x, y))
            if x is not None:                      # what lies between the tensors is as it was
                keep = torch.ones(total, dtype=torch.bool)
                for s, n in spans:
                    keep[s:s + n] = False
                assert torch.equal(x[keep], z[keep])
        assert not torch.equal(a[0], base[0])
        norm[2:3].view(torch.int32)[0] = 1         # found_inf: the list is skipped as a whole
        s3, st3, c = _step(eng, base, spans, dt, cfg, norm, lp, g_host, 0)
        assert s3 == zi.ZI_SKIPPED_OVERFLOW and st3.n_kernels == 0
        assert all(x is None or torch.equal(x, z) for x, z in zip(c, base))
    finally:
        zi.zi_engine_destroy(eng)
