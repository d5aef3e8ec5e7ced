"""The step on the host CPUs: what it does around the step itself (the norm result's way, a skipped step, calls that follow
one another through the same ring)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2104_07857_amd as zi
import zi_synth
from gpu_util import NormBuffers, compare_state, gen_numpy, to_dev, to_np

pytestmark = pytest.mark.gpu
CHUNK = 64 * 1024                                    # 16,384 elements: one block


def engine():
    e = zi.zi_engine_create(0, CHUNK, 3)
    zi.zi_engine_set_option(e, zi.ZI_OPT_HOST_RING_SLOTS, 4)
    return e


def config(**over):
    return dict(dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01, step=10, loss_scale=1.0, max_grad_norm=0.5), **over)


# The norm in device memory is brought by a kernel, one in page-locked memory by the runtime; several steps on one ring, of one use,
# as many as it has slots, and more.
@pytest.mark.parametrize("pinned_norm", [False, True])
@pytest.mark.parametrize("n,threads", [(1, 16), (1000, 1), (16384, 16), (16385, 3), (4 * 16384, 16), (9 * 16384 + 77, 5)])
def test_steps_in_a_row(n, threads, pinned_norm):
    dt = zi.ZI_BF16 if n % 2 else zi.ZI_FP16
    p, m, v, _ = gen_numpy(zi_synth.StateSpec(n, dt), n)
    state = [torch.from_numpy(x.copy()) for x in (p, m, v)]
    lp = torch.zeros(n, dtype=torch.int16, device="cuda:0")
    elp = np.zeros(n, np.uint16)
    e, nb = engine(), NormBuffers()
    try:
        for step in range(1, 6):
            g = gen_numpy(zi_synth.StateSpec(n + step, dt), n)[3]
            dg = to_dev(g.copy())
            overflow = step == 3
            if overflow:
                dg[n // 2] = 0x7F80 if dt == zi.ZI_BF16 else 0x7C00
            zi.zi_grad_norm([(None, None, None, dg, None, n)], dt, 1.0, nb.out, nb.ws)
            norm = nb.out
            if pinned_norm:
                norm = torch.empty(4, dtype=torch.float64, pin_memory=True)
                norm.copy_(nb.out)
            status = zi.zi_adamw_step_cpu(e, [(*state, dg, lp, n)], dt, zi.make_config(**config(step=step)), norm, threads)
            if overflow:
                assert status == zi.ZI_SKIPPED_OVERFLOW
                st = zi.zi_engine_last_stats(e)
                assert st.bytes_d2h == 0 and st.bytes_h2d == 0 and st.n_slot_uses == 0
            else:
                assert status == zi.ZI_OK
                sumsq, flag = oracle.grad_sumsq([g], dt)
                oracle.adamw(p, m, v, g, elp, dt, oracle.config(**config(step=step)), sumsq, flag)
            compare_state((p, m, v, elp), [x.numpy() for x in state] + [to_np(lp)], dt, f"step {step} ")
    finally:
        zi.zi_engine_destroy(e)


def test_a_captured_stream_is_refused():
    n = 1000
    p, m, v, g = gen_numpy(zi_synth.StateSpec(3, zi.ZI_BF16), n)
    dg, e = to_dev(g), engine()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    x = torch.zeros(8, device="cuda:0")
    torch.cuda.synchronize()
    try:
        with torch.cuda.stream(stream):
            graph.capture_begin()
            x.add_(1)
            with pytest.raises(Exception):
                zi.zi_adamw_step_cpu(e, [tuple(torch.from_numpy(a) for a in (p, m, v)) + (dg, None, n)], zi.ZI_BF16,
                                     zi.make_config(**config()), None, 2, stream)
            graph.capture_end()
        graph.replay()
        torch.cuda.synchronize()
        assert float(x.sum()) == 8.0
    finally:
        zi.zi_engine_destroy(e)
