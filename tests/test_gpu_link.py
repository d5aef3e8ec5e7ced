"""The step that reads and writes page-locked state over the link, against the oracle and against the chunk
pipeline (which a chosen pacing selects), at the places where its tiles, ends and launches change."""
import numpy as np
import pytest
import torch

import oracle
import paper_2104_07857_amd as zi
import zi_synth
from gpu_util import NormBuffers, compare_state, gen_numpy, oracle_cfg, progress, to_dev, to_np, zi_cfg

pytestmark = pytest.mark.gpu

TILE, GROUPS, DESCS = 512, 96, 48


def _placed(a, offset, host):
    """A copy of `a` that starts `offset` elements into a buffer of its own, with guard elements behind."""
    buf = torch.full((a.size + offset + 8,), 7, dtype=torch.int16 if a.dtype == np.uint16 else torch.float32)
    src = torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a)
    buf[offset:offset + a.size] = src
    if not host:
        return buf.cuda()
    pinned = torch.empty(buf.shape, dtype=buf.dtype, pin_memory=True)
    pinned.copy_(buf)
    return pinned


def _run(host, offsets, dt, cfg, *, g_host, lp_host, lp, pacing, norm=False):
    """One streamed step; returns status, stats and every buffer (guards included) on the host."""
    eng = zi.zi_engine_create(0, 64 * 1024, 3)
    try:
        zi.zi_engine_set_option(eng, zi.ZI_OPT_MAX_INFLIGHT, pacing)
        bufs, tl = [], []
        for (p, m, v, g), o in zip(host, offsets):
            n = p.size
            b = [_placed(p, o, True), _placed(m, o, True), _placed(v, o, True), _placed(g, o, g_host)]
            b.append(_placed(np.zeros(n, np.uint16), o, lp_host) if lp else None)
            bufs.append(b)
            tl.append(tuple(None if x is None else x[o:o + n] for x in b) + (n,))
        nb = None
        if norm:
            nb = NormBuffers()
            zi.zi_grad_norm([(None, None, None, t[3], None, t[5]) for t in tl], dt, cfg.loss_scale, nb.out, nb.ws)
        status = zi.zi_adamw_step_streamed(eng, tl, dt, cfg, nb.out if nb else None, torch.cuda.current_stream())
        return status, zi.zi_engine_last_stats(eng), [[None if x is None else to_np(x) for x in b] for b in bufs]
    finally:
        zi.zi_engine_destroy(eng)


def _same(a, b):
    for x, y in zip(a, b):
        for u, v in zip(x, y):
            assert (u is None) == (v is None)
            if u is not None:
                assert np.array_equal(u.view(np.uint8), v.view(np.uint8))


@pytest.mark.parametrize("offset", [0, 1, 2, 61, 63])
@pytest.mark.parametrize("n", [1, 3, 64, 67, TILE - 1, TILE + 1, GROUPS * TILE, GROUPS * TILE + 5, 3 * GROUPS * TILE + 259])
def test_sizes_and_offsets_against_the_oracle(n, offset):
    """Heads of 0, 63, 62, 3 and 1 elements with every tail: a head of 62 or 63 leaves less than three lanes to it."""
    w = zi_synth.workload("c2")
    dt = zi.ZI_BF16 if n % 2 else zi.ZI_FP16
    host = [gen_numpy(zi_synth.StateSpec(9000 + n, dt), n)]
    ep, em, ev, g = (a.copy() for a in host[0])
    elp = np.zeros(n, np.uint16)
    oracle.step([(ep, em, ev, g, elp)], dt, oracle_cfg(w), False)
    status, st, got = _run(host, [offset], dt, zi_cfg(w), g_host=False, lp_host=False, lp=True, pacing=0)
    assert status == zi.ZI_OK and st.n_copies == 0 and st.n_kernels == 1
    inside = [x[offset:offset + n] for x in got[0]]
    compare_state((ep, em, ev, elp), (inside[0], inside[1], inside[2], inside[4]), dt, f"n={n} offset={offset} ")
    for x in got[0]:                                           # nothing around the tensor was touched
        assert (x[:offset] == 7).all() and (x[offset + n:] == 7).all()


@pytest.mark.parametrize("g_host", [False, True])
@pytest.mark.parametrize("lp", [None, "device", "host"])
@pytest.mark.parametrize("l2,dt", [(False, zi.ZI_FP16), (True, zi.ZI_BF16)])
def test_lists_equal_the_chunk_pipeline(g_host, lp, l2, dt):
    """More tensors than one launch takes, ragged and misaligned, every placement of gradients and copy: the
    same bits as the chunk pipeline, which a pacing of two uses selects."""
    rng = np.random.default_rng(5)
    sizes = [int(x) for x in rng.integers(1, 3000, 2 * DESCS + 3)] + [70_001]
    offsets = [int(x) for x in rng.integers(0, 64, len(sizes))]
    scale = 1024.0 if dt == zi.ZI_FP16 else 1.0
    spec = zi_synth.StateSpec(31, dt, g_std=2e-3 * scale)
    host = [gen_numpy(spec, n, tensor=i) for i, n in enumerate(sizes)]
    cfg = zi_cfg(zi_synth.workload("c4"), loss_scale=scale, max_grad_norm=0.7,
                 mode=zi.ZI_MODE_ADAM_L2 if l2 else zi.ZI_MODE_ADAMW)
    kw = dict(g_host=g_host, lp_host=lp == "host", lp=lp is not None, norm=not g_host)
    s1, st1, a = _run(host, offsets, dt, cfg, pacing=0, **kw)
    s2, st2, b = _run(host, offsets, dt, cfg, pacing=2, **kw)
    assert s1 == s2 == zi.ZI_OK
    assert st1.n_copies == 0 and st1.n_kernels == 3 and st2.n_copies > 0
    assert (st1.bytes_h2d, st1.bytes_d2h, st1.n_slot_uses) == (st2.bytes_h2d, st2.bytes_d2h, st2.n_slot_uses)
    _same(a, b)
    progress(f"link step, {len(sizes)} tensors, g_host={g_host}, lp={lp}: equal to the chunk pipeline")


def test_overflow_skips_and_touches_nothing():
    w = zi_synth.workload("c2")
    host = [gen_numpy(zi_synth.StateSpec(77, zi.ZI_BF16), n) for n in (5000, 70_000)]
    host[1][3][1234] = 0x7F80
    status, st, got = _run(host, [0, 3], zi.ZI_BF16, zi_cfg(w), g_host=False, lp_host=True, lp=True, pacing=0, norm=True)
    assert status == zi.ZI_SKIPPED_OVERFLOW
    assert st.bytes_h2d == st.bytes_d2h == 0 and st.n_kernels == 0 and st.n_slot_uses == 0
    for (p, m, v, _), b, o in zip(host, got, (0, 3)):
        for x, y in zip((p, m, v, np.zeros(p.size, np.uint16)), (b[0], b[1], b[2], b[4])):
            assert np.array_equal(x.view(np.uint8), y[o:o + x.size].view(np.uint8))


SOLO = 32768                          # elements one pass of the one-workgroup reduction covers


@pytest.mark.parametrize("offset", [0, 1, 7])
@pytest.mark.parametrize("sizes", [[SOLO - 1], [SOLO + 9], [4 * SOLO], [4 * SOLO + 7], [4 * SOLO + 16], [5, 3 * SOLO],
                                   [5, 6, 7, 8], [5, 6, 7, 8, 9], [3] * 224, [3] * 225, [512 * 16384 + 11, 1]])
def test_norm_of_device_and_page_locked_gradients(sizes, offset):
    """Around the one-workgroup limit, the tensors a launch takes and the workgroups a launch has: the sum against
    the oracle for gradients in HBM and in host memory, and the flag from the very last element."""
    dt = zi.ZI_FP16 if offset else zi.ZI_BF16
    gs = [gen_numpy(zi_synth.StateSpec(60 + n, dt, g_std=1e-2), n, tensor=i)[3] for i, n in enumerate(sizes)]
    want, _ = oracle.grad_sumsq(gs, dt)
    eng = zi.zi_engine_create(0, 64 * 1024, 3)
    try:
        for planted in (False, True):
            if planted:
                gs[-1][-1] = 0x7C00 if dt == zi.ZI_FP16 else 0x7F80
            flags, sums = [], []
            for host in (False, True):
                bufs = [_placed(g, offset, host) for g in gs]
                tl = [(None, None, None, b[offset:offset + g.size], None, g.size) for b, g in zip(bufs, gs)]
                nb = NormBuffers()
                if host:
                    zi.zi_grad_norm_streamed(eng, tl, dt, 2.0, nb.out, nb.ws)
                    st = zi.zi_engine_last_stats(eng)
                    assert st.n_copies == 0 and st.bytes_h2d == 2 * sum(sizes)
                else:
                    zi.zi_grad_norm(tl, dt, 2.0, nb.out, nb.ws)
                    torch.cuda.synchronize()
                sumsq, norm, flag = nb.read()
                flags.append(flag)
                sums.append((sumsq, norm))
            assert flags == [int(planted)] * 2
            if not planted:
                for sumsq, norm in sums:
                    assert abs(sumsq - want) <= 1e-12 * want          # double sums of exact squares on both sides
                    assert abs(norm - np.sqrt(want) / 2.0) <= 1e-12 * norm
    finally:
        zi.zi_engine_destroy(eng)


BLOCK = 16384                         # elements of one block of the copies of the CPU placement


@pytest.mark.parametrize("offset", [0, 1, 6])
@pytest.mark.parametrize("sizes", [[1], [7, 8, 9], [BLOCK - 1], [BLOCK], [BLOCK + 1], [64 * BLOCK + 3], [5] * 33 + [BLOCK + 5] + [1] * 33,
                                   [3 * 65536 + 11, 200, 2 * 65536]])
def test_cpu_placement_at_block_edges(sizes, offset):
    """Gradients and copy at odd places in HBM, state in host memory: tensors of less than a vector to several slot uses,
    more segments than a use packs; the same bits as the step that goes over the link, twice in a row on one engine."""
    dt = zi.ZI_BF16
    host = [gen_numpy(zi_synth.StateSpec(500 + len(sizes), dt), n, tensor=i) for i, n in enumerate(sizes)]
    cfg = zi_cfg(zi_synth.workload("c4"))
    results = []
    eng = zi.zi_engine_create(0, 256 * 1024, 3)              # 65,536-element chunks: four blocks to a use
    try:
        zi.zi_engine_set_option(eng, zi.ZI_OPT_HOST_RING_SLOTS, 3)
        for cpu in (True, False):
            bufs, tl = [], []
            for i, (p, m, v, g) in enumerate(host):
                b = [_placed(p, 0, True), _placed(m, 0, True), _placed(v, 0, True), _placed(g, offset, False),
                     _placed(np.zeros(p.size, np.uint16), offset, False) if i % 3 != 2 else None]
                bufs.append(b)
                tl.append((b[0][:p.size], b[1][:p.size], b[2][:p.size], b[3][offset:offset + p.size],
                           None if b[4] is None else b[4][offset:offset + p.size], p.size))
            for _ in range(2):
                if cpu:
                    assert zi.zi_adamw_step_cpu(eng, tl, dt, cfg, None, 3) == zi.ZI_OK
                    st = zi.zi_engine_last_stats(eng)
                    assert st.bytes_d2h == 2 * sum(sizes)
                    assert st.bytes_h2d == 2 * sum(n for i, n in enumerate(sizes) if i % 3 != 2)
                else:
                    assert zi.zi_adamw_step_streamed(eng, tl, dt, cfg) == zi.ZI_OK
            results.append([[None if x is None else to_np(x) for x in b] for b in bufs])
    finally:
        zi.zi_engine_destroy(eng)
    _same(*results)


@pytest.mark.parametrize("nbytes", [1, 2, 6, 16, 8190, 8192, 8194, 100_001, (4 << 20) - 2, 4 << 20, (4 << 20) + 2])
@pytest.mark.parametrize("offset", [0, 2, 3, 14])
def test_offloaded_bytes_arrive(nbytes, offset):
    """Short and long partitions, odd counts and addresses among them: the bytes arrive, nothing around them changes, and a
    stream that is ordered behind the offload reads them."""
    src = torch.randint(0, 256, (nbytes + 64,), dtype=torch.uint8, device="cuda:0")
    dst = torch.full((nbytes + 64,), 7, dtype=torch.uint8).pin_memory()
    back = torch.zeros(nbytes + 64, dtype=torch.uint8, device="cuda:0")
    eng = zi.zi_engine_create(0, 64 * 1024, 3)
    try:
        zi.zi_grad_offload(eng, src.data_ptr() + offset, dst.data_ptr() + 2 * offset, nbytes, torch.cuda.current_stream())
        side = torch.cuda.Stream()
        zi.zi_grad_offload_order(eng, side)
        with torch.cuda.stream(side):
            back.copy_(dst, non_blocking=True)
        side.synchronize()
        zi.zi_grad_offload_wait(eng)
    finally:
        zi.zi_engine_destroy(eng)
    want = torch.full((nbytes + 64,), 7, dtype=torch.uint8)
    want[2 * offset:2 * offset + nbytes] = src.cpu()[offset:offset + nbytes]
    assert torch.equal(dst, want) and torch.equal(back.cpu(), want)
