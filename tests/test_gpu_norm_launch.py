"""The reduction in one launch: its last workgroup waits for the others' partials and makes the final sum."""
import ctypes
import math
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2104_07857_amd as zi
import zi_synth
from gpu_util import NormBuffers, progress, to_dev

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILE, GROUPS = 16384, 512
KEEP = 11 << 23                       # elements up to which the gradients are read with ordinary loads


def _grads(n, dt, seed):
    g = np.empty(n, np.uint16)
    zi_synth.fill_normal_lp(g, n, seed, zi_synth.STREAM_G, dt, std=1e-3 if dt == zi.ZI_BF16 else 65.536)
    return g


def _norm(views, dt, nb):
    zi.zi_grad_norm([(None, None, None, v, None, v.numel()) for v in views], dt, 2.0, nb.out, nb.ws)
    torch.cuda.synchronize()
    return nb.read()


@pytest.mark.parametrize("dt", [zi.ZI_BF16, zi.ZI_FP16])
@pytest.mark.parametrize("n", [TILE + 1, 2 * TILE, 63 * TILE + 9, 64 * TILE + 1, (GROUPS - 1) * TILE + 5, GROUPS * TILE,
                               (GROUPS + 1) * TILE + 3])
def test_every_number_of_workgroups(n, dt):
    """From two workgroups to more tiles than workgroups, whatever the workspace held before."""
    g = _grads(n + 3, dt, 40 + n)
    d = to_dev(g)[3:]
    want, _ = oracle.grad_sumsq([g[3:].copy()], dt)
    nb = NormBuffers()
    seen = set()
    for before in (0x00, 0xFF, 0x5A, None, None):                  # None: what the call before left
        if before is not None:
            nb.ws.fill_(before)
        got = _norm([d], dt, nb)
        # squares and their sums in double: n additions of 1.1e-16 each, most of them in another order
        assert got[2] == 0 and abs(got[0] - want) <= 1e-12 * want and abs(got[1] - math.sqrt(want) / 2) <= 1e-12 * got[1]
        seen.add(got)
    assert len(seen) == 1


@pytest.mark.parametrize("dt", [zi.ZI_BF16, zi.ZI_FP16])
@pytest.mark.parametrize("count", [2, 15, 16, 17, 319, 320, 321, 641])
def test_lists_around_the_lookup_s_limits(count, dt):
    """Groups of 16 tensors, 320 to a launch, one launch or several; tensors shorter than a vector and ends around a tile's at
    every distance from a 16-byte boundary."""
    rng = np.random.default_rng(count)
    lengths = [int(x) for x in rng.integers(1, 40, count)]
    for i in range(0, count, 3):
        lengths[i] = TILE * int(rng.integers(1, 4)) + int(rng.integers(-9, 16))
    starts = np.cumsum([1] + [n + int(x) for n, x in zip(lengths, rng.integers(0, 9, count))])[:-1].tolist()
    g = _grads(starts[-1] + lengths[-1] + 1, dt, count)
    want, _ = oracle.grad_sumsq([g[s:s + n].copy() for s, n in zip(starts, lengths)], dt)
    d, nb = to_dev(g), NormBuffers()
    views = [d[s:s + n] for s, n in zip(starts, lengths)]
    got = _norm(views, dt, nb)
    assert got[2] == 0 and abs(got[0] - want) <= 1e-12 * want and got == _norm(views, dt, nb)
    # an overflow in the last element of the last tensor is seen, one behind it is not
    for at, flag in ((starts[-1] + lengths[-1] - 1, 1), (starts[-1] + lengths[-1], 0)):
        h = g.copy()
        h[at] = 0x7F80 if dt == zi.ZI_BF16 else 0x7C00
        e = to_dev(h)
        assert _norm([e[s:s + n] for s, n in zip(starts, lengths)], dt, nb)[2] == flag


@pytest.mark.parametrize("n", [KEEP, KEEP + 1, KEEP + TILE + 7, 1 << 28, (1 << 28) + 1])
def test_both_ways_of_reading(n):
    g = to_dev(np.tile(_grads(1 << 16, zi.ZI_BF16, 3), n // (1 << 16) + 1))[:n]
    one, _ = oracle.grad_sumsq([g[:1 << 16].cpu().numpy().view(np.uint16)], zi.ZI_BF16)
    rest, _ = oracle.grad_sumsq([g[:n % (1 << 16)].cpu().numpy().view(np.uint16)], zi.ZI_BF16)
    want = one * (n // (1 << 16)) + rest
    got = _norm([g], zi.ZI_BF16, NormBuffers())
    assert got[2] == 0 and abs(got[0] - want) <= 1e-12 * want


def test_replays_of_a_captured_call_see_new_gradients():
    """A replay has the marks of the replay before it: its partials must not be taken for the new ones."""
    dt, n = zi.ZI_BF16, 40 * TILE + 77
    d = to_dev(_grads(n, dt, 5))
    nb, nb_e = NormBuffers(), NormBuffers()
    tl = zi.make_tensors([(None, None, None, d, None, n)])
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        graph.capture_begin()
        zi.zi_grad_norm(tl, dt, 1.0, nb.out, nb.ws, stream=side)
        graph.capture_end()
    for replay in range(6):
        d.copy_(to_dev(_grads(n, dt, 100 + replay)))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        zi.zi_grad_norm(tl, dt, 1.0, nb_e.out, nb_e.ws)
        torch.cuda.synchronize()
        want, _ = oracle.grad_sumsq([d.cpu().numpy().view(np.uint16)], dt)
        assert nb.read() == nb_e.read(), replay
        assert abs(nb.read()[0] - want) <= 1e-12 * want


def test_workspace_and_result_in_page_locked_memory():
    """The partials travel over the link then; the same bits."""
    dt, n = zi.ZI_FP16, 70 * TILE + 5
    d, nb = to_dev(_grads(n, dt, 21)), NormBuffers()
    want = _norm([d], dt, nb)
    out = torch.zeros(4, dtype=torch.float64, pin_memory=True)
    ws = torch.full((zi.zi_norm_workspace_bytes(),), 0x3C, dtype=torch.uint8, pin_memory=True)
    for _ in range(2):
        zi.zi_grad_norm([(None, None, None, d, None, n)], dt, 2.0, out, ws)
        torch.cuda.synchronize()
        assert (float(out[0]), float(out[1])) == want[:2] and int(out.view(torch.int32)[4]) == 0


@pytest.fixture(scope="module")
def launch(tmp_path_factory):
    rocm = "/opt/rocm/include"
    if shutil.which("g++") is None or not os.path.isdir(rocm):
        pytest.skip("no host compiler or no HIP headers")
    so, libdir = str(tmp_path_factory.mktemp("launch") / "norm_launch.so"), os.path.dirname(zi.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-isystem", rocm, "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(libdir, "csrc"), os.path.join(ROOT, "tests", "c", "norm_launch.cpp"), "-o", so,
                    "-L", libdir, "-lzi", "-Wl,-rpath," + libdir, "-Wl,--allow-shlib-undefined"], check=True)
    zi.lib()
    f = ctypes.CDLL(so).norm_launch
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_uint32,
                  ctypes.c_void_p, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_int]
    return f


@pytest.mark.parametrize("each,pieces,form,keep,before,accumulate", [
    (TILE * 2 + 1, 1, 0, 0, 0, 0), (TILE * 2 + 1, 1, 0, 1, 0, 0), (TILE * 600 + 11, 1, 0, 0, 0, 0), (TILE * 600 + 11, 1, 0, 1, 0, 0),
    (TILE * 2 + 1, 1, 1, 0, 0, 0), (TILE * 600 + 11, 1, 1, 1, 0, 1),                      # NormOne
    (TILE + 8, 5, 2, 1, 0, 0), (TILE * 30, 32, 2, 1, 0, 1),                               # NormFew
    (264, 1, 0, 1, 1, 0), (TILE + 8, 200, 0, 0, 321, 0), (TILE * 2, 300, 0, 1, 1024, 1), (TILE * 2, 300, 0, 0, 15871, 1)])
def test_a_last_workgroup_that_does_not_wait_does_all_the_work(launch, each, pieces, form, keep, before, accumulate):
    """With no patience at all the partials count as missing and the last workgroup goes over the launch's whole list; what the
    launches before left in the workspace, other gradients' partials among it, changes nothing.  Partials of earlier launches
    and an earlier result are added either way."""
    dt, n = zi.ZI_FP16, each * pieces
    nb = NormBuffers()
    older = np.random.default_rng(before).uniform(0.0, 1e3, before)
    bits = older.view(np.uint64)
    words = np.stack([bits << np.uint64(32) | np.uint64(3), bits >> np.uint64(32) << np.uint64(32) | np.uint64(5)], axis=1).copy()
    ws = nb.ws.view(torch.int64)
    ws[:2 * before].copy_(torch.from_numpy(words.view(np.int64).reshape(-1)))
    results = []
    for turn, patience in enumerate((0, 1 << 20, 0, 1 << 20)):
        progress(f"reduction of {pieces} x {each} elements, form {form}, keep {keep}, {before} before, patience {patience}")
        g = _grads(n, dt, 8 + min(turn, 2))                                               # the last two see the same gradients
        want = oracle.grad_sumsq([g], dt)[0] + math.fsum(older) + (7.5 if accumulate else 0.0)
        d = to_dev(g)
        nb.out.fill_(7.5)
        torch.cuda.synchronize()
        assert launch(d.data_ptr(), each, pieces, dt, form, keep, patience, nb.ws.data_ptr(), before, nb.out.data_ptr(), accumulate) == 0
        torch.cuda.synchronize()
        got = nb.read()
        assert got[2] == 0 and abs(got[0] - want) <= 1e-12 * want and abs(got[1] - math.sqrt(want) / 2) <= 1e-12 * got[1]
        results.append(got)
    assert results[0] != results[1] != results[2]


@pytest.mark.parametrize("count", [1, 2, 33, 320, 321, 700])
def test_captured_calls_give_the_bits_of_eager_ones(count):
    """Under capture a kernel of its own makes the final sum; both add in one order, over one launch's partials or several's."""
    rng = np.random.default_rng(count)
    lengths = [int(x) for x in rng.integers(1, 3 * TILE, count)]
    starts = np.cumsum([0] + lengths)[:-1].tolist()
    n = sum(lengths)
    d, nb, nb_e = to_dev(_grads(n, zi.ZI_BF16, 1)), NormBuffers(), NormBuffers()
    tl = zi.make_tensors([(None, None, None, d[s:s + k], None, k) for s, k in zip(starts, lengths)])
    out2 = torch.zeros(4, dtype=torch.float64, device="cuda:0")
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    zi.zi_grad_norm_noalloc(tl, zi.ZI_BF16, 1.0, out2)                                     # (finds the array's address)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        graph.capture_begin()
        zi.zi_grad_norm(tl, zi.ZI_BF16, 1.0, nb.out, nb.ws, stream=side)
        zi.zi_grad_norm_noalloc(tl, zi.ZI_BF16, 1.0, out2, stream=side)
        graph.capture_end()
    for replay in range(4):
        g = _grads(n, zi.ZI_BF16, 50 + replay)
        d.copy_(to_dev(g))
        torch.cuda.synchronize()
        graph.replay()
        zi.zi_grad_norm(tl, zi.ZI_BF16, 1.0, nb_e.out, nb_e.ws)
        torch.cuda.synchronize()
        want, _ = oracle.grad_sumsq([g[s:s + k].copy() for s, k in zip(starts, lengths)], zi.ZI_BF16)
        assert abs(nb.read()[0] - want) <= 1e-12 * want
        assert torch.equal(nb.out, nb_e.out) and torch.equal(out2, nb_e.out), replay
