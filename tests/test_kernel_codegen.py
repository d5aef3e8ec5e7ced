"""Properties of the compiled fused-step kernels that their bandwidth depends on, read from the
assembly hipcc emits for the library's own source (no GPU needed):

  * no scratch memory, and few enough vector registers for the wavefronts that a launch asks for: five on a SIMD for kernels
    of fine tiles (18 workgroups of one wavefront per compute unit), four for the others (16);
  * the norm result is read with one scalar load: nothing enters the vector memory pipeline before a
    wavefront's streaming loads (a vector load issued under a saturated stream queues behind it), and
    the result's fields are not fetched one dependent round trip at a time; in kernels over lists it travels beside the
    table of starts;
  * whole tiles issue their eight non-temporal loads back to back, before the first wait on any of them, and fine tiles their four;
  * paced kernels ask for a quad's loads when those before have arrived, and for its stores when those before are done;
  * every streaming access is non-temporal.

Of the kernels over the link and of the reduction only scratch, registers and the kind of loads are looked at.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2104_07857_amd import build as zb

KERNEL = re.compile(r"^(_ZN2zi17adamw_wide_kernelILi([01])ELb([01])EEEvNS_8StepArgsE):", re.M)
LIST_KERNEL = re.compile(r"^(_ZN2zi17adamw_list_kernelILi([01])ELb([01])ENS_(8ListArgs|8FlatArgs|7FlatFew)EEEvT1_):", re.M)
FINE_KERNEL = re.compile(r"^(_ZN2zi17adamw_fine_kernelILi([01])ELb([01])EEEvNS_7StepOneE):", re.M)
FINE_LIST_KERNEL = re.compile(
    r"^(_ZN2zi22adamw_fine_list_kernelILi([01])ELb([01])ELb([01])ENS_(8ListArgs|8FlatArgs|7FlatFew)EEEvT2_):", re.M)
PACED_KERNEL = re.compile(r"^(_ZN2zi18adamw_paced_kernelILi([01])ELb([01])ELi([234])EEEvNS_7StepOneE):", re.M)
PACED_LIST_KERNEL = re.compile(r"^(_ZN2zi23adamw_paced_list_kernelILi([01])ELb([01])ENS_(8ListArgs|8FlatArgs|7FlatFew)EEEvT1_):", re.M)
NORM_KERNEL = re.compile(r"^(_ZN2zi20sumsq_partial_kernelILi([01])ELb([01])ENS_(7NormOne|7NormFew|8NormArgs)EEEvT1_):", re.M)
SHORT_NORM_KERNEL = re.compile(r"^(_ZN2zi26short_sumsq_partial_kernelILi([01])ENS_(7NormOne|7NormFew|8NormArgs)EEEvT0_):", re.M)
LINK_KERNEL = re.compile(r"^(_ZN2zi(?:17adamw_link|22adamw_link_flat)_kernelILi([01])ELb([01])EEEvNS_(8LinkArgs|12LinkFlatArgs)E):", re.M)


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if shutil.which(zb.hipcc()) is None and not os.path.exists(zb.hipcc()):
        pytest.skip("no hipcc here")
    out = tmp_path_factory.mktemp("isa") / "zi_kernels.s"
    flags = [f for f in zb.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [zb.hipcc(), *flags, "-I", os.path.join(zb.ROOT, "include"), "-I", zb.CSRC, "-S", "--cuda-device-only",
           "-o", str(out), os.path.join(zb.CSRC, "zi_kernels.hip")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


def _kernels(text, pattern):
    return {mt.groups()[1:]: text[mt.end():text.index(".end_amdhsa_kernel", mt.end())] for mt in pattern.finditer(text)}


@pytest.fixture(scope="module")
def step_kernels(assembly):
    kernels = {tuple(int(x) for x in key): body for key, body in _kernels(assembly, KERNEL).items()}
    assert len(kernels) == 4, sorted(kernels)      # {bf16, fp16} x {AdamW, Adam+L2}
    return kernels


@pytest.fixture(scope="module")
def list_kernels(assembly):
    kernels = _kernels(assembly, LIST_KERNEL)
    assert len(kernels) == 8, sorted(kernels)      # {bf16, fp16} x {AdamW, Adam+L2} x {any list, flat buffers} (few of them: never whole tiles)
    return kernels


@pytest.fixture(scope="module")
def fine_kernels(assembly):
    one, lists = _kernels(assembly, FINE_KERNEL), _kernels(assembly, FINE_LIST_KERNEL)
    assert len(one) == 4, sorted(one)              # {bf16, fp16} x {AdamW, Adam+L2}
    assert len(lists) == 16, sorted(lists)         # ... x {any list, in XCD runs and in plain order, flat buffers, few of them}
    return one, lists


@pytest.fixture(scope="module")
def paced_kernels(assembly):
    one, lists = _kernels(assembly, PACED_KERNEL), _kernels(assembly, PACED_LIST_KERNEL)
    assert len(one) == 12, sorted(one)             # {bf16, fp16} x {AdamW, Adam+L2} x {two, three, four quads a lane}
    assert len(lists) == 12, sorted(lists)         # {bf16, fp16} x {AdamW, Adam+L2} x {any list, flat buffers, few of them}
    return one, lists


def instructions(body):
    out = []
    for line in body.splitlines():
        line = line.split(";")[0].strip()
        if line and not line.startswith(".") and not line.endswith(":"):
            out.append(line)
    return out


def directive(body, name):
    m = re.search(r"\.amdhsa_" + name + r"\s+(\d+)", body)
    assert m, name
    return int(m.group(1))


def test_no_scratch_and_four_wavefronts_per_simd_fit(step_kernels, list_kernels, paced_kernels, assembly):
    link = _kernels(assembly, LINK_KERNEL)
    assert len(link) == 8, sorted(link)            # {bf16, fp16} x {AdamW, Adam+L2} x {any list, flat buffers}
    one, lists = paced_kernels
    for key, body in [*step_kernels.items(), *list_kernels.items(), *one.items(), *lists.items(), *link.items()]:
        assert directive(body, "private_segment_fixed_size") == 0, key
        assert directive(body, "next_free_vgpr") <= 128, key
        assert "scratch_" not in body and "buffer_" not in body, key


def test_five_wavefronts_of_fine_tiles_per_simd_fit(fine_kernels):
    one, lists = fine_kernels
    for key, body in [*one.items(), *lists.items()]:
        assert directive(body, "private_segment_fixed_size") == 0, key
        assert directive(body, "next_free_vgpr") <= 96, key          # of 512, in eights
        assert "scratch_" not in body and "buffer_" not in body and "flat_" not in body.split(".amdhsa_kernel")[0], key


def test_reduction_reads_all_gradients_one_way(assembly):
    """Ordinary loads leave the gradients in the memory-side cache, and whatever a kernel has just written there has to leave
    first; an instantiation with streaming loads has no others."""
    kernels = _kernels(assembly, NORM_KERNEL)
    assert len(kernels) == 10, sorted(kernels)     # {bf16, fp16} x ({streaming, ordinary} x {one tensor, list}, short list)
    for key, body in kernels.items():
        loads = [x for x in instructions(body) if x.startswith("buffer_load_dwordx4")]
        assert len(loads) == (4 if key[1] == "1" else 8), (key, loads)
        assert all(x.endswith(" nt") == (key[1] == "0") for x in loads), (key, loads)
        assert directive(body, "private_segment_fixed_size") == 0, key


def test_short_reductions_read_a_vector_a_thread(assembly):
    kernels = _kernels(assembly, SHORT_NORM_KERNEL)
    assert len(kernels) == 6, sorted(kernels)      # {bf16, fp16} x {one tensor, short list, list}
    for key, body in kernels.items():
        loads = [x for x in instructions(body) if x.startswith("buffer_load")]
        assert len(loads) == 1 and loads[0].startswith("buffer_load_dwordx4") and not loads[0].endswith(" nt"), (key, loads)
        assert directive(body, "private_segment_fixed_size") == 0 and directive(body, "next_free_vgpr") <= 64, key


def test_norm_result_is_read_with_one_scalar_load(step_kernels, fine_kernels, paced_kernels):
    """Up to the prologue's fp64 arithmetic (the clip factor) the kernel has touched memory only through
    scalar loads: its arguments (base s[0:1]) and one 32-byte load of the whole norm result from another
    base; no vector memory instruction, and no field-by-field reads of the result."""
    for key, body in [*step_kernels.items(), *fine_kernels[0].items(), *paced_kernels[0].items()]:
        ins = instructions(body)
        first_f64 = next(i for i, x in enumerate(ins) if x.startswith(("v_div_scale_f64", "v_sqrt_f64", "v_rsq_f64",
                                                                       "v_mul_f64", "v_add_f64")))
        head = ins[:first_f64]
        assert not [x for x in head if x.startswith(("global_", "flat_", "buffer_", "scratch_"))], key
        other = [x for x in head if x.startswith("s_load") and not re.search(r", s\[0:1\], ", x)]
        assert len(other) == 1, (key, other)
        assert re.match(r"s_load_dwordx8 s\[\d+:\d+\], s\[\d+:\d+\], 0x0$", other[-1]), (key, other)


def test_long_lists_fetch_the_norm_result_beside_their_starts(list_kernels, fine_kernels, paced_kernels):
    """Nothing but scalar loads in front of a wavefront's first streaming load; the norm result is one 32-byte load, and no
    wait separates it from the load of the group's starts (fetched behind the descriptor it cost 8%)."""
    for key, body in [*list_kernels.items(), *fine_kernels[1].items(), *paced_kernels[1].items()]:
        ins = instructions(body)
        head = ins[:next(i for i, x in enumerate(ins) if x.startswith("global_"))]
        assert not [x for x in head if x.startswith(("flat_", "buffer_", "scratch_"))], key
        result = [i for i, x in enumerate(head) if re.match(r"s_load_dwordx8 s\[\d+:\d+\], s\[(?!0:1\])\d+:\d+\], 0x0$", x)]
        assert result, key
        wait = next(i for i in range(result[0], len(head)) if head[i].startswith("s_waitcnt"))
        starts = [x for x in head[result[0] + 1:wait] if re.match(r"s_load_dwordx(8|16) .*, 0x[1-9a-f]", x)]
        assert starts, (key, head[result[0]:wait + 1])


def test_full_tile_issues_all_loads_before_the_first_wait(step_kernels, list_kernels):
    for key, body in [*step_kernels.items(), *list_kernels.items()]:
        ins = instructions(body)
        # the full-tile block is the only place with non-temporal 16-byte loads at an immediate offset of one
        # wavefront row (the second quad of a lane)
        start = next(i for i, x in enumerate(ins) if x.startswith("global_load_dwordx") and x.endswith(" nt"))
        loads = 0
        for x in ins[start:]:
            if x.startswith("s_waitcnt") and "vmcnt" in x:
                break
            assert not x.startswith("global_store"), key
            if x.startswith("global_load_dwordx"):
                assert x.endswith(" nt"), (key, x)
                loads += 1
        assert loads == 8, (key, loads)          # 2 quads x (p, m, v, g)
        stores = [x for x in ins[start:] if x.startswith(("global_store_dwordx4", "global_store_dwordx2"))]
        assert len(stores) >= 8 and all(x.endswith(" nt") for x in stores), key


def streaming(body):
    """What a kernel does with memory on its main path: nt loads and stores in the order of the code, and waits for all of them."""
    out = []
    for x in instructions(body):
        if x.startswith(("global_load_dwordx", "global_store_dwordx")) and x.endswith(" nt"):
            out.append("load" if "load" in x else "store")
        elif x.startswith(("global_load_dwordx", "global_store_dwordx")):
            out.append(x)
        elif x.startswith("s_waitcnt") and "vmcnt(0)" in x:
            out.append("wait")
        elif x.startswith("s_waitcnt") and "vmcnt" in x:
            out.append("wait for some")
    return out


def test_fine_tile_issues_all_loads_before_the_first_wait(fine_kernels):
    one, lists = fine_kernels
    for key, body in [*one.items(), *lists.items()]:
        seen = streaming(body)
        first = seen.index("load")
        assert seen[first:first + 5] == ["load"] * 4 + [seen[first + 4]] and seen[first + 4].startswith("wait"), (key, seen)
        assert [x for x in seen if not x.startswith("wait")] == ["load"] * 4 + ["store"] * 4, (key, seen)      # p, m, v, g; p, m, v, copy


def test_paced_kernels_keep_their_pace(paced_kernels):
    """The order rests on an empty asm statement, scheduling barriers and a wait that is written out."""
    one, lists = paced_kernels
    for key, body in [*one.items(), *lists.items()]:
        quads = 2 if key in lists else int(key[2])
        seen = streaming(body)
        first, last = seen.index("load"), len(seen) - 1 - seen[::-1].index("store")
        want = (["load"] * 4 + ["wait"]) * quads + (["store"] * 4 + ["wait"]) * quads
        assert seen[first:last + 1] == want[:-1], (key, seen)
