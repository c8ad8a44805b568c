"""What the assembler does not do for inline assembly, checked in the device code compiled to assembly.

* A DPP instruction (`v_fmac_f32_dpp` of the real-input VALU kernel) must not read a VGPR that a VALU instruction wrote in
  the two instructions before it, and must not follow a write of EXEC within five.
* Kernels whose operands come to LDS by loads that write it (`buffer_load_dword* ... lds`, `global_load_lds_*`) cross their
  barriers in inline assembly, where the compiler places no waits: a wave must not cross one with LDS reads of its own
  under way, since behind it another wave's load may overwrite the place they read.
* Such a load reads its SGPRs and M0 at once: an SGPR written by a VALU instruction needs five wait states first.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _written_vgprs(ins: str):
    m = re.match(r"v_\w+\s+(?:v\[(\d+):(\d+)\]|v(\d+))", ins)
    if not m:
        return set()
    if m.group(1):
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    return {int(m.group(3))}


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """The device code of two translation units, compiled to assembly side by side."""
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not found")
    tmp = tmp_path_factory.mktemp("isa")
    names = ("bnn_api", "f32_chain_bits")
    jobs = [subprocess.Popen(["hipcc", "-O3", "--offload-arch=gfx950", "-std=c++17", "-ffp-contract=off", "-Xclang", "-target-feature",
                              "-Xclang", "-packed-fp32-ops", "-S", "--cuda-device-only", "-I", os.path.join(ROOT, "include"),
                              "-o", str(tmp / (n + ".s")), os.path.join(ROOT, "paper_1706_09453_amd", "csrc", n + ".hip")],
                             stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL) for n in names]
    assert [j.wait() for j in jobs] == [0, 0]
    return {n: (tmp / (n + ".s")).read_text() for n in names}


@pytest.fixture(scope="module")
def code(assembly):
    """The device code of bnn_api.hip as a list of instructions, with the labels of functions and blocks."""
    lines = [l.split(";")[0].strip() for l in assembly["bnn_api"].splitlines()]
    return [l for l in lines if l and not l.startswith("//") and (l.endswith(":") or not l.startswith("."))]


def _metadata(assembly):
    """The figures the compiler gives for every kernel: name, registers, LDS, size of the arguments and so on."""
    for text in assembly.values():
        for k in re.split(r"\n  - ", text[text.index("amdhsa.kernels"):])[1:]:
            fields = dict(re.findall(r"\.(\w+):\s+(\S+)", k.split(".args:")[0] + k[k.rfind(".group_segment_fixed_size"):]))
            if "name" in fields:
                yield fields


def _kernels(code):
    """(name, instructions) of every function."""
    name, body = None, []
    for l in code:
        if re.match(r"_Z\w+:$", l):
            if name:
                yield name, body
            name, body = l[:-1], []
        elif name:
            body.append(l)
    if name:
        yield name, body


def _loads_lds(ins: str):
    return bool(re.match(r"buffer_load_dword\w* .*\blds$", ins)) or ins.startswith("global_load_lds_")


def _needs_wait_for_lds(ins: str):
    return bool(re.match(r"ds_(read|swizzle|bpermute|permute)", ins)) or bool(re.match(r"ds_\w+_rtn", ins))


def _reads_pending(body):
    """For every instruction: can an LDS read of the wave still be under way in front of it, on any path?"""
    at = {l[:-1]: i for i, l in enumerate(body) if l.endswith(":")}
    pending, work = [None] * len(body), [(0, False)]
    while work:
        i, p = work.pop()
        while i < len(body) and not (pending[i] or pending[i] == p):
            pending[i] = p
            ins = body[i]
            if re.match(r"s_waitcnt .*lgkmcnt\(0\)", ins):
                p = False
            elif _needs_wait_for_lds(ins):
                p = True
            if ins.startswith(("s_endpgm", "s_setpc")):
                break
            m = re.match(r"s_c?branch\w*\s+(\S+)", ins)
            if m:
                work.append((at[m.group(1)], p))
                if ins.startswith("s_branch"):
                    break
            i += 1
    return pending


def test_no_lds_read_is_under_way_at_a_barrier_of_the_loads_that_write_lds(code):
    n, bad = 0, set()
    for name, body in _kernels(code):
        if not any(_loads_lds(l) for l in body):
            continue
        for ins, p in zip(body, _reads_pending(body)):
            if ins.startswith("s_barrier"):
                n += 1
                if p:
                    bad.add(name)
    assert n > 0 and not bad, (n, len(bad), sorted(bad)[:4])


def test_binary_product_loops_wait_for_no_more_lds_reads_than_they_need(code):
    """The words of a stage's second half are requested in front of the products of its first half, and are not to be waited
    for there: no block with products of the kernels that fetch through LDS has a wait for all LDS operations (the one at
    the stage's barrier, which also counts memory, aside)."""
    n, bad = 0, set()
    for name, body in _kernels(code):
        if "binx_mfma32_kernel" not in name or not any(_loads_lds(l) for l in body):
            continue
        products = waits = 0
        for ins in body + ["end:"]:
            if ins.endswith(":"):
                n += products > 0
                if products and waits:
                    bad.add(name)
                products = waits = 0
            products += ins.startswith("v_mfma_f32_32x32x64_f8f6f4")
            waits += ins == "s_waitcnt lgkmcnt(0)"
    assert n > 0 and not bad, (n, len(bad), sorted(bad)[:4])


def test_loads_that_write_lds_do_not_read_fresh_sgprs(code):
    n, bad = 0, []
    for name, body in _kernels(code):
        for i, ins in enumerate(body):
            if not _loads_lds(ins):
                continue
            n += 1
            regs = set()
            for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", ins):
                regs |= set(range(int(a), int(b) + 1))
            regs |= {int(a) for a in re.findall(r"\bs(\d+)\b", ins)}
            states, back = 0, i - 1
            while states < 5 and back >= 0:
                prev = body[back]
                back -= 1
                if prev.endswith(":"):
                    continue
                dst = prev.split(None, 1)[1].split(",")[0] if " " in prev else ""
                m = re.match(r"s(\d+)$", dst)
                m2 = re.match(r"s\[(\d+):(\d+)\]$", dst)
                hit = {int(m.group(1))} if m else set(range(int(m2.group(1)), int(m2.group(2)) + 1)) if m2 else set()
                if prev.startswith("v_") and hit & regs:
                    bad.append((name, prev, ins))
                k = re.match(r"s_nop\s+(\d+)", prev)
                states += int(k.group(1)) + 1 if k else 1
    assert n > 0 and not bad, bad[:4]


def test_dpp_fmac_sources_are_not_fresh_valu_results(code):
    code = [l for l in code if not l.endswith(":")]
    n_dpp, bad = 0, []
    for i, ins in enumerate(code):
        if not ins.startswith("v_fmac_f32_dpp"):
            continue
        n_dpp += 1
        src = int(re.match(r"v_fmac_f32_dpp v\d+, v(\d+),", ins).group(1))
        states, back = 0, 1          # wait states between the instruction `back` places earlier and this one
        while states < 5:
            prev = code[i - back]
            if states < 2 and prev.startswith("v_") and src in _written_vgprs(prev):
                bad.append((prev, ins))
            dst = prev.split(",")[0]
            if re.search(r"\bexec", dst) and (prev.startswith("s_") or prev.startswith("v_cmpx")):
                bad.append((prev, ins))
            m = re.match(r"s_nop\s+(\d+)", prev)
            states += int(m.group(1)) + 1 if m else 1
            back += 1
    assert n_dpp > 0, "the kernel no longer uses the DPP fmac: delete this test"
    assert not bad, bad[:5]


def test_first_layers_take_few_launch_arguments(assembly):
    """A launch with more than 112 bytes of arguments (the 256 that hold the grid's size among them) takes the host 3.5 us instead of
    2.9: the kernels that may stand in front of a run of binary layers keep below that wherever they stand, but for the two that also
    pull the run's weights."""
    first = r"realx_valu_kernel|realx_sign_fused_kernel|realx_resolve_rows|realx_quantize_nat|f32_chain_kernel"
    sizes = {k["name"]: int(k["kernarg_segment_size"]) for k in _metadata(assembly) if re.search(first, k["name"]) and "4Pull" not in k["name"]}
    assert len(sizes) > 80 and max(sizes.values()) <= 112, [k for k in sizes.items() if k[1] > 112][:4]


def test_four_launches_of_a_run_of_binary_layers_fit_on_a_cu(assembly):
    """Their workgroups, one to a CU, wait for each other: where the runs of four streams (as many queues as the device runs at once) do
    not all fit, each of them gets a part of its workgroups and all wait until they give up.  512 registers and a wave of each
    workgroup per SIMD, 160 KB of LDS.  (2048 units have at most 128 frames, of which one wave per workgroup takes care.)"""
    runs = [k for k in _metadata(assembly) if re.search(r"few_chain_kernel|hidden_run_kernel", k["name"])]
    assert len(runs) >= 14
    for k in runs:
        most = 168 if "hidden_run_kernelILi4ELi1E" in k["name"] else 128
        assert int(k["max_flat_workgroup_size"]) <= 256 and int(k["vgpr_count"]) <= most and 4 * int(k["group_segment_fixed_size"]) <= 160 * 1024, k
