"""The device code inside libpgmoe.so, disassembled here: rules of the hardware that the compiler keeps
for its own instructions but cannot keep inside an inline-assembly statement, and what a launch that
uses an option of a kernel must not cost the launches that do not."""
import os
import re
import subprocess

import pytest

from paper_2308_12066_amd import binding as B, build

LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "llvm", "bin")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """Paths of the gfx950 code objects the library carries, one per source file."""
    objdump = os.path.join(LLVM, "llvm-objdump")
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump")
    folder = tmp_path_factory.mktemp("code")
    lib = folder / "lib.so"
    lib.write_bytes(open(B.LIB_PATH, "rb").read())
    subprocess.run([objdump, "--offloading", str(lib)], check=True, stdout=subprocess.DEVNULL, cwd=folder)
    objs = sorted(str(p) for p in folder.iterdir() if "gfx950" in p.name)
    assert len(objs) == len(build.SOURCES)
    return objs


def writes_m0(instruction):
    return re.match(r"s_\S+\s+m0\b", instruction) is not None


def test_a_load_into_lds_leaves_a_wait_state_after_m0_is_written(code_objects):
    """A direct-to-LDS load takes its LDS address from M0 and needs one instruction between a scalar write of
    M0 and itself; without it the tile may land where the load before it put its own."""
    seen, bad = 0, []
    for obj in code_objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
        kernel, before = "", ""
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if m:
                kernel, before = m.group(1), ""
                continue
            ins = line.split("//")[0].strip()
            if not ins:
                continue
            if ins.startswith("global_load_lds") or (ins.startswith("buffer_load") and ins.endswith(" lds")):
                seen += 1
                if writes_m0(before):
                    bad.append((kernel, before, ins))
            before = ins
    assert seen > 0
    assert not bad, f"{len(bad)} of {seen} loads follow the write of M0 at once, the first in {bad[0]}"


def test_waits_of_the_one_token_step_read_no_clock(code_objects):
    """Its workgroups wait for each other for a number of looks.  The clock goes on while other processes
    have the GPU: a wait that it bounds may give up on its first look after a pause."""
    seen = 0
    for obj in code_objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout
        for body in re.split(r"^[0-9a-f]+ (?=<)", text, flags=re.M):
            if "ffn_decode_stack_kernel" in body.split("\n", 1)[0]:
                seen += 1
                assert not re.search(r"s_mem(real)?time|s_getreg_b32", body), body.split("\n", 1)[0]
    assert seen == 4


def kernels(code_objects):
    """{mangled name: {field: integer}} of the code objects' kernel metadata."""
    out = {}
    for obj in code_objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", obj], check=True, capture_output=True, text=True).stdout
        for entry in re.split(r"\n  - (?=\.)", text)[1:]:
            name = re.search(r"^\s*\.name:\s+'?(_Z\w+)", entry, re.M)
            if name:
                out[name.group(1)] = {k: int(v) for k, v in re.findall(r"^\s*\.(\w+):\s+(\d+)$", entry, re.M)}
    return out


def test_a_combine_without_a_carried_gate_has_no_arguments_of_one(code_objects):
    """The host writes a launch's arguments one by one: the combine of a batch-1 block has 64 bytes of them."""
    found = {n: k for n, k in kernels(code_objects).items() if "combine_partials_kernel" in n}
    plain = {n: k["kernarg_segment_size"] for n, k in found.items() if "CarriedGate" not in n}
    assert len(plain) == 3 and len(found) == 6, sorted(found)
    assert max(plain.values()) <= 64, plain


def test_a_fused_expert_launch_without_a_carried_gate_keeps_its_occupancy(code_objects):
    """Wavefronts per SIMD (512 registers a lane, dealt out eight at a time, at most eight wavefronts) of the
    variants that a launch without a gate runs; the gate's code would take one to four of them."""
    waves = {}
    for name, k in kernels(code_objects).items():
        m = re.search(r"ffn_fused_kernelILi(\d+)ELi(\d+)ELi(\d+)E", name)
        if m and "CarriedGate" not in name:
            waves[tuple(map(int, m.groups()))] = min(8, 512 // (-(-k["vgpr_count"] // 8) * 8))
    for case, want in {(1, 2, 4): 8, (2, 2, 4): 8, (1, 4, 4): 5, (1, 16, 4): 3}.items():    # (row tiles, d_model / 32, wavefronts)
        assert waves.get(case, 0) >= want, (case, waves)


def test_latency_bound_kernels_have_no_stack_frame(code_objects):
    """The batch-1 stack and the matrix-core gates of up to 128 experts: a frame makes every workgroup wait for scratch memory to be set up, and
    it is there because registers ran out."""
    found = kernels(code_objects)
    names = [n for n in found if re.search(r"ffn_decode_stack|gate_small_kernel|gate_topk_mfma_kernelILi1E|gate_topk_tiles_kernel", n)]
    assert len(names) == 4 + 2 + 1 + 6 + 4, sorted(names)
    framed = {n: found[n]["private_segment_fixed_size"] for n in names if found[n]["private_segment_fixed_size"]}
    assert not framed


def test_fused_expert_launches_of_d_model_256_keep_their_occupancy(code_objects):
    """Launches of d_model 256 have a few small workgroups per CU: wavefronts per SIMD by rows per chunk."""
    waves = {}
    for name, k in kernels(code_objects).items():
        m = re.search(r"ffn_fused_kernelILi(\d+)ELi8ELi4E", name)
        if m:
            waves.setdefault(int(m.group(1)), []).append(min(8, 512 // (-(-k["vgpr_count"] // 8) * 8)))
    assert {mt: min(w) for mt, w in waves.items() if mt < 4} == {1: 4, 2: 4} and min(waves[4]) >= 2, waves
