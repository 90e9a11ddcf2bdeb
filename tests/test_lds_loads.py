"""The asynchronous loads into LDS (csrc/tiled_core.h) are inline assembly, in which the compiler keeps no hazard away.  Here the
compiler has to put what it must not get wrong right in front of such loads, and the AMD assembly it makes of that is read.  (Nothing is run.)"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_02006_amd", "csrc")


def assembly(tmp_path, body):
    from paper_2506_02006_amd import build as hb
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text('#include "tiled_core.h"\nusing namespace morph;\n' + body)
    flags = [f for f in hb.HIPCC_FLAGS if not f.startswith(("-R", "-W"))]
    r = subprocess.run([hb._hipcc(), *flags, "-w", "-I", CSRC, "--offload-device-only", "-S", str(src), "-o", str(out)], stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    lines = (l.split(";")[0].strip() for l in out.read_text().splitlines())
    return [l for l in lines if l and not l.startswith(".") and not l.endswith(":")]


def scalars(text):
    found = set()
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        found |= set(range(int(a), int(b) + 1))
    return found | {int(a) for a in re.findall(r"\bs(\d+)\b", text)}


def is_lds_load(line):
    return line.startswith("buffer_load") and line.split()[-1] == "lds"


def states_before_loads(lines):
    """For every load into LDS: the fewest wait states between a vector instruction that wrote one of its scalar registers and the load."""
    written, now, got = {}, 0, []
    for line in lines:
        op, _, args = line.partition(" ")
        if is_lds_load(line):
            got.append(min((now - written[r] for r in scalars(args) if r in written), default=None))
        now += int(args, 0) + 1 if op == "s_nop" else 1
        for r in scalars(args.split(",")[0]):
            if op.startswith("v_"):
                written[r] = now
            elif op.startswith("s_") and not op.startswith(("s_cmp", "s_nop", "s_wait", "s_barrier", "s_cbranch")):
                written.pop(r, None)
    return got


@pytest.mark.parametrize("load", ["dma16<false>", "dma16<true>", "dma4"])
def test_five_wait_states_before_a_load_that_reads_restored_registers(tmp_path, load):
    """Descriptor words and offset come out of vector lanes (as the compiler restores parked scalar registers) right before the load."""
    lines = assembly(tmp_path, """
extern "C" __global__ void probe(const int* q, int* out)
{
    __shared__ __align__(16) int buf[1024];
    const int v = q[threadIdx.x];
    u32x4 r; uint32_t soff;
    for (int i = 0; i < 4; i++) r[i] = (uint32_t)__builtin_amdgcn_readlane(v, i);
    soff = (uint32_t)__builtin_amdgcn_readlane(v, 4);
    %s((uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)buf, threadIdx.x * 16, r, soff);
    wait_vm<0>();
    wg_barrier();
    out[threadIdx.x] = buf[threadIdx.x];
}
""" % load)
    got = states_before_loads(lines)
    assert len(got) == 1 and got[0] is not None, (got, lines)
    assert got[0] >= 5, (got, [l for l in lines if "readlane" in l or "lds" in l or "nop" in l])


def test_m0_is_known_to_be_written(tmp_path):
    """A value that the compiler keeps in m0 does not outlive a load that writes m0: its own loads to one place, with one of ours between them."""
    lines = assembly(tmp_path, """
extern "C" __global__ void probe(const int* q, int* out, int to)
{
    __shared__ __align__(16) int buf[1024];
    const __amdgpu_buffer_rsrc_t r = make_rsrc(q, 4096);
    int* const at = buf + 256;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)at, 4, threadIdx.x * 4, 0, 0, 0);
    dma4((uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)buf, threadIdx.x * 4, rsrc_words(q, 4096), 0u);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)at, 4, threadIdx.x * 4, 256, 0, 0);
    wait_vm<0>();
    wg_barrier();
    out[threadIdx.x] = buf[threadIdx.x + to];
}
""")
    seen = [l for l in lines if is_lds_load(l) or re.match(r"s_\w+ m0,", l)]
    assert sum(map(is_lds_load, seen)) == 3, seen
    assert all(not is_lds_load(a) for a, b in zip(seen, seen[1:]) if is_lds_load(b)) and not is_lds_load(seen[0]), seen
