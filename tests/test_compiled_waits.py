"""What the compiler made of the kernels' hand-written ordering, read from the machine code of the library built here (no GPU).

A workgroup of a fused split-K kernel stores its plane, counts itself in, and the one that finds all others counted sums the planes.  Nothing but a
wait for a wave's own stores (vmcnt) puts them before the count: the release half of a workgroup barrier does not, for waves of a workgroup
see each other's stores without it."""
import os
import re
import subprocess

import pytest

import paper_2512_02551_amd as hg

LLVM = "/opt/rocm/llvm/bin/"
FUSED = re.compile(r"mfma_gemm_kernelINS_7MfmaCfg\w+ELi(3|10)ELb[01]ENS_8GemmArgsE|skinny_gemm_kernelILi\dELb1E|skinny_tn_gemm_kernelILi\dELb1E")


@pytest.fixture(scope="module")
def fused_kernels(tmp_path_factory):
    """name -> instructions."""
    where = tmp_path_factory.mktemp("code")
    os.symlink(hg.lib_path(), where / "lib.so")
    subprocess.run([LLVM + "llvm-objdump", "--offloading", "lib.so"], cwd=where, check=True, stdout=subprocess.DEVNULL)
    out = {}
    for obj in sorted(where.glob("lib.so.*gfx950")):
        names = subprocess.run([LLVM + "llvm-objdump", "-t", str(obj)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()
        names = [n for n in names if FUSED.search(n) and "." not in n]
        if not names:
            continue
        text = subprocess.run([LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", "--disassemble-symbols=" + ",".join(names), str(obj)], check=True,
                              stdout=subprocess.PIPE, text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"<([^>]+)>:", line)
            if m:
                name = m[1] if m[1] in names else name         # labels inside a kernel are not its end
                out.setdefault(name, [])
            elif name and line.strip():
                out[name].append(line.split("//")[0].strip())
    return out


def test_every_fused_reduction_waits_for_its_stores_before_it_counts_itself_in(fused_kernels):
    assert len(fused_kernels) > 150
    for name, code in fused_kernels.items():
        counts = [i for i, line in enumerate(code) if line.startswith("global_atomic_add")]
        assert counts, name
        barrier = max(i for i in range(counts[0]) if code[i].startswith("s_barrier"))
        store = max(i for i in range(barrier) if code[i].startswith(("global_store", "buffer_store")))
        assert any("vmcnt(0)" in line for line in code[store:barrier]), (name, code[store:barrier + 1])


def test_the_loops_over_k_tiles_start_on_32_bytes(tmp_path):
    """A loop that starts in the last bytes of a line waits for the next one on every pass.  The loop over K-tiles is the shortest way back over both
    matrix instructions and copies (blocks that are laid out behind their place also jump back, once)."""
    os.symlink(hg.lib_path(), tmp_path / "lib.so")
    subprocess.run([LLVM + "llvm-objdump", "--offloading", "lib.so"], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    kernels = 0
    for obj in sorted(tmp_path.glob("lib.so.*gfx950")):
        names = subprocess.run([LLVM + "llvm-objdump", "-t", str(obj)], check=True, stdout=subprocess.PIPE, text=True).stdout.split()
        names = [n for n in names if re.search(r"mfma_gemm_kernelINS_7MfmaCfg\w+ELi0ELb[01]ENS_8GemmArgsE", n) and "." not in n]
        if not names:
            continue
        text = subprocess.run([LLVM + "llvm-objdump", "-d", "--disassemble-symbols=" + ",".join(names), str(obj)], check=True, stdout=subprocess.PIPE, text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(_ZN5hgemm16mfma_gemm_kernel[^>]*)>:\n(.*?)(?=^[0-9a-f]+ <_ZN5hgemm|\Z)", text, re.M | re.S):
            code = [(int(m[2], 16), m[1]) for m in re.finditer(r"^\s+(\S.*?)\s*// ([0-9A-F]+):", body, re.M)]
            mfma = [at for at, line in code if line.startswith("v_mfma")]
            copies = [at for at, line in code if line.startswith("buffer_load") and line.endswith("lds")]
            back = [(at, at + 4 + 4 * (int(m[1]) - (1 << 16))) for at, line in code for m in [re.match(r"s_c?branch\S*\s+(\d+)", line)] if m and int(m[1]) >= 1 << 15]
            loops = sorted((at - head, head) for at, head in back if any(head <= x <= at for x in mfma) and any(head <= x <= at for x in copies))
            assert loops, name
            assert loops[0][1] % 32 == 0, (name, hex(loops[0][1]))
            kernels += 1
    assert kernels > 100
