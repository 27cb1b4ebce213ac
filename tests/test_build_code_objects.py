"""The built gfx950 code objects: no kernel keeps values in scratch memory, and
what the GEMM's inline assembly relies on holds in every instance.

A kernel whose accumulators or staged values spill to scratch still gives the
right results, so no parity test notices, but it runs several times slower
(a rolled loop over the GEMM epilogue's passes once moved the 256-wide tiles'
accumulators to scratch: the fused bias epilogue took 287 us instead of 31).
This reads the AMDGPU metadata of every kernel in the objects the build left
in ``paper_2608_27370_amd/_build``: no private segment, no dynamic stack, no
VGPR or SGPR spills.
"""

import glob
import os
import re
import subprocess
import tempfile

import pytest
import yaml

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BUILD = os.path.join(ROOT, "paper_2608_27370_amd", "_build")
LLVM = "/opt/rocm/llvm/bin"
TARGET = "hipv4-amdgcn-amd-amdhsa--gfx950"


def _dump(obj, tool, *args):
    """The output of an LLVM tool on the gfx950 code object embedded in obj."""
    with tempfile.TemporaryDirectory() as d:
        fat, co = os.path.join(d, "fatbin"), os.path.join(d, "co")
        subprocess.run([os.path.join(LLVM, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, obj, os.devnull],
                       check=True, capture_output=True)
        subprocess.run([os.path.join(LLVM, "clang-offload-bundler"), "--unbundle", "--type=o", "--targets=" + TARGET,
                        "--input=" + fat, "--output=" + co], check=True, capture_output=True)
        return subprocess.run([os.path.join(LLVM, tool), *args, co], check=True, capture_output=True,
                              text=True).stdout


def _kernels(obj):
    """Metadata of every kernel in the gfx950 code object embedded in obj."""
    notes = _dump(obj, "llvm-readelf", "--notes")
    doc = re.search(r"^(amdhsa\..*?)^\s*\.\.\.\s*$", notes, re.S | re.M)
    assert doc, "no AMDGPU metadata in %s" % obj
    return yaml.safe_load(doc.group(1))["amdhsa.kernels"]


def _listings(obj):
    """(name, instructions) of every kernel in the gfx950 code object embedded in obj."""
    out = []
    for line in _dump(obj, "llvm-objdump", "-d", "--no-show-raw-insn").splitlines():
        head = re.match(r"^[0-9a-f]+ <(.*)>:", line)
        if head:
            out.append((head.group(1), []))
        elif out and line.strip():
            out[-1][1].append(line.split("//")[0].strip())
    return out


def _objects():
    tools = all(os.access(os.path.join(LLVM, t), os.X_OK)
                for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf", "llvm-objdump"))
    objs = [o for o in sorted(glob.glob(os.path.join(BUILD, "*.o"))) if not o.endswith("api.o")]
    if not tools or not objs:
        pytest.skip("needs the built objects (paper_2608_27370_amd/build.py) and the ROCm LLVM tools")
    return objs


def test_no_kernel_uses_scratch():
    seen = 0
    bad = []
    for obj in _objects():
        for k in _kernels(obj):
            seen += 1
            if (k.get(".private_segment_fixed_size", 0) or k.get(".uses_dynamic_stack", False)
                    or k.get(".vgpr_spill_count", 0) or k.get(".sgpr_spill_count", 0)):
                bad.append((os.path.basename(obj), k[".name"], k.get(".private_segment_fixed_size"),
                            k.get(".vgpr_spill_count"), k.get(".sgpr_spill_count")))
    assert seen > 100, "expected every GEMM and quantise instance, found %d kernels" % seen
    assert not bad, bad


def test_m0_belongs_to_the_dma_loads():
    """The LDS-DMA loads write M0 from inline assembly without saving it: each
    such statement names it as a clobber, and the GEMM kernels use M0 for
    nothing else."""
    asm = []
    for src in glob.glob(os.path.join(os.path.dirname(BUILD), "csrc", "*.h*")):
        with open(src) as f:
            asm += [a for a in re.findall(r"asm volatile\((.*?)\);", f.read(), re.S) if "m0, %" in a]
    assert len(asm) == 2
    for a in asm:
        assert '"m0"' in a.rsplit(":", 1)[1], a
    seen = 0
    for obj in _objects():
        if os.path.basename(obj).startswith("gemm_kernel"):
            for name, ins in _listings(obj):
                bad = [i for i in ins if re.search(r"\bm0\b", i) and not i.startswith("s_mov_b32 m0,")]
                seen += len([i for i in ins if i.startswith("s_mov_b32 m0,")])
                assert not bad, (name, bad[:4])
    assert seen > 1000


def test_accumulator_reads_wait_for_the_matrix_instructions():
    """The epilogue reads accumulators in inline assembly, where the compiler
    places no wait states for the matrix instruction that wrote them: between
    a kernel's last MFMA and the first such read stand 20 explicit ones (16
    passes and 4)."""
    seen = 0
    for obj in _objects():
        if not os.path.basename(obj).startswith("gemm_kernel"):
            continue
        for name, ins in _listings(obj):
            mfma = [i for i, x in enumerate(ins) if x.startswith("v_mfma")]
            if not mfma:
                continue
            seen += 1
            waits = 0
            for x in ins[mfma[-1] + 1:]:
                if x.startswith("s_nop"):
                    waits += int(x.split()[1], 0) + 1
                if x.startswith("v_accvgpr_read"):
                    break
            assert waits >= 20, (name, waits)
    assert seen > 100


def test_bf16_outputs_stream_by_operand_format():
    """The BF16 outputs of FP8 operands leave by non-temporal stores in every
    store path of a tile, those of BF16 operands in none."""
    seen = 0
    for obj in _objects():
        if not os.path.basename(obj).startswith("gemm_kernel"):
            continue
        for name, ins in _listings(obj):
            # template arguments: tile (2), wave grid (2), operand formats (2), output kind
            t = re.search(r"gemm_fp8_kernelI((?:Li\d+E){7})", name)
            if not t:
                continue
            fa, _, out = [int(v) for v in re.findall(r"\d+", t.group(1))][4:]
            if out not in (0, 3):          # BF16, alone or with bias / residual
                continue
            seen += 1
            stores = [i for i in ins if i.startswith("buffer_store")]
            streamed = [i for i in stores if re.search(r"\bnt\b", i)]
            assert stores and len(streamed) == (0 if fa == 2 else len(stores)), (name, len(stores), len(streamed))
    assert seen > 100
