"""Static checks on the generated gfx950 code (CPU only: hipcc cross-compiles).

The kernels' launch shapes depend on register and LDS budgets that only the
compiler's output shows:

  * the dK/dV kernel runs eight waves per workgroup, two per SIMD, so each
    wave may use at most 256 registers (VGPRs and AGPRs together) or the
    launch fails;
  * the forward and dQ kernels are written for two 256-thread workgroups per
    CU (same limit), and the dK/dV kernel's LDS must fit one CU's 160 KiB;
  * no kernel may spill to scratch memory (a silent, large slowdown); the
    LM-head GEMM, which fills all 512 registers of a wave, keeps a few dwords
    there around its main loop, never in it;
  * the main loops of the forward and dQ kernels read their LDS operands ahead
    of the MFMAs (a compiler that drops the requested order does so silently),
    and their diagonal steps copy the next tile without a test; the decode
    kernels' tile loops do the same and wait for no copy between their MFMAs.

Each source is compiled to device assembly with the library's own flags and
the kernel metadata is checked, so a change that breaks a budget fails here
instead of at launch time on the GPU.
"""
from __future__ import annotations

import re
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]
CSRC = ROOT / "paper_2512_22234_amd" / "csrc"
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
LDS_PER_CU = 160 * 1024


def _metadata(asm: str) -> dict:
    """Kernel name -> {field: int} from the AMDGPU metadata block of a .s file."""
    out = {}
    for block in re.split(r"\n\s+- \.", asm):
        name = re.search(r"\.name:\s+(\S+)", block)
        if not name or not name.group(1).startswith("_Z"):
            continue
        fields = {}
        for key in ("vgpr_count", "agpr_count", "sgpr_count", "private_segment_fixed_size",
                    "group_segment_fixed_size"):
            m = re.search(r"\.?" + key + r":\s+(\d+)", "." + block)
            if m:
                fields[key] = int(m.group(1))
        out[name.group(1)] = fields
    return out


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """Source name -> device assembly."""
    if not Path(HIPCC).exists():
        pytest.skip("hipcc not available")
    from paper_2512_22234_amd.build import compile_flags
    texts = {}
    for src in ("fwd.hip", "bwd.hip", "decode.hip", "lce.hip"):
        out = tmp_path_factory.mktemp("isa") / (src + ".s")
        flags = [f for f in compile_flags(src) if f != "-fPIC"]
        cmd = [HIPCC, *flags, f"-I{CSRC}", "--cuda-device-only", "-S", "-o", str(out), str(CSRC / src)]
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, r.stderr[-2000:]
        texts[src] = out.read_text()
    return texts


@pytest.fixture(scope="module")
def kernels(assembly):
    return {k: v for text in assembly.values() for k, v in _metadata(text).items()}


def _find(meta, part):
    found = {k: v for k, v in meta.items() if part in k}
    assert found, f"no kernel matching {part}"
    return found


# The LM-head GEMM's variants (epilogue, A and B side read transposed) that may
# keep something in scratch memory, and how many bytes per lane.
GEMM_SCRATCH = {"lce_gemm_kernelILi3ELb0ELb0E": 32, "lce_gemm_kernelILi2ELb1ELb0E": 12,
                "lce_gemm_kernelILi2ELb1ELb1E": 16}


def test_no_scratch_spills(kernels):
    assert len(kernels) >= 6  # fwd, dkdv, dq at D = 64 and 128
    for name, f in kernels.items():
        allowed = next((n for part, n in GEMM_SCRATCH.items() if part in name), 0)
        assert f.get("private_segment_fixed_size", 0) <= allowed, name


@pytest.mark.parametrize("part", ["dkdv_kernelILi128", "dkdv_kernelILi64", "fwd_kernelILi128",
                                  "fwd_kernelILi64", "dq_kernelILi128", "dq_kernelILi64"])
def test_two_waves_per_simd_fit(kernels, part):
    for name, f in _find(kernels, part).items():
        # gfx950 metadata: vgpr_count counts architectural VGPRs, agpr_count the
        # accumulation registers; a wave's allocation is their sum (each rounded
        # to 8), and two waves share a SIMD's 512
        total = -(-f["vgpr_count"] // 8) * 8 + -(-f.get("agpr_count", 0) // 8) * 8
        assert total <= 256, (name, f)


@pytest.mark.parametrize("part", ["dec_kernel", "lce_gemm_kernel"])
def test_lds_fits_one_cu(kernels, part):
    for name, f in _find(kernels, part).items():
        assert 0 < f["group_segment_fixed_size"] <= LDS_PER_CU, (name, f)


def test_dkdv_lds_fits_one_cu(kernels):
    for name, f in _find(kernels, "dkdv_kernel").items():
        assert 0 < f["group_segment_fixed_size"] <= LDS_PER_CU, (name, f)


def _blocks(text, part):
    """Basic blocks (as lists of instructions) of every kernel whose name holds `part`."""
    found = 0
    for kernel in re.split(r"\n(?=_Z\S+:)", text):
        if part not in kernel.split(":", 1)[0]:
            continue
        found += 1
        for block in re.split(r"\n(?=\.LBB\S+:)", kernel):
            yield [line.strip() for line in block.split("\n")[1:] if line.startswith("\t")]
    assert found, part


@pytest.mark.parametrize("src,part", [("fwd.hip", "fwd_kernelILi128"), ("fwd.hip", "fwd_kernelILi64"),
                                      ("bwd.hip", "dq_kernelILi128"), ("bwd.hip", "dq_kernelILi64")])
def test_main_loops_read_operands_ahead(assembly, src, part):
    """Blocks that multiply without a wait for LDS in between let each MFMA wait
    for its own operands while later reads are in flight: lgkmcnt(0) only at the
    end of a run of MFMAs."""
    loops = 0
    for block in _blocks(assembly[src], part):
        mfmas = sum("v_mfma" in x for x in block)
        barrier = any("s_barrier" in x for x in block)
        copies = any("buffer_load" in x for x in block)
        if mfmas < 8 or not (barrier or copies):  # the main loop's blocks hold the step's copies or its end
            continue
        loops += 1
        drained = sum("v_mfma" in y and "lgkmcnt(0)" in x for x, y in zip(block, block[1:]))
        assert drained <= 2, (part, drained, mfmas)
    assert loops >= 2, loops  # bf16 and float32 results


@pytest.mark.parametrize("src,part", [("fwd.hip", "fwd_kernelILi128"), ("fwd.hip", "fwd_kernelILi64"),
                                      ("bwd.hip", "dq_kernelILi128"), ("bwd.hip", "dq_kernelILi64")])
def test_step_copies_are_unconditional(assembly, src, part):
    """Only the prologue's copies stand behind a test (is there a key tile at all?)."""
    tested = 0
    for block in _blocks(assembly[src], part):
        first = next((i for i, x in enumerate(block) if "buffer_load" in x), None)
        tested += first is not None and any(x.startswith("s_cbranch") for x in block[:first])
    assert tested <= 2, tested  # one per kernel: bf16 and float32 results


@pytest.mark.parametrize("team", [1, 2, 4])
def test_decode_tile_loop_waits(assembly, team):
    """No wait for copies between a tile's MFMAs, which would drain the ring, and
    operands read ahead of them (D = 128, with and without the streaming hint)."""
    loops = 0
    for block in _blocks(assembly["decode.hip"], f"dec_kernelILi128ELi{team}"):
        if sum("v_mfma" in x for x in block) < 8:
            continue
        loops += 1
        assert not any("vmcnt" in x for x in block), block[0]
        drained = sum("v_mfma" in y and "lgkmcnt(0)" in x for x, y in zip(block, block[1:]))
        assert drained <= 2, (team, drained)
    assert loops == 4, loops  # scores and output, twice


def test_gemm_main_loop_has_no_scratch_access(assembly):
    """A reload from scratch memory in the k loop would wait for every copy in
    flight.  Checked per basic block: those with a whole step's MFMAs."""
    bodies = 0
    for block in _blocks(assembly["lce.hip"], "lce_gemm_kernel"):
        if sum("v_mfma" in x for x in block) >= 16:
            bodies += 1
            assert not any("scratch_" in x for x in block), block[0]
    assert bodies >= 6


def test_metadata_parser():
    asm = "\n".join([
        "amdhsa.kernels:",
        "  - .agpr_count:     4",
        "    .group_segment_fixed_size: 1024",
        "    .name:           _Zfoo",
        "    .private_segment_fixed_size: 16",
        "    .sgpr_count:     20",
        "    .vgpr_count:     100",
        "  - .agpr_count:     0",
        "    .name:           _Zbar",
        "    .vgpr_count:     12",
    ])
    m = _metadata(asm)
    assert m["_Zfoo"] == {"vgpr_count": 100, "agpr_count": 4, "sgpr_count": 20,
                          "private_segment_fixed_size": 16, "group_segment_fixed_size": 1024}
    assert m["_Zbar"]["vgpr_count"] == 12 and m["_Zbar"]["agpr_count"] == 0
