"""The direct-to-LDS kernels as the compiler makes them: inside the K loop every wait for memory is one that the source counts.  A wait of
the compiler's own there (for a register that a load still owes, or for one reloaded from scratch) knows nothing of the requests issued
in inline assembly and waits for all of them, K tile after K tile."""
import re
import subprocess

import pytest

from paper_2505_18574_amd import build

ROLLING_64 = "64, 64, 2, 2, 0, 4, 128, DTL_ROLLING"
PINGPONG_256 = "256, 256, 2, 4, 0, 4, 64, DTL_PINGPONG"
INTERLEAVED_256 = "256, 256, 2, 2, 0, 4, 64, DTL_INTERLEAVED"
# element type, output stage, tile and schedule, A^T, on dwords
KERNELS = {"i32_64": ("TypeI8", "EpilogueRawI32", ROLLING_64, "false", "false"), "i32_64_dw": ("TypeI8", "EpilogueRawI32", ROLLING_64, "false", "true"),
           "i32_256": ("TypeI8", "EpilogueRawI32", PINGPONG_256, "false", "false"), "i32_256_dw": ("TypeI8", "EpilogueRawI32", PINGPONG_256, "false", "true"),
           "at_256": ("TypeI8", "EpilogueI8", PINGPONG_256, "true", "false"), "at_256_dw": ("TypeI8", "EpilogueI8", PINGPONG_256, "true", "true"),
           "bf16_64": ("TypeBF16", "EpilogueF32", ROLLING_64, "false", "false"), "bf16_256": ("TypeBF16", "EpilogueF32", PINGPONG_256, "false", "false")}
# K loops in rounds of four K tiles, 256 products, of which only the rounds are held to it
ROUNDS = {"i32_interleaved": ("TypeI8", "EpilogueRawI32", INTERLEAVED_256, "false", "false"), "bf16_interleaved": ("TypeBF16", "EpilogueF32", INTERLEAVED_256, "false", "false"),
          "bf16_interleaved_dw": ("TypeBF16", "EpilogueF32", INTERLEAVED_256, "false", "true")}


def code_of(kernels, tmp_path):
    """The instructions of each kernel as lists of basic blocks; those of inline assembly are marked with a leading '!'."""
    src = tmp_path / "k.hip"
    src.write_text('#include "common.hpp"\n#include "gemm_dtl.hpp"\nnamespace ac {\n' + "".join(
        f"template __global__ void gemm_dtl_kernel<{t}, {epi}, {tile}, {ta}, false, {dw}>(const dtl_args<{tile.split(',')[0]}, 0>);\n" for t, epi, tile, ta, dw in kernels.values()) + "}\n")
    cmd = [build._hipcc(), "-x", "hip", "-S", "--cuda-device-only", str(src), "-o", str(tmp_path / "k.s"), "-I" + build.CSRC] + build.COMMON + build.DEVICE_FLAGS
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    bodies, asm = [], False
    for line in (tmp_path / "k.s").read_text().splitlines():
        if re.match(r"_Z\S*gemm_dtl_kernel\S*:", line):
            bodies.append([[]])
        elif line.startswith(".Lfunc_end"):
            asm = False
        elif "#ASMSTART" in line or "#ASMEND" in line:
            asm = "#ASMSTART" in line
        elif bodies:
            text = line.split(";")[0].strip()
            if text.startswith(".LBB"):
                bodies[-1].append([])
            elif text and not text.startswith("."):
                bodies[-1][-1].append(("!" if asm else "") + text)
    assert len(bodies) == len(kernels)
    return dict(zip(kernels, bodies))


def test_blocks_are_told_apart(tmp_path):
    """The source's own waits are in the K loop and are seen as its own."""
    blocks = code_of({"i32_64": KERNELS["i32_64"]}, tmp_path)["i32_64"]
    loop = [b for b in blocks if sum("v_mfma" in x for x in b) == 16]
    assert loop and all(any(x.startswith("!s_waitcnt vmcnt") for x in b) for b in loop)


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    return code_of({**KERNELS, **ROUNDS}, tmp_path_factory.mktemp("dtl"))


@pytest.mark.parametrize("kernel", [*KERNELS, *ROUNDS])
def test_no_wait_of_the_compiler_in_the_k_loop(code, kernel):
    products = [sum("v_mfma" in x for x in b) for b in code[kernel]]
    assert kernel in KERNELS or max(products) == 256
    bad = [x for b, n in zip(code[kernel], products) if n >= (1 if kernel in KERNELS else 256) for x in b if x.startswith("s_waitcnt") and "vmcnt" in x or "scratch_" in x]
    assert not bad, bad


def test_arguments_stay_in_scalar_registers(code):
    """The dword form of A^T products keeps few of its scalars in lanes of a vector register (it had 660 reads of them)."""
    assert sum(x.startswith("v_readlane") for b in code["at_256_dw"] for x in b) <= 200


@pytest.mark.parametrize("kernel", ["i32_256", "i32_256_dw", "bf16_256", "i32_interleaved", "bf16_interleaved", "bf16_interleaved_dw"])
def test_staged_values_are_written_in_pairs(code, kernel):
    """A lane's sixteen rows lie at two addresses and immediates, not at sixteen addresses."""
    single, pairs = (sum(x.startswith(op) for b in code[kernel] for x in b) for op in ("ds_write_b32", "ds_write2"))
    assert pairs >= 100 and single <= pairs // 2, (single, pairs)
