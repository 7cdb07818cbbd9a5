"""The build-time scan of the generated device assembly (host logic, no GPU): a value that the register
allocator brings back from the accumulation registers right in front of an asm matrix instruction that reads
it must fail the build; the same move far enough away, or feeding another register, must not.  Likewise for the data of a wide asm store
that is overwritten right behind it."""
import os
import subprocess

from paper_2303_02191_amd import build
from paper_2303_02191_amd.build import check_matrix_hazards, check_store_hazards

MFMA = "\t;;#ASMSTART\n\tv_smfmac_f32_16x16x64_bf16 a[0:3], v[10:13], v[20:27], v5 cbsz:0 abid:0\n\t;;#ASMEND\n"


def _scan(tmp_path, text):
    p = os.path.join(str(tmp_path), "k.s")
    with open(p, "w") as f:
        f.write(text)
    return check_matrix_hazards(p)


def test_parked_value_restored_in_front_of_matrix_instruction_is_flagged(tmp_path):
    found = _scan(tmp_path, "kernel:\n\tv_accvgpr_read_b32 v22, a200\n\tv_add_u32_e32 v1, v2, v3\n" + MFMA)
    assert len(found) == 1 and "v_accvgpr_read_b32 v22" in found[0][0] and "v_smfmac" in found[0][1]
    # the index register and the A operand count as sources too
    assert len(_scan(tmp_path, "\tv_accvgpr_read_b32 v5, a7\n" + MFMA)) == 1
    assert len(_scan(tmp_path, "\tv_accvgpr_mov_b32 v11, a7\n" + MFMA)) == 1


def test_distance_other_registers_and_compiler_emitted_instructions_pass(tmp_path):
    far = "\tv_accvgpr_read_b32 v22, a200\n" + "\tv_add_u32_e32 v1, v2, v3\n" * 4 + MFMA
    assert _scan(tmp_path, far) == []
    # s_nop N idles N + 1 cycles: s_nop 3 alone is distance enough
    assert _scan(tmp_path, "\tv_accvgpr_read_b32 v22, a200\n\ts_nop 3\n" + MFMA) == []
    assert len(_scan(tmp_path, "\tv_accvgpr_read_b32 v22, a200\n\ts_nop 1\n" + MFMA)) == 1
    # a restored value the matrix instruction does not read
    assert _scan(tmp_path, "\tv_accvgpr_read_b32 v40, a200\n" + MFMA) == []
    # an ordinary vector-ALU producer is interlocked by the hardware
    assert _scan(tmp_path, "\tv_perm_b32 v22, v1, v2, v3\n" + MFMA) == []
    # a matrix instruction the compiler emitted itself (no asm markers) gets its wait states from the compiler
    plain = "\tv_accvgpr_read_b32 v22, a200\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[10:13], v[20:23], a[0:3]\n"
    assert _scan(tmp_path, plain) == []
    # the destination of the matrix instruction is not a source
    assert _scan(tmp_path, "\tv_accvgpr_read_b32 v0, a200\n" + MFMA) == []


def test_accumulator_moves_right_behind_an_asm_matrix_instruction_are_flagged(tmp_path):
    # the compiler copying an accumulator that the asm instruction in front is still writing
    assert len(_scan(tmp_path, MFMA + "\ts_nop 0\n\tv_accvgpr_read_b32 v9, a2\n")) == 1
    assert len(_scan(tmp_path, MFMA + "\tv_accvgpr_mov_b32 a200, a3\n")) == 1
    assert len(_scan(tmp_path, MFMA + "\tv_accvgpr_write_b32 a0, v9\n")) == 1
    assert len(_scan(tmp_path, MFMA + "\tscratch_load_dwordx4 a[0:3], off, off offset:660\n")) == 1
    # other accumulators, or the same ones after the instruction has drained (two s_nop 15, as in front of the epilogues)
    assert _scan(tmp_path, MFMA + "\tv_accvgpr_read_b32 v9, a8\n") == []
    assert _scan(tmp_path, MFMA + "\ts_nop 15\n\ts_nop 15\n\tv_accvgpr_read_b32 v9, a2\n") == []
    # the next matrix instruction on the same accumulator is the hardware's business
    assert _scan(tmp_path, MFMA + MFMA) == []


def _scan_stores(tmp_path, text):
    p = os.path.join(str(tmp_path), "k.s")
    with open(p, "w") as f:
        f.write(text)
    return check_store_hazards(p)


def test_store_data_overwritten_too_early_is_flagged(tmp_path):
    store = "\t;;#ASMSTART\n\tglobal_store_dwordx4 v[8:9], v[0:3], off sc1\n\ts_nop %d\n\t;;#ASMEND\n"
    over = "\tv_add_u32_e32 v2, v4, v5\n"
    assert len(_scan_stores(tmp_path, store % 0 + over)) == 1
    assert _scan_stores(tmp_path, store % 1 + over) == []
    assert _scan_stores(tmp_path, store % 0 + "\ts_add_u32 s0, s1, s2\n" + over) == []
    assert _scan_stores(tmp_path, store % 0 + "\tv_add_u32_e32 v8, v4, v5\n") == []  # the address is read at once
    assert _scan_stores(tmp_path, store % 0 + "\tv_add_u32_e32 v4, v0, v1\n") == []
    # stores the compiler emitted itself get their distance from it
    assert _scan_stores(tmp_path, "\tglobal_store_dwordx4 v[8:9], v[0:3], off\n" + over) == []
    wide = "\t;;#ASMSTART\n\tbuffer_store_dwordx4 v[0:3], v8, s[0:3], 0 offen sc1\n\t;;#ASMEND\n"
    assert len(_scan_stores(tmp_path, wide + over)) == 1


def test_store_past_the_write_back_keeps_its_data(tmp_path):
    """mma.h's asm store, with its value changed as soon as it is issued."""
    src, asm = os.path.join(str(tmp_path), "k.hip"), os.path.join(str(tmp_path), "k.s")
    with open(src, "w") as f:
        f.write("""#include "mma.h"
namespace rtoss {
__global__ void store_and_change(u32x4* p, u32x4 v)
{
    v.x += threadIdx.x;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        store16_through(p + threadIdx.x + i * 64, v);
        v.x = v.x * 3 + v.w;
        v.y ^= v.x;
        v.w += v.y;
    }
}
}
""")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                           "-S", "--cuda-device-only", src, "-o", asm], stderr=subprocess.DEVNULL)
    assert open(asm).read().count("global_store_dwordx4") == 6
    assert check_store_hazards(asm) == []
