"""What the build refuses: scratch memory and compiler-made copies of accumulators in kernels that cannot bear them."""
import pytest

from paper_2602_23592_amd import build

KERNEL = "_ZN4keep10k_gemm_256ILi0EEEv"


def _assembly(inside, outside):
    return "_Zother:\n\tv_accvgpr_read_b32 v0, a1\n.Lfunc_end0:\n%s: ; @\n\t;;#ASMSTART\n\t%s\n\t;;#ASMEND\n\t%s ; a7\n.Lfunc_end1:\n" % (
        KERNEL, inside, outside)


@pytest.mark.parametrize("line", ["v_accvgpr_mov_b32 a3, a4", "v_accvgpr_read_b32 v3, a0", "scratch_store_dwordx4 off, a[0:3], s0",
                                  "v_mfma_f32_16x16x32_bf16 a[4:7], v[0:3], v[4:7], a[4:7]"])
def test_accumulators_belong_to_the_inline_assembly(line):
    build.check_accumulators("gemm_mfma.hip", _assembly(line, "v_mov_b32 v1, v2"))
    with pytest.raises(RuntimeError, match="touches an accumulator"):
        build.check_accumulators("gemm_mfma.hip", _assembly("v_nop", line))


def test_a_report_that_names_no_kernel_is_refused():
    with pytest.raises(RuntimeError):
        build.check_accumulators("gemm_mfma.hip", "_Zother:\n.Lfunc_end0:\n")
    with pytest.raises(RuntimeError):
        build.check_scratch("gemm_stream.hip", "")


@pytest.mark.parametrize("src,kernel", [("gemm_mfma.hip", "k_gemm_256"), ("gemm_stream.hip", "k_gemm_stream")])
def test_scratch_is_refused(src, kernel):
    report = "remark: Function Name: _Z%s\nremark: ScratchSize [bytes/lane]: %d\nremark: Function Name: _Zother\n" \
             "remark: ScratchSize [bytes/lane]: 8\n"
    build.check_scratch(src, report % (kernel, 0))
    with pytest.raises(RuntimeError, match="scratch"):
        build.check_scratch(src, report % (kernel, 4))
