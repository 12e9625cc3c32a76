"""The build-time device-code checker recognises a barrier inside a loop that
lanes leave one by one (the shape that livelocks a persistent tile loop) and
accepts the same loop with a wave-uniform exit."""
import importlib.util
import os

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CHECKER = os.path.join(HERE, "..", "paper_2212_08058_amd", "isa_check.py")

LANE_EXIT = """_Z6kernelv:                              ; @_Z6kernelv
; %bb.0:
	s_branch .LBB0_2
.LBB0_1:                                ;   in Loop: Header=BB0_2 Depth=1
	s_andn2_b64 exec, exec, s[4:5]
	s_cbranch_execz .LBB0_3
.LBB0_2:                                ; =>This Loop Header: Depth=1
	s_barrier
	ds_read_b32 v0, v1
	s_branch .LBB0_1
.LBB0_3:
	s_endpgm
.Lfunc_end0:
"""

UNIFORM_EXIT = LANE_EXIT.replace("s_andn2_b64 exec, exec, s[4:5]\n\ts_cbranch_execz", "s_cmp_ge_i32 s6, s7\n\ts_cbranch_scc1")


@pytest.fixture(scope="module")
def checker():
    if not os.path.exists(CHECKER):
        pytest.skip("device-code checker not present in this tree")
    spec = importlib.util.spec_from_file_location("stpi_isa_check_test", CHECKER)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("words,bad", [
    (("s", "load", "dwordx4"), False), (("s", "buffer", "load", "dword"), False), (("s", "mov", "b32"), False),
    (("global", "store", "dword"), False), (("ds", "add", "u32"), False), (("s", "store", "dword"), True),
    (("s", "buffer", "store", "dword"), True), (("s", "atomic", "add"), True), (("s", "dcache", "wb"), True)])
def test_scalar_memory_is_for_loads(checker, words, bad):
    assert checker._scalar_memory_write("_".join(words)) == bad


def test_flags_barrier_in_lane_divergent_loop(checker):
    assert checker._loops_with_barrier_and_lane_exit(LANE_EXIT) == [("_Z6kernelv", "BB0_2")]


def test_accepts_uniform_loop_exit(checker):
    assert checker._loops_with_barrier_and_lane_exit(UNIFORM_EXIT) == []


def test_accepts_lane_divergent_loop_without_barrier(checker):
    assert checker._loops_with_barrier_and_lane_exit(LANE_EXIT.replace("\ts_barrier\n", "")) == []


PRODUCT = """_Z6kernelv:
.LBB0_1:
	v_mfma_f32_16x16x32_f16 v[0:3], v[4:7], v[8:11], v[12:15]
{between}	;;#ASMSTART
	v_fma_mixlo_f16 {dst}, {src}, v41, 0
	;;#ASMEND
{back}	s_cbranch_scc1 .LBB0_1
	s_endpgm
.Lfunc_end0:
"""


@pytest.mark.parametrize("dst,src,states,ok", [
    ("v2", "v40", 7, False), ("v2", "v40", 8, True),      # writes the result
    ("v42", "v1", 7, False), ("v42", "v1", 8, True),      # reads it
    ("v13", "v40", 2, False), ("v13", "v40", 3, True),    # writes the C operand
    ("v42", "v13", 0, True), ("v42", "v40", 0, True),     # reads the C operand; no overlap
])
def test_inline_assembly_behind_a_product(checker, dst, src, states, ok):
    between = "" if states == 0 else "\ts_nop %d\n" % (states - 1)
    text = PRODUCT.format(between=between, dst=dst, src=src, back="\ts_nop 0\n")
    found = checker._matrix_core_waits(text)
    assert (found == []) == ok, found
    # the compiler's own instructions are its business
    assert checker._matrix_core_waits(text.replace("\t;;#ASMSTART\n", "").replace("\t;;#ASMEND\n", "")) == []


@pytest.mark.parametrize("back,ok", [("", False), ("\ts_nop 0\n", True)])
def test_inline_assembly_in_front_of_a_product(checker, back, ok):
    # around the loop: a write of an operand, a branch, the product
    found = checker._matrix_core_waits(PRODUCT.format(between="", dst="v9", src="v40", back=back))
    assert [(n, need) for _, _, _, n, need in found] == ([] if ok else [(1, 2)])


@pytest.mark.parametrize("second,states,ok", [
    ("v_mfma_f32_16x16x16_bf16 v[0:3], v[16:17], v[18:19], v[0:3]", 0, False),
    ("v_mfma_f32_16x16x16_bf16 v[0:3], v[16:17], v[18:19], v[0:3]", 3, False),
    ("v_mfma_f32_16x16x16_bf16 v[0:3], v[16:17], v[18:19], v[0:3]", 4, True),
    ("v_mfma_f32_16x16x32_bf16 v[0:3], v[16:19], v[20:23], v[0:3]", 0, True),       # the same shape
    ("v_mfma_f32_16x16x16_bf16 v[24:27], v[16:17], v[18:19], v[24:27]", 0, True)])  # another accumulator
def test_products_of_two_shapes_on_one_accumulator(checker, second, states, ok):
    nop = "\ts_nop %d\n" % (states - 1) if states else ""
    text = ("_Z6kernelv:\n\tv_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], v[8:11], v[12:15]\n" + nop + "\t" + second +
            "\n\ts_endpgm\n.Lfunc_end0:\n")
    found = checker._matrix_core_waits(text)
    assert [(n, need) for _, _, _, n, need in found] == ([] if ok else [(states, 4)])


def test_built_device_code_keeps_the_waits(checker):
    """The assembly the last build left: matrix-core products are there, and
    nothing lies too close to one."""
    path = os.path.join(HERE, "..", "_build")
    files = [f for f in ("kernels_f32.hip.s", "kernels_bf16.hip.s", "sfseg.hip.s", "net.hip.s") if os.path.exists(os.path.join(path, f))]
    if not files:
        pytest.skip("no device assembly here")
    for f in files:
        with open(os.path.join(path, f)) as fh:
            text = fh.read()
        assert "v_mfma_f32_" in text
        assert checker._matrix_core_waits(text) == []
