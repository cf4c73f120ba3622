"""The same assembly checks as for the other kernels with transposing LDS reads, for the launches that
read W itself or rows past 32-bit offsets: every such read is waited for before its registers are
touched; and the K loops of the bf16 GEMM kernels hold no scratch access (a reload there would wait for
the loads in flight)."""
import os

import pytest

from tests.test_kernel_asm import CSRC, _body, _compile, _regs, _uses_before_wait

DIRECT = "_ZN6fastrl20lm_bwd_direct_kernelENS_10GemmParamsES0_"
BWD = "_ZN6fastrl13lm_bwd_kernelENS_10GemmParamsES0_"
GEMM = "_ZN6fastrl14lm_gemm_kernelItLi%dEEEvNS_10GemmParamsE"  # 0 logits, 1 dhidden, 3 dW
WIDE = "_ZN6fastrl14lm_wide_kernelILi%dEEEvNS_10GemmParamsE"   # 3 dW, 4 dhidden from W itself


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    return _compile(os.path.join(CSRC, "lmhead.hip"), tmp_path_factory.mktemp("asm"))


@pytest.mark.parametrize("kernel, at_least", [(DIRECT, 48), (WIDE % 3, 24), (WIDE % 4, 24)])
def test_direct_transposing_reads_are_waited_for(asm, kernel, at_least):
    lines = _body(asm, kernel)
    reads = [k for k, (kind, op, _) in enumerate(lines) if op == "ds_read_b64_tr_b16"]
    assert len(reads) >= at_least, len(reads)  # (DIRECT: dhidden and dW)
    for k in reads:
        dest = _regs(lines[k][2].split(",")[0])
        assert len(dest) == 2 and not _uses_before_wait(lines, k, dest), lines[k]


def _k_loops(asm, kernel):
    """(MFMAs, direct loads, operations) of each backward branch over one K tile: 16, 32, 48 or 64 MFMAs
    for 64 to 256 tokens, four loads of A and one of B per 64 columns."""
    lines = _body(asm, kernel)
    where = {name: k for k, (kind, name, _) in enumerate(lines) if kind == "label"}
    for k, (kind, op, args) in enumerate(lines):
        if not op.startswith("s_cbranch") or where.get(args.strip(), k) >= k:
            continue
        ops = [o for kind2, o, _ in lines[where[args.strip()]:k] if kind2 == "inst"]
        mfma = sum(o.startswith("v_mfma") for o in ops)
        loads = sum(o.startswith("global_load_lds") for o in ops)
        if mfma in (16, 32, 48, 64) and loads == 4 + mfma // 16:
            yield mfma, loads, ops


@pytest.mark.parametrize("kernel", [DIRECT, BWD, GEMM % 0, GEMM % 1, GEMM % 3])
def test_no_scratch_in_the_main_k_loops(asm, kernel):
    """No K loop touches scratch, and each of a kernel's contractions has its loops among those looked
    at: all four widths of logits tiles, dhidden and dW of the joint launches."""
    loops = list(_k_loops(asm, kernel))
    for mfma, loads, ops in loops:
        assert not [o for o in ops if o.startswith("scratch_")], (kernel, mfma)
    transposing = [sum(o.startswith("ds_read_b64_tr") for o in ops) for _, _, ops in loops]
    # rows of W past the vocabulary's end are clamped, in the loop of dhidden alone
    clamped = [any(o.startswith("s_min") for o in ops) for _, _, ops in loops]
    if kernel == GEMM % 0:
        assert {m for m, _, _ in loops} == {16, 32, 48, 64} and not any(transposing)
    else:
        assert {m for m, _, _ in loops} == {64}
        if kernel == BWD:
            assert set(transposing) == {0, 16}
        elif kernel == DIRECT:
            assert set(transposing) == {16} and set(clamped) == {False, True}
        else:
            assert set(transposing) == {16 if kernel == GEMM % 3 else 0}
