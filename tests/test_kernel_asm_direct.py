"""The same assembly checks as for the other kernels with transposing LDS reads, for the launch that
reads W itself: every such read is waited for before its registers are touched, and the K loops of the
bf16 GEMM kernels hold no scratch access (a reload there would wait for the loads in flight)."""
import os
import re

import pytest

from tests.test_kernel_asm import CSRC, _body, _compile, _regs, _uses_before_wait

DIRECT = "_ZN6fastrl20lm_bwd_direct_kernelENS_10GemmParamsES0_"
GEMMS = [DIRECT, "_ZN6fastrl13lm_bwd_kernelENS_10GemmParamsES0_",
         "_ZN6fastrl14lm_gemm_kernelItLi0EEEvNS_10GemmParamsE"]


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    return _compile(os.path.join(CSRC, "lmhead.hip"), tmp_path_factory.mktemp("asm"))


def test_direct_transposing_reads_are_waited_for(asm):
    lines = _body(asm, DIRECT)
    reads = [k for k, (kind, op, _) in enumerate(lines) if op == "ds_read_b64_tr_b16"]
    assert len(reads) >= 48, len(reads)  # dhidden and dW
    for k in reads:
        dest = _regs(lines[k][2].split(",")[0])
        assert len(dest) == 2 and not _uses_before_wait(lines, k, dest), lines[k]


@pytest.mark.parametrize("kernel", GEMMS)
def test_no_scratch_in_the_main_k_loops(asm, kernel):
    """The main K loops are the backward branches over at least 60 MFMAs and 8 direct loads."""
    lines = _body(asm, kernel)
    where = {name: k for k, (kind, name, _) in enumerate(lines) if kind == "label"}
    loops = 0
    for k, (kind, op, args) in enumerate(lines):
        if not op.startswith("s_cbranch") or where.get(args.strip(), k) >= k:
            continue
        ops = [o for kind2, o, _ in lines[where[args.strip()]:k] if kind2 == "inst"]
        mfma = sum(o.startswith("v_mfma") for o in ops)
        if 60 <= mfma <= 80 and sum(o.startswith("global_load_lds") for o in ops) >= 8:
            loops += 1
            assert not [o for o in ops if o.startswith("scratch_")], (kernel, k)
    assert loops >= 1
