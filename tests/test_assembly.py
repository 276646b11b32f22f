"""What the compiler cannot see to: instructions written as inline assembly, whose hazards it does not know.  Checked in the built library's gfx950
code, without a GPU.  (CDNA3 / CDNA4 instruction set, the wait states that the program has to insert.)
"""
import os

import pytest

import assembly
import paper_2604_28175_amd

LIBRARY = os.path.join(os.path.dirname(paper_2604_28175_amd.__file__), "libstrait.so")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not (os.path.exists(assembly.OBJDUMP) and os.path.exists(assembly.OBJCOPY)):
        pytest.skip("no disassembler")
    k = assembly.kernels(LIBRARY, str(tmp_path_factory.mktemp("code")))
    assert sum("conv_igemm_dma_kernel" in name for name in k) > 50 and any("classify_out_kernel" in name for name in k)
    return k


def test_scalar_operands_of_transfers_into_lds(kernels):
    """A transfer reads its scalar registers five wait states after a vector instruction (v_readlane of a spilled one, for instance) has written them."""
    transfers, early = 0, []
    for name, code in kernels.items():
        for i, ins in enumerate(code):
            if not (ins.startswith("buffer_load_dword") and ins.endswith(" lds")):
                continue
            transfers += 1
            reads = set().union(*(assembly.registers(o) for o in assembly.operands(ins)))
            reads = {r for r in reads if r[0] == "s"}
            states = 0
            for before in reversed(code[max(0, i - 5):i]):
                if states >= 5 or before.startswith(("s_branch", "s_endpgm")):
                    break
                if before.startswith("v_") and reads & assembly.registers(assembly.operands(before)[0]):
                    early.append((name, before, ins, states))
                states += assembly.wait_states(before)
    assert transfers > 1000
    assert not early, (len(early), early[:5])
