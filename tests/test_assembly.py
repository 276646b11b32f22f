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


def test_data_of_wide_stores_is_not_overwritten(kernels):
    """A store of more than eight bytes reads its data for two wait states after it was issued.  Those that are inline assembly bring the wait along,
    since what the compiler places behind them changes with every change of the kernel."""
    through, overwritten = 0, []
    for name, code in kernels.items():
        for i, ins in enumerate(code):
            if not ins.startswith(("global_store_dwordx4", "global_store_dwordx3", "flat_store_dwordx4", "flat_store_dwordx3", "buffer_store_dwordx4", "buffer_store_dwordx3")):
                continue
            if ins.endswith("sc0 sc1"):
                through += 1
                assert code[i + 1] == "s_nop 1", (name, code[i:i + 3])
            data = assembly.registers(assembly.operands(ins)[0 if ins.startswith("buffer") else 1])
            states = 0
            for behind in code[i + 1:i + 3]:
                if behind.startswith(("s_branch", "s_endpgm", "s_setpc")):
                    break
                if states < 2 and behind.startswith("v_") and data & assembly.registers(assembly.operands(behind)[0]):
                    overwritten.append((name, ins, behind, states))
                states += assembly.wait_states(behind)
    assert through >= 8                                    # copy out, and four forms of the classifier's end
    assert not overwritten, (len(overwritten), overwritten[:5])


def test_the_end_of_a_classifier_writes_everything_through(kernels):
    """The launch that raises the host's flag itself: the host may then give the instance, and with it the device's copy of the result, to another stream
    before that launch has ended.  None of its stores may stay in a compute unit's or a chiplet's cache until then."""
    ends = {name: [i for i in code if "_store_" in i and not i.startswith("ds_")] for name, code in kernels.items() if "classify_out_kernel" in name}
    assert len(ends) == 4
    for name, stores in ends.items():
        assert len(stores) >= 6                            # logits, probabilities, index, stamps, flag
        cached = [i for i in stores if not i.endswith("sc1")]
        assert not cached, (name, cached)
