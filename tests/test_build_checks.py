"""The build's checks on the compiler's resource remarks (no GPU, no compiler)."""
import pytest

from paper_1712_01537_amd import build


def _remarks(name, scratch):
    return (f"a.hip:1:1: remark: Function Name: {name} [-Rpass-analysis=kernel-resource-usage]\n"
            f"a.hip:1:1: remark:     ScratchSize [bytes/lane]: {scratch} [-Rpass-analysis]\n")


SP3 = "_ZN12_GLOBAL__N_110k_conv_sp3ILi4ELi8ELb0ELb1ELb%dEEEvPKilPKfiS4_iPfi"


@pytest.mark.parametrize("text,name,scratch,word", [
    ("", SP3 % 0, 0, ""),
    ("", SP3 % 0, 448, "registers"),
    ("", SP3 % 1, 64, ""),  # inputs of 4 GiB and more
    ("", "_ZN12_GLOBAL__N_110k_conv_dwsILi2ELb0EEEvPKillPKf", 8, "registers"),
    ("", "_ZN12_GLOBAL__N_16k_quantEv", 8, ""),
    ('asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N));', "_ZN12_GLOBAL__N_16k_quantEv", 8, "counted"),
])
def test_scratch_fault(text, name, scratch, word):
    why = build.scratch_fault(text, _remarks("other", 0) + _remarks(name, scratch))
    assert bool(why) == bool(word) and word in why
