"""The build's own checks of the compiled convolution kernel refuse what it cannot run with."""
import pytest

GOOD = """_ZN2hb19conv3x3_mfma_kernelENS_8ConvArgsE:
\t;;#ASMSTART
\ts_mov_b32 m0, s4
\t;;#ASMEND
""" + "\tv_mfma_f32_16x16x32_f16 v[78:81], a[72:75], v[0:3], 0\n" * 64 + "\ts_endpgm ; m0\n.Lfunc_end0:\n\ts_mov_b32 m0, s4\n"


@pytest.mark.parametrize("bad", [GOOD.replace("\ts_endpgm", "\tv_accvgpr_write_b32 a0, v1\n\ts_endpgm"), GOOD.replace("\ts_endpgm", "\ts_mov_b32 m0, s7\n\ts_endpgm"),
                                 GOOD.replace(", a[", ", v[")],
                         ids=["copy", "m0", "weights"])
def test_conv3x3_registers(bad):
    import __graft_entry__ as entry
    entry._check_conv3x3(GOOD)
    with pytest.raises(RuntimeError, match="conv3x3_mfma_kernel"):
        entry._check_conv3x3(bad)
