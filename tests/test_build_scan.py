"""The build refuses kernels that take the amount of a 64-bit shift from the last vector register of their allocation, and float32 product kernels that spill vector registers."""
from paper_1808_05488_amd import build

ASM = """
_Z1kPf:
\tv_lshlrev_b64 v[2:3], v%d, v[4:5]
\ts_endpgm
\t.amdhsa_kernel _Z1kPf
\t\t.amdhsa_next_free_vgpr %d
\t.end_amdhsa_kernel
"""


def test_the_form_is_found_and_no_other():
    for used, last in ((33, 39), (40, 39), (41, 47), (8, 7)):
        assert build.shifts_by_last_register(ASM % (last, used)) == [("_Z1kPf", f"v_lshlrev_b64 v[2:3], v{last}, v[4:5]")]
        assert build.shifts_by_last_register(ASM % (last - 1, used)) == []
    assert build.shifts_by_last_register(ASM.replace("v%d, v[4:5]", "s%d, v[4:5]") % (39, 40)) == []


METADATA = """
amdhsa.kernels:
  - .agpr_count:     0
    .name:           _Z1kPf
    .private_segment_fixed_size: %d
    .sgpr_spill_count: 7
    .symbol:         _Z1kPf.kd
    .vgpr_count:     168
    .vgpr_spill_count: %d
  - .agpr_count:     0
    .name:           _Z1lPf
    .vgpr_count:     40
    .vgpr_spill_count: %d
"""


def test_spilled_registers_are_found():
    assert build.spilled_registers(METADATA % (0, 0, 0)) == []
    assert build.spilled_registers(METADATA % (8, 1, 0)) == [("_Z1kPf", 1)]
    assert build.spilled_registers(METADATA % (8, 12, 3)) == [("_Z1kPf", 12), ("_Z1lPf", 3)]
    assert build.UNSPILLED <= set(build.SOURCES)
