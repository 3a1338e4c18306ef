"""The build's check of the register-plane kernels' register allocation
(check_regplane_alloc).  No GPU needed."""
import pytest

from paper_2105_01533_amd.build import check_regplane_alloc


def _kernel(name, total, arch):
    return (f"\t.amdhsa_kernel {name}\n\t\t.amdhsa_group_segment_fixed_size 2048\n"
            f"\t\t.amdhsa_next_free_vgpr {total}\n\t\t.amdhsa_next_free_sgpr 100\n"
            f"\t\t.amdhsa_accum_offset {arch}\n\t.end_amdhsa_kernel\n")


ALONE, SHARED = "_Z10kb_mono_rpPK5BTick", "_Z9k_mono_rpILb1EEv3Buf"


@pytest.mark.parametrize("kernels, ok", [
    ([(ALONE, 296, 232), (SHARED, 231, 232)], True),
    ([(ALONE, 257, 232), (SHARED, 231, 232)], True),
    ([(ALONE, 256, 232), (SHARED, 231, 232)], False),   # two waves fit
    ([(ALONE, 231, 232), (SHARED, 231, 232)], False),   # the AGPRs are gone
    ([(ALONE, 296, 80), (SHARED, 231, 232)], False),    # the planes' registers are
    ([(ALONE, 296, 232), (SHARED, 80, 80)], False),
    ([(SHARED, 231, 232)], False),                      # the kernel is not there
])
def test_allocation_guard(kernels, ok):
    assert (check_regplane_alloc("".join(_kernel(*k) for k in kernels)) == []) is ok
