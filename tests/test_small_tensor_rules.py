"""CPU: up to which size a tensor takes the small-tensor kernels (csrc/small_tensors.hpp, compiled for the
host), on both sides of every line, at sizes where both were timed."""
import pytest

from . import _host_model as hm

KIB = 1024


@pytest.mark.parametrize("kib,with_scratch,without", [(16, True, True), (128, True, True), (160, False, True),
                                                      (256, False, True), (512, False, True),
                                                      (768, False, True), (832, False, False),
                                                      (1024, False, False)])
def test_tensor_scale_in_one_workgroup(kib, with_scratch, without):
    """One workgroup reads at what one compute unit can: called one by one, 1 MiB takes it 11.2 us, as three
    launches; with scratch words, where it saves no launch, 160 KiB from memory 5.7 / 4.3."""
    assert hm.scale_in_one_workgroup(kib * KIB, True) == with_scratch
    assert hm.scale_in_one_workgroup(kib * KIB, False) == without


@pytest.mark.parametrize("kib,with_scratch,without", [(64, True, True), (256, True, True), (320, True, True),
                                                      (384, True, True), (448, False, True), (512, False, True),
                                                      (768, False, True), (832, False, False), (1024, False, False)])
def test_scale_and_codes_in_one_launch(kib, with_scratch, without):
    """Every workgroup reads the whole tensor: 448 KiB take 8.0 us, the two launches with scratch words 7.3, those
    without 9.8; 896 KiB 11.6 and the four launches without 11.0."""
    assert hm.scale_and_codes_in_one_launch(kib * KIB, True) == with_scratch
    assert hm.scale_and_codes_in_one_launch(kib * KIB, False) == without
