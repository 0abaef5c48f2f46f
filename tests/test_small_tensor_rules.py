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


@pytest.mark.parametrize("kib,one", [(16, True), (128, True), (256, True), (512, True), (640, False), (1024, False)])
def test_tensor_scale_on_the_default_stream(kib, one):
    """Scale, codes and values of 512 KiB take 15.2 us by one workgroup, 15.8 on lent words, which cost the host more;
    scale and fake-quant of 640 KiB 10.0 and 9.3."""
    assert hm.scale_in_one_workgroup_lent(kib * KIB) == one


@pytest.mark.parametrize("kib,with_scratch,without", [(64, True, True), (256, True, True), (320, True, True),
                                                      (384, True, True), (448, False, True), (512, False, True),
                                                      (768, False, True), (832, False, False), (1024, False, False)])
def test_scale_and_codes_in_one_launch(kib, with_scratch, without):
    """Every workgroup reads the whole tensor: 448 KiB take 8.0 us, the two launches with scratch words 7.3, those
    without 9.8; 896 KiB 11.6 and the four launches without 11.0."""
    assert hm.scale_and_codes_in_one_launch(kib * KIB, True) == with_scratch
    assert hm.scale_and_codes_in_one_launch(kib * KIB, False) == without


@pytest.mark.parametrize("rows,cols,bf16,fp32", [(256, 512, True, True), (1024, 1024, True, True), (480, 4096, True, True),
                                                 (1920, 1024, True, True), (1024, 2048, True, False), (256, 8192, True, False),
                                                 (2048, 2048, True, False), (2048, 4096, False, False), (4096, 4096, False, False)])
def test_tensor_scale_after_the_columnwise_transform(rows, cols, bf16, fp32):
    """4 bytes of a row per lane, or 16: 1024 x 2048 fp32 5.3 us by 4, 5.1 by 16; 480 x 4096 5.0 and 5.15."""
    assert hm.scale_by_words(rows // 16 * (cols // 2), False) == bf16
    assert hm.scale_by_words(rows // 16 * cols, True) == fp32
