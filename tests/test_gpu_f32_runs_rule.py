"""GPU parity of fp32 products in tiles of 32 x 32 on either side of the line between results that leave in runs of four and one by one,
the instance asserted: columns two apart with whole and with dropped rows, three apart, none dropped; all three operand layouts."""
import pytest

import dryrun as D
import test_gpu_f32_runs as runs

pytestmark = pytest.mark.gpu

RUNS, SINGLE = "gemm_f32_kernel<runs><32, 32, 0>", "gemm_f32_kernel<32, 32, 0>"


def _instances(B, I, O, po, pi, flags, op):
    with D.dry_run() as lib:
        D.launches(lib)
        assert D.layer_calls(lib, D.FakeHeap(), D.F32, B, I, O, po, pi, flags, ops=(op,)) == [0]
        return [i for i in D.instances(lib) if i.startswith("gemm_f32_kernel")]


@pytest.mark.parametrize("B,I,O,po,pi,want", [(55, 254, 2688, (1, 1), (2, 2), SINGLE), (55, 254, 2688, (2, 1), (2, 1), RUNS), (81, 476, 768, (1, 1), (3, 2), RUNS),
                                              (55, 258, 1344, (2, 2), (1, 1), SINGLE)])
def test_weight_gradient(B, I, O, po, pi, want):
    assert _instances(B, I, O, po, pi, D.ard.IN_COMPACT | D.ard.OUT_COMPACT, 2) == [want]
    runs.test_weight_gradient_of_compact_operands(B, I, O, po, pi)


@pytest.mark.parametrize("B,I,O,po,pi,want", [(208, 251, 2240, (2, 2), (3, 1), SINGLE), (188, 124, 3456, (5, 2), (6, 4), RUNS)])
def test_forward(B, I, O, po, pi, want):
    assert _instances(B, I, O, po, pi, 0, 0) == [want]
    runs.test_strided_operands(B, I, O, po, pi)


@pytest.mark.parametrize("B,I,O,po,pi,want", [(131, 2752, 396, (4, 3), (2, 2), SINGLE), (251, 3005, 430, (2, 1), (3, 2), RUNS)])
def test_data_gradient(B, I, O, po, pi, want):
    assert _instances(B, I, O, po, pi, 0, 1) == [want]
    runs.test_strided_operands(B, I, O, po, pi)
