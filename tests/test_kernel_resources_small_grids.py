"""Occupancy of the kernels that small grids and open boundaries run (direct
stores, open faces) and of the FP32 step, from the compiler's report: a code
change that costs one of them a wave shows up here."""
import pytest

from test_kernel_resources import _find, report  # noqa: F401


def _mangled(name, storage, model, offset="j"):
    return f"_ZN4tlbm{len(name)}{name}ILi{storage}ELi{model}E{offset}EE"


@pytest.mark.parametrize("name", ["k_step", "k_step_direct"])
@pytest.mark.parametrize("storage,model,waves", [(0, 0, 4), (0, 1, 5), (0, 2, 4), (0, 3, 4), (1, 0, 8), (1, 1, 8), (1, 2, 8),
                                                 (1, 3, 8), (2, 0, 7), (2, 1, 7), (2, 2, 7), (2, 3, 7)])
def test_steps(report, name, storage, model, waves):  # noqa: F811
    assert _find(report, _mangled(name, storage, model))["Occupancy"] >= waves


@pytest.mark.parametrize("name", ["k_step_open", "k_step_open_direct"])
@pytest.mark.parametrize("storage,model,waves", [(0, 0, 4), (0, 1, 5), (0, 2, 4), (1, 0, 7), (1, 1, 7), (2, 0, 7), (2, 1, 7)])
def test_open_steps(report, name, storage, model, waves):  # noqa: F811
    assert _find(report, _mangled(name, storage, model))["Occupancy"] >= waves


# staged and direct; of the FP64 LBMRT ones the direct serve the grids of fuller tiles, on 2 waves
@pytest.mark.parametrize("storage,model,staged,direct", [(0, 0, 3, 3), (0, 1, 3, 3), (0, 2, 3, 2), (0, 3, 3, 2),
                                                         (1, 0, 6, 6), (1, 1, 8, 8), (1, 2, 4, 4), (1, 3, 5, 5)])
def test_adjoint_steps(report, storage, model, staged, direct):  # noqa: F811
    assert _find(report, _mangled("k_adj_step", storage, model))["Occupancy"] >= staged
    assert _find(report, _mangled("k_adj_step_direct", storage, model))["Occupancy"] >= direct


@pytest.mark.parametrize("storage,fields,sums", [(0, 5, 6), (1, 6, 7), (2, 6, 7)])
def test_macroscopic(report, storage, fields, sums):  # noqa: F811
    assert _find(report, f"_ZN4tlbm8k_fieldsILi{storage}ELb1EE")["Occupancy"] >= fields
    assert _find(report, f"_ZN4tlbm8k_fieldsILi{storage}ELb0EE")["Occupancy"] >= sums
