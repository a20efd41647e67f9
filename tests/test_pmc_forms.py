"""Which kernels a class of the traffic table may be made of (no GPU): every
entry of the committed table is one of its class's forms, so that bench.py can
report it, a form of one method is not taken for another's, and the step's
coefficient kernel counts where it is launched."""
import json
from pathlib import Path

from paper_1701_02005_amd import pmc_traffic as T

ROOT = Path(__file__).resolve().parent.parent


def test_entries_of_the_table_are_known_forms():
    for key, ent in json.loads((ROOT / "profiles" / "traffic.json").read_text()).items():
        workload, precision, cls = key.split("/")
        cn_rows = "k_cn_rows" in ent["kernels"]
        assert tuple(ent["kernels"]) in T.class_forms(cls, cn_rows=cn_rows), key


def test_forms_of_other_methods_stay_apart():
    assert ("k_lines_z",) in T.class_forms("fft_z_fwd") and ("k_lines_z",) not in T.class_forms("fft_z_fwd", z_fused=True)
    assert T.class_forms("fft_z_inv", z_fused=True) == (("k_zthomas_bwd",),)
    assert T.class_forms("cn_tridiag") == (("k_cn_coef", "k_cn_scan"),)
    assert T.class_forms("cn_tridiag", cn_rows=True) == (("k_cn_coef", "k_cn_rows"),)
    assert {("k_thomas_tile",), ("k_mode_rows",), ("k_mode_columns",)} == set(T.class_forms("thomas_modes"))
    assert ("k_lines_r2c",) in T.class_forms("fft_x_r2c", z_fused=True)


def test_coefficient_kernel_in_the_step_class():
    assert T.class_kernels("dt") == ("k_dt_partial", "k_cn_coef")
