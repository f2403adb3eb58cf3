"""The word exchange of the eigensolver's reduction on the chip, modelled on the CPU: no order of its workgroups' memory accesses may
make one wait for ever or take the words of another column."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("ring") / "chip_ring_model")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2007_00784_amd", "csrc"), os.path.join(ROOT, "tests", "chip_ring_model.cpp"), "-o", exe],
                   check=True, timeout=120)
    return lambda rule, orders: subprocess.run([exe, rule, str(orders)], check=True, timeout=120, capture_output=True, text=True).stdout.strip()


def test_exchange_in_any_order(model):
    assert model("ring", 60) == "ok"


def test_model_sees_a_workgroup_that_leaves_without_a_receipt(model):
    """Others then empty the words of its last column while it may still look for them."""
    assert model("unacknowledged", 60) != "ok"
