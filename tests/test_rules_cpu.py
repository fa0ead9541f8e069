"""The rules that kernels and host code share (csrc/rules.h) and the gate that resident launches pass
(csrc/chip_gate.h), checked on the CPU by a host build."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "driver")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", os.path.join(ROOT, "paper_0811_2518_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host_rules", "driver.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def check(driver, name):
    r = subprocess.run([driver, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_check_sums_are_never_overwritten_while_read(driver):
    check(driver, "sum_words")


def test_partials_keep_their_bits_and_are_not_taken_early(driver):
    check(driver, "partials")


def test_no_team_is_larger_than_the_grid(driver):
    check(driver, "teams")


def test_groups_of_right_hand_sides(driver):
    check(driver, "groups")


def test_launches_that_wait_for_each_other_enter_in_turn(driver):
    check(driver, "gate")


def test_failed_launches_are_tried_ever_more_rarely(driver):
    check(driver, "backoff")
