"""Host side of the one-launch tree levels: trees dealt out to groups, levels listed group by group."""
import os

from tests.test_sanitizers import CSRC, ROOT, build_and_run


def test_groups_partition_the_internal_levels(tmp_path):
    src = [os.path.join(ROOT, "tests", "sanitize", "grouping_driver.cpp"), os.path.join(CSRC, "scheduler.cpp")]
    build_and_run(tmp_path, "g++", "-std=c++17", src, "grouping_driver", [])
