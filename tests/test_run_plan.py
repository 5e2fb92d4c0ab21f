"""The schedule words of a run (gem_plan.hpp, plan_run), replayed on the CPU the
way the run kernel moves chunks, with the sanitizers the pass plan's test uses."""
import shutil

import pytest

from test_plan import _build_and_run


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
@pytest.mark.parametrize("seed", [1, 2018])
def test_run_words_replay_the_sequential_commits(tmp_path, seed):
    _build_and_run(tmp_path, "run_plan_driver.cpp", seed)
