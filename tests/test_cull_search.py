"""The constant-culling search (csrc/pa_search.hpp), compiled for the CPU, against
the 64-halving bisection that defines the step: equal in every bit, for both ways
the evaluations are summed and both numbers of evaluations per round."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1711_02146_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("cull") / "cull_search_ref")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I" + CSRC,
                           os.path.join(HERE, "cull_search_ref.cpp"), "-o", exe])
    return exe


@pytest.mark.parametrize("lanes", [7, 3])
@pytest.mark.parametrize("sums", ["sequential", "exact"])
def test_search_equals_bisection(program, lanes, sums):
    p = subprocess.run([program, "1500", str(lanes), sums], capture_output=True, text=True)
    bad, n, evals, rounds = (int(v) for v in p.stdout.split())
    assert n == 1500 and bad == 0 and p.returncode == 0
    assert rounds <= (40 if lanes == 7 else 70)  # 64 halvings and the interpolation's rounds
    assert evals < 66 * n                        # the bisection's own count


@pytest.mark.parametrize("lanes", [7, 3])
def test_search_is_exact_within_the_evaluations_error_bound(tmp_path, lanes):
    """Evaluations as far off as their bound allows, on curves that are flat next to
    the target, with a bound that grows by much over the range: a candidate above the
    target decides the ones beyond it only by the bound that holds there."""
    exe = str(tmp_path / "cull_bounds_ref")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I" + CSRC,
                           os.path.join(HERE, "cull_bounds_ref.cpp"), "-o", exe])
    bad, n = (int(v) for v in subprocess.check_output([exe, "20000", str(lanes)]).split())
    assert n == 20000 and bad == 0
