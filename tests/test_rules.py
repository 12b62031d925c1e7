"""The scheduler's rules, walked on the CPU: csrc/dfx_rules.h is what the kernel compiles, tests/rules/rules_check.cpp puts its functions
through small models of what the kernel does with them (a fetch that runs on, ...), plain g++, no GPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rules") / "rules_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "rules", "rules_check.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("model", ["tables", "gangs", "turns", "rings"])
def test_rules(check, model):
    """tables: a job moves the buffers of its own invocation, also where the collective comes again in the fetch that brought a table.
    gangs: a pass hands the movers its bytes and no more, however many short collectives go together, but for a first one that is longer.
    turns: while short collectives keep coming, one that is not short has its turn, also behind others that look runnable and are not.
    rings: a fetch goes on only where its 32-bit offsets reach every slot of the SQ."""
    res = subprocess.run([check, model], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
