"""The rules that pick a launch's form (csrc/launch_rules.h), evaluated on the host: where
they were measured to be right, they stay.  CPU only."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2606_21712_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="session")
def rules(tmp_path_factory):
    """rules(lines) -> the choice for each line "rule arg arg ..."."""
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC,
                    os.path.join(HERE, "native", "launch_rules.cpp"), "-o", exe], check=True)

    def ask(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        out = r.stdout.splitlines()
        assert len(out) == len(lines)
        return out
    return ask


def test_permute_groups(rules):
    """Every size fits its groups; the largest sizes get no more than they fill by a third."""
    sizes = [1, 64, 1024, 1025, 2048, 2049, 4096, 4097, 6144, 6145, 8192, 8193, 12288, 12289, 16384]
    for R, n in zip(sizes, map(int, rules([f"permute {R}" for R in sizes]))):
        assert n <= 16 and n * 1024 >= R, (R, n)
        assert R <= 4096 or n * 1024 < 1.5 * R + 1024, (R, n)
