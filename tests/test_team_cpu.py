"""The rules by which a team of workgroups meets and by which the next launch
takes its projector (csrc/team.h), in 20000 random orders of events: a projector
that stands has every workgroup's blocks, whoever was late, and where nobody is
late it stands."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2506_10257_amd", "csrc")


def test_a_projector_that_stands_is_complete(tmp_path):
    exe = str(tmp_path / "team_model")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, os.path.join(HERE, "team_model.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe, "20000"], check=True, capture_output=True, text=True, timeout=100).stdout
    stands, falls, wrong = map(int, out.split())
    assert stands > 1000 and falls > 1000, out
    assert wrong == 0, out
