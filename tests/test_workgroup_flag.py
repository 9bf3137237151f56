"""What one thread of a workgroup finds out for all, by threads of the host under ThreadSanitizer: the word that carries
it may be written again at once, so every thread must have read it before any leaves."""
import os
import shutil
import subprocess

import pytest

from paper_2604_16855_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = os.path.join(HERE, "host_sanitizer", "workgroup_flag.cpp")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_flag_is_read_by_all_before_it_is_written_again(tmp_path):
    exe = str(tmp_path / "workgroup_flag")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-pthread", "-I", B.CSRC, SOURCE, "-o", exe],
                       capture_output=True, text=True)
    if r.returncode != 0 and "tsan" in r.stderr:
        pytest.skip("no ThreadSanitizer for g++")
    assert r.returncode == 0, r.stderr
    # (it needs fixed places for its own memory)
    run = ["setarch", "-R", exe] if shutil.which("setarch") else [exe]
    r = subprocess.run(run, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "0 wrong" in r.stdout, r.stdout + r.stderr[-4000:]


def test_the_rank_select_asks_through_it():
    """Workgroups that share a set find out by this alone whether they are the last and what has been reached."""
    text = open(os.path.join(B.CSRC, "tdq_rank.hip")).read()
    body = text[text.index("auto shared_rank ="):text.index("auto one_rank =")]
    used = body.count("known_to_all(&s_known,")
    assert used >= 2 and body.count("s_known") == used
    assert text.count("s_known") == used + 1                     # its declaration
    # thread 0 polls and counts nowhere else
    assert body.count("until(patience,") == 1 and body.count("arrive(n_parts) ==") == 1
