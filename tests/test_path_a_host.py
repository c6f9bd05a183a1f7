"""The host side of a whole failure event (csrc/path_a.cpp) against a stand-in for the device: where the search's ids come from, and that
errors cost nothing that later events need.  Compiled with the host compiler, under sanitizers."""
import os

from test_sanitize_host import CSRC, ROOT, build_and_run


def test_event_after_errors(tmp_path):
    t = os.path.join(ROOT, "tests")
    build_and_run(tmp_path, "g++", ["-std=c++17", "-Wall", "-I", os.path.join(t, "stub"), "-I", os.path.join(ROOT, "include"), "-I", CSRC],
                  [os.path.join(CSRC, "path_a.cpp"), os.path.join(CSRC, "arc.cpp"), os.path.join(t, "host_path_a.cpp")], "path_a")
