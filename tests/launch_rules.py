"""Asks the library's launch rules on the CPU (launch_rules_driver.cpp)."""
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2601_07892_amd", "csrc")


@functools.lru_cache(maxsize=None)
def _driver():
    out = os.path.join(tempfile.mkdtemp(prefix="launch_rules"), "driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + CSRC,
                    os.path.join(HERE, "launch_rules_driver.cpp"), "-o", out], check=True)
    return out


def ask(*queries):
    """Each query is (name, int, ...); returns one list of ints per query."""
    text = "".join(" ".join(str(v) for v in q) + "\n" for q in queries)
    r = subprocess.run([_driver()], input=text, text=True, stdout=subprocess.PIPE, check=True)
    return [[int(v) for v in line.split()] for line in r.stdout.splitlines()]
