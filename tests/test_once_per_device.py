"""The library's host code raises a kernel's LDS limit once on every GPU: csrc/psa_once.h, compiled here by itself."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2503_00392_amd", "csrc")

PROGRAM = r"""
#include "psa_once.h"
#include <stdio.h>
static int calls, answer;
static int work() { ++calls; return answer; }
#define EXPECT(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main() {
    psa::OncePerDevice once, other;
    answer = 700;                                              // the first device refuses: handed on, and asked again
    EXPECT(once(0, work) == 700 && calls == 1);
    EXPECT(once(0, work) == 700 && calls == 2);
    answer = 0;
    EXPECT(once(0, work) == 0 && calls == 3);
    EXPECT(once(0, work) == 0 && calls == 3);                  // done
    EXPECT(once(1, work) == 0 && calls == 4);                  // another GPU is another matter
    EXPECT(once(63, work) == 0 && calls == 5);
    EXPECT(once(63, work) == 0 && once(1, work) == 0 && once(0, work) == 0 && calls == 5);
    answer = 9;
    EXPECT(once(2, work) == 9 && calls == 6);
    EXPECT(once(64, work) == 9 && once(-1, work) == 9 && calls == 8);   // no bit for these: asked every time
    EXPECT(other(0, work) == 9 && calls == 9);                 // another kernel's flag
    return 0;
}
"""


def test_once_per_device_and_failures_are_not_kept(tmp_path):
    src, exe = tmp_path / "once.cpp", tmp_path / "once"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout


def test_no_launcher_keeps_the_answer_of_one_gpu_for_all():
    """hipFuncSetAttribute is called in the one function that goes through OncePerDevice."""
    users = [n for n in sorted(os.listdir(CSRC)) if "hipFuncSetAttribute(" in open(os.path.join(CSRC, n)).read()]
    assert users == ["psa_host.h"]
