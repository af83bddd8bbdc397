"""Stream capture of the batched solve (csrc/capture.hpp): an exception between
begin and end leaves no stream capturing and no graph behind.  Host code only,
compiled against stand-ins of the four runtime calls that keep count; that the
batched solve opens its capture through it is read from the source."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_24256_amd", "csrc")

STAND_IN = """
#pragma once
typedef int hipError_t;
typedef struct St { int capturing, graphs; }* hipStream_t;
typedef St* hipGraph_t;
enum { hipSuccess = 0, hipErrorIllegalState = 401, hipStreamCaptureModeThreadLocal = 1 };
inline hipError_t hipStreamBeginCapture(hipStream_t s, int) {
  if (s->capturing) return hipErrorIllegalState;
  s->capturing = 1;
  return hipSuccess;
}
inline hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  if (!s->capturing) return hipErrorIllegalState;
  s->capturing = 0;
  s->graphs += 1;
  *g = s;
  return hipSuccess;
}
inline hipError_t hipGraphDestroy(hipGraph_t g) { g->graphs -= 1; return hipSuccess; }
"""

MAIN = """
#include "capture.hpp"
#include <cstdio>
int main() {
  St s{0, 0};
  for (int turn = 0; turn < 2; ++turn) {  // an exception while capturing, then again on the same stream
    try {
      zr::StreamCapture c;
      if (c.begin(&s) != hipSuccess) return 1;
      throw 7;
    } catch (int) {
    }
    if (s.capturing || s.graphs) return 2;
  }
  {  // the ordinary way: the graph is the caller's
    zr::StreamCapture c;
    hipGraph_t g = nullptr;
    if (c.begin(&s) != hipSuccess || c.end(&g) != hipSuccess || !g) return 3;
  }
  if (s.capturing || s.graphs != 1) return 4;
  {  // a begin that failed is not ended
    St busy{1, 0};
    zr::StreamCapture c;
    if (c.begin(&busy) == hipSuccess) return 5;
    hipGraph_t g = nullptr;
    if (c.end(&g) != hipSuccess || g || !busy.capturing) return 6;
  }
  { zr::StreamCapture unused; }
  puts("ok");
  return 0;
}
"""


def test_exception_ends_the_capture(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STAND_IN)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = tmp_path / "main"
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", str(tmp_path), "-I", CSRC,
                    str(tmp_path / "main.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.returncode


def test_captures_are_opened_through_it():
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".cpp", ".hpp")) and name != "capture.hpp":
            with open(os.path.join(CSRC, name)) as f:
                assert not re.search(r"hipStream(Begin|End)Capture\s*\(", f.read()), name
