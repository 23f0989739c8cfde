"""The host's wait for the stage report of Algorithm 1, with the three HIP calls it makes replaced: compiled for the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdint>
#include <cstdio>
typedef void* hipStream_t;
enum hipError_t { hipSuccess, hipErrorNotReady, hipErrorUnknown };
static int32_t word;
static int queries, busy_for, lands_at;
static hipError_t last, after;
// keeps its not-ready answer as the last error, as a runtime may
static hipError_t hipStreamQuery(hipStream_t) {
  ++queries;
  if (queries == lands_at) word = 7;
  const hipError_t e = queries <= busy_for ? hipErrorNotReady : after;
  if (e != hipSuccess) last = e;
  return e;
}
static hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
#include "stage_report.h"
static int failures;
static void expect(const char* what, int busy, int lands, hipError_t then, int start, bool landed, hipError_t left) {
  word = start; queries = 0; busy_for = busy; lands_at = lands; after = then; last = hipSuccess;
  const bool got = adac::report_landed(&word, 7, nullptr);
  if (got != landed || last != left) { std::printf("%s: landed %d, error left %d\n", what, got, last); ++failures; }
}
int main() {
  expect("there at once", 0, 0, hipSuccess, 7, true, hipSuccess);
  expect("lands while the stream is busy", 5, 3, hipSuccess, 6, true, hipSuccess);
  expect("lands with the stream's last kernel", 2, 3, hipSuccess, 6, true, hipSuccess);
  expect("the stream runs dry", 4, 0, hipSuccess, 6, false, hipSuccess);
  expect("the stream fails", 4, 0, hipErrorUnknown, 6, false, hipErrorUnknown);
  return failures;
}
"""


def test_wait_ends_with_the_report_or_a_dry_stream_and_leaves_no_error(tmp_path):
    src, exe = tmp_path / "wait.cpp", tmp_path / "wait"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2604_18348_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    out = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
