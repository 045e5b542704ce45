"""How many frames a dependency-driven launch covers (csrc/sr_internal.h), compiled for the host."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "sr_internal.h"
#define CHECK(c, ...) do { if (!(c)) { std::printf(__VA_ARGS__); std::printf("  (%s)\n", #c); std::exit(1); } } while (0)
int main() {
  // what the caller asks for, up to what an entry of the order holds
  for (int wanted = 1; wanted <= 1024; ++wanted)
    for (int items : {1, 8, 500, 30000}) CHECK(sr_flow_frames(wanted, items) == (wanted < 255 ? wanted : 255), "%d wanted, %d items", wanted, items);
  // unasked: 64 frames, fewer of frames of very many items, but never fewer than eight that fit a grid
  CHECK(sr_flow_frames(0, 500) == 64, "500 items");
  CHECK(sr_flow_frames(0, 65536) == 64, "65536 items");
  CHECK(sr_flow_frames(0, 300000) == 13, "300000 items");
  CHECK(sr_flow_frames(0, 600000) == 8, "600000 items");
  CHECK(sr_flow_frames(0, 1 << 20) == 8, "2^20 items");
  for (int wanted : {0, 1, 8, 64, 255, 1024})
    for (long long items = 1; items < ((long long)1 << 31); items = items * 3 / 2 + 1) {
      const int n = sr_flow_frames(wanted, items);
      CHECK(n >= 0 && n <= 255, "%d frames", n);
      CHECK(n * items <= ((long long)1 << 23), "a grid of %lld workgroups", n * items);
      CHECK(n == 0 || items < (1 << 24), "%lld items", items);
    }
  std::printf("ok\n");
}
"""


def test_frames_of_a_dependency_driven_launch(tmp_path):
    src, exe = tmp_path / "flow.cpp", tmp_path / "flow"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=undefined", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I", os.path.join(ROOT, "paper_1806_04965_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr
