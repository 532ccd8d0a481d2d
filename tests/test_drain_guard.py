"""A scope whose kernels write the context's pinned buffer waits for the stream
when an exception leaves it, and only then (host code, with the stream's wait
replaced by a counter)."""
import subprocess

from paper_2411_05869_amd import build

PROGRAM = r"""
#include "internal.hpp"
static int waits = 0;
extern "C" hipError_t hipStreamSynchronize(hipStream_t s) {
  waits += s == reinterpret_cast<hipStream_t>(64);
  return hipSuccess;
}
static void scope(gp_ctx* c, bool fail) {
  const gps::DrainGuard drain(c);
  if (fail) throw gps::Error{GP_EDEVICE, "a launch failed"};
}
struct DuringUnwinding {  // a scope that ends well while another exception passes
  gp_ctx* c;
  ~DuringUnwinding() { scope(c, false); }
};
int main() {
  gp_ctx c;
  c.stream = reinterpret_cast<hipStream_t>(64);
  auto waited = [&](auto&& f) {
    waits = 0;
    try { f(); } catch (const gps::Error&) {}
    return waits;
  };
  if (waited([&] { scope(&c, false); }) != 0) return 1;
  if (waited([&] { scope(&c, true); }) != 1) return 2;
  if (waited([&] { scope(nullptr, true); }) != 0) return 3;
  if (waited([&] { DuringUnwinding d{&c}; throw gps::Error{GP_EDEVICE, ""}; }) != 0) return 4;
  return 0;
}
"""


def test_waits_on_an_exception_only(tmp_path):
    src, exe = tmp_path / "guard.cpp", tmp_path / "guard"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "-std=c++17", f"-I{build.CSRC}", f"-I{build.ROOT}/include", str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    assert subprocess.run([str(exe)]).returncode == 0
