"""staging.h on the host: compiled with g++ against a few stand-ins for the HIP
calls it makes (copies that take place at once, and are counted), so that no GPU
is needed.  Checks which copies go through the ring, that every byte arrives,
and that an error ends a copy."""
import shutil
import subprocess

import pytest

from paper_2509_25840_amd import build as hip_build

STUB = r"""
#pragma once
#include <cstddef>
#include <cstdlib>
#include <cstring>
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorOther = 2 };
enum { hipMemcpyHostToDevice, hipMemcpyDeviceToHost };
enum { hipHostMallocDefault = 0, hipEventDisableTiming = 2 };
enum hipMemoryType { hipMemoryTypeUnregistered = 0, hipMemoryTypeHost = 1, hipMemoryTypeDevice = 2, hipMemoryTypeManaged = 3 };
struct hipPointerAttribute_t { hipMemoryType type; };
typedef void *hipStream_t;
typedef void *hipEvent_t;
struct Fake {
  int copies = 0, pinned = 0, queries = 0, fail_at = -1;
  size_t largest = 0;
  hipError_t last = hipSuccess;
  const void *known = nullptr;      // an array with attributes of `type`
  hipMemoryType type = hipMemoryTypeHost;
  bool unknown_is_error = false;    // how other arrays are answered
};
extern Fake fake;
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int, hipStream_t) {
  if (fake.copies++ == fake.fail_at) return hipErrorOther;
  if (n > fake.largest) fake.largest = n;
  std::memcpy(d, s, n);
  return hipSuccess;
}
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned) { ++fake.pinned; *p = std::malloc(n); return hipSuccess; }
inline hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = nullptr; return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipGetLastError() { const hipError_t e = fake.last; fake.last = hipSuccess; return e; }
inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  ++fake.queries;
  if (p == fake.known) { a->type = fake.type; return hipSuccess; }
  if (fake.unknown_is_error) { fake.last = hipErrorInvalidValue; return hipErrorInvalidValue; }
  a->type = hipMemoryTypeUnregistered;
  return hipSuccess;
}
"""

MAIN = r"""
#include <cstdio>
#include <vector>
#include "staging.h"
Fake fake;
int main() {
  using chfpe::Staging;
  const size_t n = 70000001;
  std::vector<char> a(n), b(n), c(n);
  for (size_t i = 0; i < n; ++i) a[i] = (char)(i * 2654435761u >> 13);
  auto report = [&](const char *what, hipError_t e) {
    std::printf("%s rc=%d copies=%d largest=%zu pinned=%d last=%d same=%d\n", what, e, fake.copies, fake.largest,
                fake.pinned, fake.last, (int)(a == c));
    std::fflush(stdout);
  };
  auto both = [&](const char *what, size_t bytes) {
    Staging s;
    std::fill(c.begin(), c.end(), 0);
    hipError_t e = s.in(b.data(), a.data(), bytes, nullptr);
    if (!e) e = s.out(c.data(), b.data(), bytes, nullptr);
    report(what, e);
  };
  both("pageable", n);
  fake = Fake{}; fake.unknown_is_error = true;
  both("pageable-error", n);
  for (hipMemoryType t : {hipMemoryTypeHost, hipMemoryTypeManaged}) {
    Staging s;
    fake = Fake{}; fake.known = a.data(); fake.type = t;
    report("in", s.in(b.data(), a.data(), n, nullptr));
    fake = Fake{}; fake.known = c.data(); fake.type = t;
    report("out", s.out(c.data(), b.data(), n, nullptr));
  }
  for (int at : {0, 5, 20}) {
    fake = Fake{}; fake.fail_at = at;
    Staging s;
    report("fail-in", s.in(b.data(), a.data(), n, nullptr));
    fake = Fake{}; fake.fail_at = at;
    Staging t;
    report("fail-out", t.out(c.data(), b.data(), n, nullptr));
  }
}
"""


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("staging")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STUB)
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-I", str(d), "-I", hip_build.CSRC, str(d / "main.cpp"), "-o",
                    str(d / "main")], check=True)
    out = subprocess.run([str(d / "main")], check=True, capture_output=True, text=True, timeout=60).stdout
    return [(ln.split()[0], dict(f.split("=") for f in ln.split()[1:])) for ln in out.splitlines()]


def of(lines, what):
    return [f for name, f in lines if name == what]


def test_pageable_arrays_go_through_the_ring(lines):
    for what in ("pageable", "pageable-error"):
        (f,) = of(lines, what)
        assert f["rc"] == "0" and f["same"] == "1" and f["pinned"] == "1"
        assert int(f["copies"]) == 2 * 34 and int(f["largest"]) == 2 << 20
        assert f["last"] == "0"  # the query leaves no error for the next launch check


def test_arrays_the_link_reaches_are_copied_directly(lines):
    for f in of(lines, "in") + of(lines, "out"):
        assert f["rc"] == "0" and f["same"] == "1"
        assert f["copies"] == "1" and f["largest"] == "70000001" and f["pinned"] == "0"


def test_an_error_ends_the_copy(lines):
    for f in of(lines, "fail-in") + of(lines, "fail-out"):
        assert f["rc"] == "2"
