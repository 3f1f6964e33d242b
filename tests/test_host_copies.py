"""Large host batches: csrc/host_copy.h compiled for the host against a HIP runtime that keeps account.  Every column is copied once and
in time, the extra streams belong to the context's device, are made only once they are worth it, and are given back."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_04478_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <chrono>
#include <cstddef>
#include <cstdint>
#include <map>
#include <mutex>
#include <set>
#include <thread>
#include <vector>
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1 };
enum hipMemcpyKind { hipMemcpyHostToDevice };
constexpr unsigned hipStreamNonBlocking = 1;
struct FakeStream { int device; };
typedef FakeStream* hipStream_t;
namespace fake {
inline std::mutex m;
inline thread_local int current = 0;
inline std::set<FakeStream*> made;
inline int fail_create_after = -1, created = 0, failing_column = -1, sync_fails = 0;
inline std::map<const void*, std::vector<hipStream_t>> copied;       // source -> streams that it went over
inline std::map<hipStream_t, intptr_t> pending;                       // batch that the stream has copies of
inline bool mixed = false;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { *d = fake::current; return hipSuccess; }
inline hipError_t hipSetDevice(int d) { fake::current = d; return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  std::lock_guard<std::mutex> l(fake::m);
  if (fake::fail_create_after >= 0 && (int)fake::made.size() >= fake::fail_create_after) return hipErrorInvalidValue;
  ++fake::created;
  *s = new FakeStream{fake::current};
  fake::made.insert(*s);
  return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s) {
  std::lock_guard<std::mutex> l(fake::m);
  if (!fake::made.erase(s)) return hipErrorInvalidValue;
  delete s;
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s) {
  std::lock_guard<std::mutex> l(fake::m);
  fake::pending.erase(s);
  return fake::sync_fails ? hipErrorInvalidValue : hipSuccess;
}
inline hipError_t hipMemcpyAsync(void*, const void* src, size_t, hipMemcpyKind, hipStream_t s) {
  // the calling thread is slow, so that the helpers, where there are any, get their share
  if (!s) { bool help; { std::lock_guard<std::mutex> l(fake::m); help = !fake::made.empty(); } std::this_thread::sleep_for(std::chrono::milliseconds(help ? 50 : 0)); }
  std::lock_guard<std::mutex> l(fake::m);
  if ((intptr_t)src == fake::failing_column) return hipErrorInvalidValue;
  if (s && s->device != fake::current) return hipErrorInvalidValue;
  fake::copied[src].push_back(s);
  if (s) { const intptr_t b = (intptr_t)src / 1000; fake::mixed |= fake::pending.emplace(s, b).first->second != b; }
  return hipSuccess;
}
"""

PROGRAM = r"""
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include "host_copy.h"
using namespace ccld;
#define CHECK(x) do { if (!(x)) { std::printf("%s: line %d: %s\n", what, __LINE__, #x); std::exit(1); } } while (0)
static const char* what = "";
static CopyStreams pool;
// a batch of seven columns; returns whether it went over other streams than the caller's too
static bool batch(uint64_t mb, int d, uint64_t& earned, hipError_t want = hipSuccess, uintptr_t base = 1000) {
  { std::lock_guard<std::mutex> l(fake::m); for (int k = 0; k < 7; ++k) fake::copied.erase((void*)(base + k)); }
  HostCopy c[7];
  uint64_t left = mb << 20;
  for (int k = 0; k < 7; ++k) { c[k] = {nullptr, (void*)(base + k), k < 6 ? (mb << 20) / 7 : left}; left -= c[k].bytes; }
  const hipError_t e = copy_from_host(pool, d, earned, nullptr, c, 7);
  CHECK(e == want);
  std::lock_guard<std::mutex> l(fake::m);
  std::set<hipStream_t> over;
  for (int k = 0; k < 7 && want == hipSuccess; ++k) {
    const auto& v = fake::copied[(void*)(base + k)];
    CHECK(v.size() == 1);                                  // every column once
    if (v[0]) { CHECK(fake::made.count(v[0]) && v[0]->device == d && !fake::pending.count(v[0])); over.insert(v[0]); }
  }
  return !over.empty();
}
static void earn(int d, uint64_t& earned) {
  for (uint64_t mb = 0; mb < COPY_EARN_BYTES >> 20; mb += 256) CHECK(!batch(256, d, earned) && fake::made.empty());
}
int main() {
  uint64_t a = 0, b = 0, c = 0;
  what = "batches below the line and first large ones are copied alone";
  pool.join(0); pool.join(0);
  for (int i = 0; i < 100; ++i) CHECK(!batch(31, 0, a));
  CHECK(a == 0);
  earn(0, a);
  what = "streams once they are worth it, on the context's device";
  fake::current = 3;
  CHECK(!batch(31, 0, a) && fake::made.empty());
  CHECK(batch(40, 0, a) && fake::made.size() == 2);
  for (FakeStream* s : fake::made) CHECK(s->device == 0);
  CHECK(fake::current == 3);                               // the caller's device is left as it was
  fake::current = 0;
  what = "kept, and used by other contexts of the device at once";
  CHECK(batch(40, 0, a) && batch(40, 0, b) && b == 0 && fake::created == 2);
  what = "not by those of another device";
  pool.join(1);
  fake::current = 1;
  CHECK(!batch(40, 1, c) && c == 40 << 20 && fake::created == 2);
  pool.leave(1);
  fake::current = 0;
  what = "two contexts in two threads";
  for (int i = 0; i < 5; ++i) {
    bool n[2];
    std::thread t([&] { fake::current = 0; n[0] = batch(40, 0, b, hipSuccess, 2000); });
    n[1] = batch(40, 0, a, hipSuccess, 3000);
    t.join();
    CHECK((n[0] || n[1]) && fake::created == 2 && !fake::mixed);
  }
  what = "a column that fails, wherever it is copied";
  for (int k = 0; k < 7; ++k) {
    fake::failing_column = 1000 + k;
    batch(40, 0, a, hipErrorInvalidValue);
    fake::failing_column = -1;
    CHECK(batch(40, 0, a));
  }
  what = "a staging area that cannot be waited for";
  fake::sync_fails = 1;
  batch(40, 0, a, hipErrorInvalidValue);
  fake::sync_fails = 0;
  CHECK(batch(40, 0, a));
  what = "given back with the last context";
  pool.leave(0);
  CHECK(fake::made.size() == 2);
  pool.leave(0);
  CHECK(fake::made.empty());
  what = "made again for later contexts, or done without";
  for (int fail : {0, 1}) {
    pool.join(0);
    a = 0;
    fake::created = 0;
    earn(0, a);
    fake::fail_create_after = fail;
    CHECK(!batch(40, 0, a) && fake::made.empty() && a == 0);
    CHECK(!batch(40, 0, a) && fake::created == fail);          // not tried again in every batch
    fake::fail_create_after = -1;
    a = COPY_EARN_BYTES;
    CHECK(batch(40, 0, a));
    pool.leave(0);
    CHECK(fake::made.empty());
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def account(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_copies")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-Wall", "-I", str(d), "-I", CSRC, "-o", str(d / "main"), str(d / "main.cpp")])
    return d / "main"


def test_account_of_large_host_batches(account):
    run = subprocess.run([str(account)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout
