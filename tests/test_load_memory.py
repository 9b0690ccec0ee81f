"""Host memory that runs out while a network is created or loaded: each allocation of the call fails in turn, on
the calling thread or on one that packs layers, and the call answers SDNN_ENOMEM; no exception leaves the
library and the process goes on. A small program replaces operator new for the library it loads.
Without a GPU a load that gets all its memory ends at the first device call (SDNN_EDEVICE)."""
import os
import shutil
import subprocess

import pytest

from paper_1909_05631_amd import sdnn

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <dlfcn.h>
#include <new>
#include <vector>
#include "sdnn.h"

static std::atomic<long> left{-1};  // allocations until the one that fails (-1: none does)
static std::atomic<bool> hit{false};

void *operator new(std::size_t n) {
  if (left.load() >= 0 && left.fetch_sub(1) == 0) {
    hit = true;
    throw std::bad_alloc();
  }
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void *operator new(std::size_t n, const std::nothrow_t &) noexcept {
  if (left.load() >= 0 && left.fetch_sub(1) == 0) {
    hit = true;
    return nullptr;
  }
  return std::malloc(n ? n : 1);
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }
void operator delete(void *p, const std::nothrow_t &) noexcept { std::free(p); }

int main(int argc, char **argv) {
  void *so = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
  if (!so) { std::fprintf(stderr, "%s\n", dlerror()); return 2; }
  auto create = reinterpret_cast<decltype(&sdnn_create)>(dlsym(so, "sdnn_create"));
  auto load = reinterpret_cast<decltype(&sdnn_load_layers)>(dlsym(so, "sdnn_load_layers"));
  auto destroy = reinterpret_cast<decltype(&sdnn_destroy)>(dlsym(so, "sdnn_destroy"));
  auto error = reinterpret_cast<decltype(&sdnn_last_error)>(dlsym(so, "sdnn_last_error"));
  auto opt = reinterpret_cast<decltype(&sdnn_enable_equal_value_kernels)>(dlsym(so, "sdnn_enable_equal_value_kernels"));
  const int N = std::atoi(argv[2]), L = 5, equal = std::atoi(argv[3]);
  std::vector<int64_t> cp;
  std::vector<int32_t> ri;
  std::vector<float> v, b((size_t)L * N, -0.3f);
  for (int l = 0; l < L; ++l)
    for (int j = 0; j <= N; ++j) {
      cp.push_back((int64_t)ri.size());
      if (j == N) break;
      const int d = equal ? 32 : 1 + (j * 7 + l) % 40;
      for (int s = 0; s < d; ++s) {
        ri.push_back(s * (N / 64) + (j / 4 + l) % (N / 64));
        v.push_back(0.0625f);
      }
    }
  long failed = 0, created = 0;
  for (long k = -1;; ++k) {  // k = -1: the device calls' own start-up, nothing fails
    sdnn_net *net = nullptr;
    hit = false;
    left = k;
    sdnn_status st = create(&net, N, L, 32.0f);
    left = -1;
    if (hit) {
      if (st != SDNN_ENOMEM || net) { std::printf("create: allocation %ld: status %d\n", k, (int)st); return 1; }
      ++created;
      st = create(&net, N, L, 32.0f);
    }
    if (st != SDNN_OK) { std::printf("create: status %d\n", (int)st); return 1; }
    if (equal && opt(net, 1) != SDNN_OK) return 1;
    hit = false;
    left = k;
    st = load(net, 0, L, cp.data(), ri.data(), v.data(), b.data(), nullptr);
    left = -1;
    const bool failed_here = hit;
    // (an allocation may be one that the call does without, as a thread or a message)
    if (st != SDNN_ENOMEM && st != SDNN_EDEVICE && st != SDNN_OK) {
      std::printf("load: allocation %ld: status %d (%s)\n", k, (int)st, error());
      return 1;
    }
    failed += st == SDNN_ENOMEM;
    destroy(net);
    if (k >= 0 && !failed_here) break;
    if (st == SDNN_ENOMEM && !failed_here) return 1;
  }
  std::printf("%ld loads and %ld creations ran out of memory\n", failed, created);
  return failed > 0 && created > 0 ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    if not os.path.exists(sdnn.library_path()):
        from paper_1909_05631_amd import build
        build.build()
    d = tmp_path_factory.mktemp("load_memory")
    src, exe = d / "program.cc", d / "program"
    src.write_text(PROGRAM)
    subprocess.run([gxx, "-O1", "-std=c++17", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", str(exe), str(src),
                    "-ldl"], check=True)
    return str(exe)


@pytest.mark.parametrize("n,equal", [(256, 0), (4224, 0), (4224, 1)])
def test_out_of_host_memory(program, n, equal):
    r = subprocess.run([program, sdnn.library_path(), str(n), str(equal)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, f"exit status {r.returncode}: {r.stdout[-500:]}{r.stderr[-500:]}"
