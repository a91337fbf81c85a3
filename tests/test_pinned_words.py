"""The pool of pinned words that contexts with a tolerance share, on the CPU with stub HIP calls: it keeps
at most 8 words, hands a kept word out before it pins another, and giving a word back neither allocates
(it happens in a destructor under a C entry point) nor depends on the pool's own destruction."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = """
#include <stdlib.h>
typedef int hipError_t;
enum { hipSuccess = 0, hipHostMallocMapped = 2, hipHostMallocPortable = 1 };
extern int pinned, freed;
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) { ++pinned; *p = malloc(n); return hipSuccess; }
inline hipError_t hipHostFree(void* p) { ++freed; free(p); return hipSuccess; }
"""
PROGRAM = """
#include <new>
#include <set>
#include <thread>
#include <type_traits>
#include "kbe_pinned.hpp"
int pinned, freed;
static bool no_memory;
void* operator new(size_t n) { if (no_memory) throw std::bad_alloc(); return malloc(n); }
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
static_assert(std::is_trivially_destructible<kbe::PinnedWords>::value, "contexts may outlive it");
static kbe::PinnedWords words;
struct Context { double* w = nullptr; ~Context() { words.give_back(w); } };
int main() {
  { Context none; }
  Context* c = new Context[10];
  std::set<double*> distinct;
  for (int i = 0; i < 10; ++i) {
    if (words.take(&c[i].w) != hipSuccess) return 1;
    distinct.insert(c[i].w);
  }
  if (distinct.size() != 10 || pinned != 10) return 2;
  no_memory = true;
  for (int i = 0; i < 10; ++i) { c[i].~Context(); c[i].w = nullptr; }
  if (freed != 2) return 3;
  for (int i = 0; i < 9; ++i) if (words.take(&c[i].w) != hipSuccess) return 4;
  if (pinned != 11) return 5;
  no_memory = false;
  std::thread t[4];
  for (auto& x : t) x = std::thread([] { for (int i = 0; i < 20000; ++i) { Context k; words.take(&k.w); *k.w = i; if (*k.w != i) abort(); } });
  for (auto& x : t) x.join();
  return pinned - freed > 9 + 8 ? 6 : 0;
}
"""


def test_pool(tmp_path):
    os.mkdir(tmp_path / "hip")
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    (tmp_path / "main.cpp").write_text(PROGRAM)
    exe = str(tmp_path / "pool")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", str(tmp_path), "-I",
                    os.path.join(ROOT, "paper_2505_19467_amd", "csrc"), str(tmp_path / "main.cpp"), "-o", exe], check=True)
    assert subprocess.run([exe], timeout=60).returncode == 0
