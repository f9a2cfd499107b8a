"""The bookkeeping of kept device memory (csrc/block_pool.h, plain C++), compiled with the host
compiler: what a request may take, that a full pool makes room by age, and that nothing is lost
or handed out twice."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include "block_pool.h"
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

static char space[1 << 20];
static void* at(size_t i) { return space + i; }

// as the library does it
static bool give(wc::BlockPool& b, void* p, size_t n, std::set<void*>* freed) {
  while (!b.fits(n)) {
    void* old = n > b.limit() ? nullptr : b.oldest(nullptr);
    if (!old) return false;
    freed->insert(old);
  }
  return b.give(p, n);
}

int main() {
  size_t got = 0;
  std::set<void*> freed;
  {
    wc::BlockPool b(1000);
    CHECK(!b.take(1, &got) && !b.oldest(nullptr) && b.bytes() == 0);
    CHECK(b.fits(1000) && !b.fits(1001) && !b.fits(~size_t(0)));
    CHECK(!give(b, at(0), 1001, &freed) && freed.empty() && b.bytes() == 0);
    CHECK(give(b, at(1), 1000, &freed) && !b.fits(1));
    CHECK(b.take(1000, &got) == at(1) && got == 1000 && b.bytes() == 0);
  }
  {  // the size window: at least the request, at most a quarter and a page more
    wc::BlockPool b(1 << 30);
    CHECK(b.give(at(1), 125000 + 4096));
    CHECK(!b.take(125000 + 4097, &got));
    CHECK(!b.take(99999, &got));
    CHECK(b.take(100000, &got) == at(1) && got == 129096);
    CHECK(b.give(at(1), 9000) && b.give(at(2), 8000) && b.give(at(3), 8500));
    CHECK(b.take(8100, &got) == at(3) && got == 8500);
  }
  {  // one large block, then smaller ones: the large one goes, the small ones stay
    wc::BlockPool b(1000);
    CHECK(give(b, at(0), 900, &freed));
    for (int i = 1; i <= 5; ++i) CHECK(give(b, at(i), 200, &freed));
    CHECK(freed.size() == 1 && freed.count(at(0)) && b.bytes() == 1000);
    CHECK(give(b, at(6), 300, &freed));  // the two oldest of them
    CHECK(freed.size() == 3 && freed.count(at(1)) && freed.count(at(2)) && b.bytes() == 900);
    for (int i = 3; i <= 5; ++i) CHECK(b.take(200, &got) == at(i) && got == 200);
    CHECK(b.oldest(&got) == at(6) && got == 300 && b.bytes() == 0 && !b.oldest(nullptr));
  }
  {  // a taken block given again is the youngest
    wc::BlockPool b(300);
    CHECK(b.give(at(1), 100) && b.give(at(2), 110) && b.give(at(3), 90));
    CHECK(b.take(100, &got) == at(1));
    CHECK(b.give(at(1), 100));
    freed.clear();
    CHECK(give(b, at(4), 50, &freed) && freed.size() == 1 && freed.count(at(2)));
  }
  // random gives and takes: every block is in exactly one place, the sum is right
  wc::BlockPool b(5000);
  std::set<void*> kept, outside;
  size_t size[64], sum = 0;
  for (int i = 0; i < 64; ++i) {
    size[i] = 1 + std::rand() % 700;
    outside.insert(at(i));
  }
  for (int step = 0; step < 200000; ++step) {
    if (std::rand() % 2) {
      if (outside.empty()) continue;
      void* p = *outside.begin();
      freed.clear();
      CHECK(give(b, p, size[(char*)p - space], &freed));
      outside.erase(p);
      for (void* q : freed) CHECK(kept.erase(q) && outside.insert(q).second);
      CHECK(kept.insert(p).second);
    } else {
      const size_t want = 1 + std::rand() % 700;
      void* p = b.take(want, &got);
      size_t best = 0;
      for (void* q : kept) {
        const size_t n = size[(char*)q - space];
        if (n >= want && n <= want + want / 4 + 4096 && (!best || n < best)) best = n;
      }
      CHECK(p ? got == best && size[(char*)p - space] == got : !best);
      if (p) CHECK(kept.erase(p) && outside.insert(p).second);
    }
    sum = 0;
    for (void* q : kept) sum += size[(char*)q - space];
    CHECK(sum == b.bytes() && sum <= 5000);
  }
  return 0;
}
"""


def test_block_pool(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "pool.cpp", tmp_path / "pool"
    src.write_text(PROGRAM)
    cc = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I",
                         os.path.join(ROOT, "paper_1109_4279_amd", "csrc"), str(src), "-o", str(exe)],
                        capture_output=True, text=True, timeout=120)
    assert cc.returncode == 0, cc.stderr
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout
