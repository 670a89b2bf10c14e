"""CPU test of the page-locked slots for status words: built with the host
compiler alone, with an ordinary allocation in place of the page-locked one."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "status_slots.h"
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <thread>
#include <vector>

static int pages = 0;
static void* page(size_t bytes) { ++pages; return std::aligned_alloc(64, bytes); }
static void* none(size_t) { return nullptr; }

int main() {
  using wsr::StatusSlots;
  StatusSlots& s = StatusSlots::process();
  if (s.take(none)) return 1;                       // no memory: no slot, and the next thread may try again
  std::set<void*> seen;
  for (int k = 0; k < 300; ++k) {                   // one after another: the same slot
    std::thread t([&] { void* p = s.take(page); seen.insert(p); s.give(p); });
    t.join();
  }
  if (pages != 1 || seen.size() != 1 || seen.count(nullptr)) return 2;
  for (int round = 0; round < 3; ++round) {         // more at once than there are slots
    std::mutex m;
    std::condition_variable cv;
    std::vector<void*> got;
    std::vector<std::thread> ts;
    const size_t n = StatusSlots::kSlots + 40;
    for (size_t k = 0; k < n; ++k)
      ts.emplace_back([&] {
        void* p = s.take(page);
        std::unique_lock<std::mutex> lock(m);
        got.push_back(p);
        cv.notify_all();
        cv.wait(lock, [&] { return got.size() == n; });
        lock.unlock();
        if (p) s.give(p);
      });
    for (auto& t : ts) t.join();
    std::set<char*> some;
    for (void* p : got)
      if (p) some.insert(static_cast<char*>(p));
    if (some.size() != StatusSlots::kSlots) return 3;
    char* last = nullptr;
    for (char* p : some) {
      if (last && p - last < static_cast<long>(StatusSlots::kSlotBytes)) return 4;
      last = p;
    }
  }
  if (pages != 1) return 5;
  std::puts("ok");
  return 0;
}
"""


def test_threads_share_one_page_and_give_their_slots_back(tmp_path):
    src, exe = tmp_path / "slots.cpp", tmp_path / "slots"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2410_18931_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", csrc, str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.returncode


def test_a_thread_end_makes_no_runtime_call():
    """What runs when a thread ends gives its slot back and calls nothing of HIP."""
    with open(os.path.join(ROOT, "paper_2410_18931_amd", "csrc", "api.hip")) as f:
        text = f.read()
    end = text[text.index("~PinnedFlags()"):]
    end = end[:end.index("DevFlags* get()")]
    assert "give(" in end and "hip" not in end
