"""csrc/plan.h built with the host compiler, for tests of its rules."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WRAPPERS = r"""
#include "plan.h"
extern "C" {
void bin_grid(int64_t nblk, int64_t bands, int64_t nv, int64_t* g) {
  const wsr::GridShape s = wsr::bin_grid(nblk, bands, nv);
  g[0] = s.x; g[1] = s.y; g[2] = s.z;
}
void sum_grid(int64_t slots, int64_t* g) {
  const wsr::GridShape s = wsr::sum_grid(slots);
  g[0] = s.x; g[1] = s.y; g[2] = s.z;
}
int64_t bin_blocks(int64_t n, int64_t chunk) { return wsr::bin_blocks(n, chunk); }
int64_t bin_chunk(int64_t n, int64_t views, int64_t tiles, int64_t largest) {
  return wsr::bin_chunk(n, views, tiles, largest);
}
int64_t bin_matrix_room(int64_t n, int64_t tiles, int64_t largest) { return wsr::bin_matrix_room(n, tiles, largest); }
int64_t bin_tag_pitch(int64_t tiles_x) { return wsr::bin_tag_pitch(tiles_x); }
// pairs of one step of a splat `width` tiles wide that share a tag
int64_t shared_tags(int64_t width, int64_t pitch) {
  int64_t shared = 0;
  for (int64_t first = 0; first < width; ++first) {
    bool seen[wsr::kTags] = {};
    for (int64_t i = first; i < first + 64; ++i) {
      bool& s = seen[wsr::bin_tag(i / width, i % width, pitch)];
      shared += s;
      s = true;
    }
  }
  return shared;
}
int64_t bin_rows(int64_t tiles_x, int64_t max_tiles_y) { return wsr::bin_rows(tiles_x, max_tiles_y); }
int64_t loss_in_strips(int64_t tiles, int64_t strips, int64_t pixels) {
  return wsr::loss_in_strips(tiles, strips, pixels);
}
int64_t few_tiles() { return wsr::kFewTiles; }
int64_t bin_threads() { return wsr::kBinThreads; }
int64_t sum_waves() { return wsr::kSumWaves; }
int64_t sum_per_wave() { return wsr::kSumPerWave; }
}
"""


@functools.lru_cache(None)
def load():
    out = tempfile.mkdtemp(prefix="wsr_plan_")
    src, lib = os.path.join(out, "plan.cpp"), os.path.join(out, "libplan.so")
    with open(src, "w") as f:
        f.write(WRAPPERS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2410_18931_amd", "csrc"), src, "-o", lib], check=True)
    plan = C.CDLL(lib)
    for name in ("bin_blocks", "bin_rows", "shared_tags", "bin_chunk", "bin_matrix_room", "loss_in_strips"):
        getattr(plan, name).argtypes = [C.c_int64] * {"bin_chunk": 4, "bin_matrix_room": 3, "loss_in_strips": 3}.get(name, 2)
        getattr(plan, name).restype = C.c_int64
    for name in ("bin_tag_pitch", "bin_threads", "few_tiles", "sum_waves", "sum_per_wave"):
        getattr(plan, name).restype = C.c_int64
    plan.bin_tag_pitch.argtypes = [C.c_int64]
    plan.bin_grid.argtypes = [C.c_int64, C.c_int64, C.c_int64, C.c_void_p]
    plan.sum_grid.argtypes = [C.c_int64, C.c_void_p]
    return plan


def grid(name, *args):
    g = (C.c_int64 * 3)()
    getattr(load(), name)(*args, g)
    return tuple(g)


def loss_forms(sizes):
    """Form of the loss of each launch of up to 16 views: strips or tiles."""
    out = []
    for k in range(0, len(sizes), 16):
        views = sizes[k:k + 16]
        cut = lambda a, b: sum(-(-w // a) * -(-h // b) for w, h in views)  # noqa: E731
        strips = load().loss_in_strips(cut(16, 16), cut(64, 34), sum(w * h for w, h in views))
        out.append("strips" if strips else "tiles")
    return out
