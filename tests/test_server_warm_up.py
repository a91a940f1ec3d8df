"""The serving loop's warm-up batches launch every kernel that a later batch may launch (no GPU needed): the rule
that picks a batch's kernels, walked over every batch size and beam."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2411_12229_amd")
LIB = os.path.join(PKG, "libqg.so")

SOURCE = r"""
#include <cstdio>
#include "qg_internal.h"
int main() {
  const int shapes[][2] = {{96, 32}, {96, 64}, {128, 32}, {128, 64}, {768, 32}, {768, 64}, {960, 32}, {960, 64}};
  const int bounds[][2] = {{1, 1}, {64, 64}, {65, 129}, {512, 256}, {3072, 512}, {3073, 257}, {3500, 512}, {8192, 512},
                           {9000, 1536}, {8192, 2048}};
  int bad = 0;
  for (auto& sh : shapes)
    for (auto& b : bounds)
      for (int stop = 0; stop < 2; ++stop)
        for (int form = 0; form < 3; ++form) {  // registers, beams in LDS, int32 table entries
          const qgi::Setting s{sh[0], sh[1], 1000000, form != 1, form == 2};
          const int mode = stop ? 4 : 3;
          const auto warm = qgi::warm_batches(s, b[0], b[1], stop);
          std::vector<qgi::Route> loaded;
          for (auto& w : warm) {
            if (w.nq < 1 || w.nq > b[0] || w.ef < 1 || w.ef > b[1]) ++bad;
            loaded.push_back(qgi::search_route(s, w.nq, w.ef, mode, 0, true));
          }
          if (warm.size() > 16) ++bad;
          for (int ef = 1; ef <= b[1]; ++ef)
            for (int64_t n = 1; n <= b[0]; n = n < 4096 && (ef % 64 == 1 || n < 80) ? n + 1 : n + 61) {
              const qgi::Route r = qgi::search_route(s, n, ef, mode, 0, true);
              bool tiles = false, search = false;
              for (auto& o : loaded) tiles |= o.tiles == r.tiles, search |= o.same_search(r);
              if (!(tiles && search) && bad++ < 10)
                std::printf("%d x %d stop %d form %d max_batch %d ef_max %d: not loaded: %lld queries, ef %d\n", sh[0], sh[1], stop,
                            form, b[0], b[1], (long long)n, ef);
            }
        }
  std::printf("%d\n", bad);
  return bad != 0;
}
"""


def test_every_route_is_loaded(tmp_path):
    if not os.path.exists(LIB):
        from paper_2411_12229_amd import build
        build.build()
    src, exe = tmp_path / "warm.cpp", str(tmp_path / "warm")
    src.write_text(SOURCE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cc = subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                         "-I", os.path.join(PKG, "csrc"), "-I", os.path.join(rocm, "include"), str(src), LIB,
                         f"-Wl,-rpath,{PKG}", f"-Wl,-rpath,{rocm}/lib", f"-Wl,-rpath-link,{rocm}/lib", "-o", exe],
                        capture_output=True, text=True)
    assert cc.returncode == 0, cc.stderr
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
