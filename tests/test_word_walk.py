"""How a workgroup reads the words that a scale comes from (csrc/words.h), on the host: every word once, and never the history entry that
workgroup 0 of the same launch stores."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_20524_amd", "csrc")
SOURCE = r"""
#include <cstdio>
#include <vector>
#define FOG_DEVICE static inline
#include "words.h"
struct Words {                      // counts the loads of every word
  std::vector<int>* loads;
  float operator[](int i) const { ++loads->at(i); return i + 0.5f; }
};
int main() {
  const int lengths[] = {1, 2, 15, 16, 17, 63, 64, 65, 129, 200};
  for (int n : lengths)
    for (int skip = -1; skip < n; ++skip) {
      std::vector<int> loads(n + 1, 0), taken(n, 0);
      for (int tid = 0; tid < 16; ++tid)
        for_words<16>(Words{&loads}, n, skip, tid, [&](int i, float v) { if (v == i + 0.5f) ++taken.at(i); });
      for (int i = 0; i <= n; ++i) {
        const int want = i < n && i != skip;
        if (loads[i] != want || (i < n && taken[i] != want)) {
          std::printf("n %d, skip %d: word %d loaded %d times, taken %d times\n", n, skip, i, loads[i], i < n ? taken[i] : 0);
          return 1;
        }
      }
    }
  return 0;
}
"""


def test_every_word_once_and_never_the_one_that_is_stored(tmp_path):
    (tmp_path / "walk.cpp").write_text(SOURCE)
    exe = str(tmp_path / "walk")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wno-unknown-pragmas", "-I", CSRC, "-o", exe, str(tmp_path / "walk.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
