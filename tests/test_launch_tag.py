"""The tags of the one-launch step's words, compiled for the CPU into a model of
launches whose workgroup 0 may give up waiting: it never takes a word of an earlier
launch, whenever the workgroups that write the words read the number of launches and
write.  With the rule `tag = launches + 1, then launches = tag` also after giving up
it does: the model finds that."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_00539_amd", "csrc")

PROGRAM = """
#include <cstdio>
#include <cstdlib>
#include "launch_tag.h"
struct Kept {
  static uint32_t tag(uint32_t l) { return gnmr::tag_of(l); }
  static uint32_t after(uint32_t t, bool all) { return gnmr::launches_after(t, all); }
  static bool none(uint32_t t) { return gnmr::words_lost(t); }
};
struct Plain {
  static uint32_t tag(uint32_t l) { return l + 1; }
  static uint32_t after(uint32_t t, bool) { return t; }
  static bool none(uint32_t) { return false; }
};
constexpr int kItems = 2, kLaunches = 4;
struct State {
  uint32_t launches, word_tag[kItems];
  int word_of[kItems];  // the launch that wrote the word
};
long stale = 0, lost = 0, whole = 0;
// Each item of a launch: 0 reads and writes in time; 1 reads before workgroup 0 ends
// and writes after; 2 reads and writes after.
template <typename Rule>
void launch(State s, int n, bool was_lost) {
  if (n == kLaunches) return;
  for (int when = 0; when < 9; ++when) {
    const int of[kItems] = {when % 3, when / 3};
    State e = s;
    const uint32_t tag = Rule::tag(s.launches);
    auto write = [&](int i, uint32_t t) {
      if (Rule::none(t)) return;
      e.word_tag[i] = t;
      e.word_of[i] = n;
    };
    for (int i = 0; i < kItems; ++i)
      if (of[i] == 0) write(i, tag);
    int here = 0;
    for (int i = 0; i < kItems; ++i)
      if (e.word_tag[i] == tag) {
        ++here;
        if (e.word_of[i] != n) ++stale;
      }
    if (was_lost && here) ++stale;
    (here == kItems ? whole : lost) += 1;
    e.launches = Rule::after(tag, here == kItems);
    for (int i = 0; i < kItems; ++i)
      if (of[i] > 0) write(i, of[i] == 1 ? tag : Rule::tag(e.launches));
    launch<Rule>(e, n + 1, was_lost || here != kItems);
  }
}
int main(int argc, char** argv) {
  const uint32_t start = uint32_t(strtoul(argv[2], nullptr, 10));
  // (the words as the launches before left them; the largest tag leaves 0)
  const uint32_t last = start == 0 && argc > 3 ? gnmr::kWordsLost - 1 : start;
  State s{start, {last, last}, {-1, -1}};
  if (argv[1][0] == 'k') launch<Kept>(s, 0, false);
  else launch<Plain>(s, 0, false);
  printf("%ld %ld %ld\\n", stale, lost, whole);
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("tags")
    (d / "tags.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, "-o",
                    str(d / "tags"), str(d / "tags.cpp")], check=True)
    return lambda *a: tuple(map(int, subprocess.run(
        [str(d / "tags"), *map(str, a)], check=True, capture_output=True, text=True,
        timeout=60).stdout.split()))


# a new context, in use, around the largest tag (2^31 - 1) and after it
@pytest.mark.parametrize("launches", [(0,), (1,), (12345,), (2**31 - 5,), (2**31 - 4,),
                                      (2**31 - 3,), (2**31 - 2,), (0, "again")])
def test_no_word_of_an_earlier_launch_is_taken(model, launches):
    stale, lost, whole = model("kept", *launches)
    assert stale == 0 and lost > 0 and whole > 0
    assert model("plain", *launches)[0] > 0
