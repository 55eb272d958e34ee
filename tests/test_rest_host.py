"""Units at rest (device code), compiled for the host from the same source text: a unit that stayed
with some slack counts as at rest only while the degree moved since then could not have used the
slack up (exact fractions), for nearly as long as that holds, and never when it moved, had no slack,
or a comparison of its decision was left open."""
import os
import random
import shutil
import subprocess
from fractions import Fraction as F

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
KERNELS_HPP = os.path.join(HERE, "..", "paper_2608_03695_amd", "csrc", "kernels.hpp")

MAIN = r"""
int main() {
  // per case: slices of the unit, its p*b, degree, counter, slack, moved, open comparison; then
  // counter values to ask about
  int m, moved, open, asked;
  long long pb, k;
  unsigned long long ctr;
  double slack;
  while (scanf("%d %lld %lld %llu %lf %d %d %d", &m, &pb, &k, &ctr, &slack, &moved, &open,
               &asked) == 8) {
    int64_t counters[4] = {0, 0, 0, 0};
    Rest records[1] = {};
    SolveDev sd{};
    sd.rest = records;
    sd.ctr = counters;
    sd.nsl = 2;
    UnitCtx u{};
    u.v = 0;
    u.j = 1;
    u.m = m;
    u.gs0 = 1;
    u.k0 = k;
    u.pb = pb;
    const int which = m <= 1 ? 1 : 3;
    counters[which] = (int64_t)ctr;
    settle(sd, u, moved ? 7u : kNone, slack, (double)k, open != 0);
    for (int i = 0; i < asked; i++) {
      unsigned long long now;
      if (scanf("%llu", &now) != 1) return 1;
      counters[which] = (int64_t)now;
      printf("%d ", at_rest(sd, 0) ? 1 : 0);
    }
    printf("\n");
  }
  return 0;
}
"""


def _piece(src, start):
    """The text from `start` to the end of its braces."""
    a = src.index(start)
    depth, i = 0, src.index("{", a)
    while True:
        depth += {"{": 1, "}": -1}.get(src[i], 0)
        i += 1
        if depth == 0:
            break
    return src[a:i] + (";\n" if start.startswith("struct") else "\n")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    src = open(KERNELS_HPP).read()
    d = tmp_path_factory.mktemp("rest")
    text = ("#include <cstdint>\n#include <cstdio>\n#define __device__\n"
            "constexpr uint32_t kNone = 0xffffffffu;\nstruct SliceRecip;\n")
    for start in ("struct SolveDev {", "struct Rest {", "__device__ inline bool at_rest(",
                  "struct UnitCtx {", "__device__ inline void settle("):
        text += _piece(src, start)
    (d / "rest.cpp").write_text(text + MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", str(d / "rest.cpp"), "-o", str(d / "rest")],
                   check=True)

    def run(cases):
        """cases: (m, pb, k, ctr, slack, moved, open, [counter values]) -> at rest, per value"""
        text = "".join(f"{m} {pb} {k} {c} {s!r} {mv} {op} {len(at)} {' '.join(map(str, at))}\n"
                       for m, pb, k, c, s, mv, op, at in cases)
        out = subprocess.run([str(d / "rest")], input=text, capture_output=True, text=True,
                             check=True).stdout.split("\n")
        return [[x == "1" for x in line.split()] for line in out[:len(cases)]]
    return run


def _last(m, pb, k, ctr, slack):
    """The largest counter value at which the unit still may be at rest."""
    unit = 1 if m <= 1 else F(1, 2 ** 32)   # degree, or degree over slice totals
    return ctr + int(F(slack) / (2 * pb * k * unit))


def _cases(rnd, n):
    out = []
    for _ in range(n):
        m = rnd.choice([1, 1, 2, 40])
        pb, k = rnd.randint(1, 2 ** rnd.randint(1, 31)), rnd.randint(1, 2 ** rnd.randint(1, 30))
        top = min(62, 60 if m <= 1 else 30)
        slack = float(2 * pb * k) * rnd.random() * 2.0 ** rnd.randint(-3, top) * (m <= 1 or 2.0 ** -32)
        ctr = rnd.choice([0, rnd.getrandbits(20), rnd.getrandbits(40)])
        out.append((m, pb, k, ctr, slack))
    return out


def test_rest_ends_before_the_slack_is_used_up(ask):
    rnd = random.Random(5)
    cases, want = [], []
    for m, pb, k, ctr, slack in _cases(rnd, 3000):
        last = _last(m, pb, k, ctr, slack)
        near = ctr + int((last - ctr) * (1 - F(1, 2 ** 28)))
        cases.append((m, pb, k, ctr, slack, 0, 0, [last + 1, last + 1000, max(near - 1, ctr)]))
        want.append([False, False, last > ctr])
    for case, got, exp in zip(cases, ask(cases), want):
        assert got[:2] == exp[:2], case
        assert got[2] or not exp[2], case


def test_no_rest_without_a_settled_decision(ask):
    rnd = random.Random(6)
    cases = []
    for m, pb, k, ctr, slack in _cases(rnd, 300):
        cases += [(m, pb, k, ctr, slack, 1, 0, [ctr]), (m, pb, k, ctr, -slack - 1.0, 0, 0, [ctr]),
                  (m, pb, k, ctr, slack, 0, 1, [ctr])]
    assert not any(any(got) for got in ask(cases))
    # no null term: nothing that moves elsewhere matters
    free = [(m, pb, k, 5, s, 0, 0, [5, 10 ** 17]) for m in (0, 1, 2) for pb, k in ((0, 3), (2, 0))
            for s in (0.0, 1.0)]
    assert all(all(got) for got in ask(free))


@pytest.mark.parametrize("ctr", [2 ** 63 - 2 ** 40, 2 ** 63 - 1, 2 ** 63, 2 ** 64 - 2 ** 41])
def test_counters_beyond_63_bits_end_rest(ask, ctr):
    """The moved degree of a CPM solve adds up to 2^64 when every copy moves in every sweep."""
    case = (2, 3, 10, ctr, 60.0 * 0.5, 0, 0)          # rests for half a unit of moved degree
    got, = ask([case + ([ctr, ctr + 2 ** 30, ctr + 2 ** 31 + 1, ctr + 2 ** 40],)])
    assert got == [True, True, False, False]
