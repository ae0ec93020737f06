"""The task order of the k-center in rounds, checked on the host.

`decode_task` in rounds.hip maps a queue position to a task (select, greedy or
fold tile of one request and round) and `tasks_before` says how many of the
request's tasks must be complete for it. The persistent kernel is deadlock-free
and its completion counts are exact only if, in every macro-round, each task of
each request appears exactly once, each task's dependencies (Sec. 3.4: a
round's select needs the previous round's folds; the greedy needs the select;
the folds need the greedy) sit at smaller queue positions, and the count is
that of the dependencies. This test compiles the functions' own text with the
host compiler and checks all three on batches of several shapes.

The queue itself is then run in a model on the host: blocks that take task
indices in turn, wait for a task's dependencies and pass over the tasks of
finished requests, with the task order and the fault check of the kernel's own
text. A batch whose rounds all go well must end every request.
"""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2607_27952_amd", "csrc", "rounds.hip")
HDR = os.path.join(ROOT, "paper_2607_27952_amd", "csrc", "last_internal.h")


def _constant(text, name):
    m = re.search(r"constexpr int %s = (\d+);" % name, text)
    assert m, name
    return int(m.group(1))


def _functions():
    """The text of the queue's functions, for the host compiler."""
    src, fns = open(SRC).read(), "#include <cstdint>\n"
    for head in ("template <typename Ft>\n__device__ __forceinline__ int64_t decode_task",
                 "__device__ __forceinline__ int64_t tasks_a_round", "__device__ __forceinline__ int64_t tasks_before",
                 "__device__ __forceinline__ bool past_last_round"):
        a = src.index(head)
        eol = src.index("\n", a)
        b = eol if src[eol - 1] == "}" else src.index("\n}\n", a) + 2   # a function on one line or several
        fns += src[a:b].replace("__device__ __forceinline__ ", "") + "\n"
    return fns


def _compile(tmp_path_factory, name, text):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp(name)
    cpp, exe = d / f"{name}.cpp", d / name
    cpp.write_text(_functions() + text)
    subprocess.run([gxx, "-O2", "-std=c++17", "-o", str(exe), str(cpp)], check=True)
    return str(exe), _constant(open(HDR).read(), "kRoundFoldRows")


@pytest.fixture(scope="module")
def decoder(tmp_path_factory):
    return _compile(tmp_path_factory, "decode", r"""
#include <cstdio>
#include <vector>
int main() {
  int R, M;
  if (scanf("%d %d", &R, &M) != 2) return 1;
  std::vector<int64_t> ft(R + 1, 0);
  for (int i = 0; i < R; ++i) { long t; if (scanf("%ld", &t) != 1) return 1; ft[i + 1] = ft[i] + t; }
  auto fta = [&](int64_t i) -> int64_t { return ft[i]; };
  int64_t Q = 0;
  for (int i = 0; i < R; ++i) Q += tasks_a_round(ft[i + 1] - ft[i]);
  for (int64_t m = 0; m < M; ++m)
    for (int64_t u = 0; u < Q; ++u) {
      int kind = 0, r = 0, sub = 0;
      const int64_t n = m + decode_task(u, (int64_t)R, fta, kind, r, sub);
      printf("%ld %ld %d %d %ld %d %ld\n", (long)m, (long)u, kind, r, (long)n, sub,
             (long)tasks_before(n, kind, ft[r + 1] - ft[r]));
    }
  return 0;
}
""")


CASES = [
    [85, 183, 295],          # three small requests, both halves
    [150],                   # one request: no second half
    [1, 1],                  # one-token requests
    [0, 512, 0, 700, 3],     # empty requests
    [16384] * 8,             # the video batch
    [32768, 32768],          # the long-video batch
]


@pytest.mark.parametrize("N", CASES + ["ragged128", "ragged33"], ids=str)
def test_decode_order(decoder, N):
    exe, f_rows = decoder
    rng = np.random.default_rng(7)
    if N == "ragged128":
        N = list(rng.integers(256, 16385, 128))
    elif N == "ragged33":
        N = list(rng.integers(0, 3000, 33))
    R, M = len(N), 4
    tiles = [(int(n) + f_rows - 1) // f_rows for n in N]
    out = subprocess.run([exe], input=f"{R} {M} " + " ".join(map(str, tiles)), capture_output=True, text=True,
                         check=True).stdout
    rows = np.array([list(map(int, line.split())) for line in out.split("\n") if line], np.int64)
    Q = sum(2 + t for t in tiles)
    assert len(rows) == M * Q
    RA = (R + 1) // 2
    pos = {}
    for m in range(M):
        got = [tuple(x) for x in rows[rows[:, 0] == m][:, 2:6]]
        assert len(set(got)) == Q, "a task listed twice in one macro-round"
        want = set()
        for r in range(R):
            for kind, count in ((0, 1), (1, 1), (2, tiles[r])):
                n = m - 1 if (kind == 2 and r >= RA) else m   # the second half folds a round behind
                want.update((kind, r, n, s) for s in range(count))
        assert set(got) == want
        for u, key in enumerate(got):
            if key[2] >= 0:
                pos[key] = m * Q + u
    need = {tuple(x[2:6]): x[6] for x in rows}
    for (kind, r, n, s), p in pos.items():
        # every task of the request that must come first: all of round n - 1, and
        # in round n the select before the greedy and both before the folds
        if kind == 0:
            deps = [(2, r, n - 1, t) for t in range(tiles[r])] or [(1, r, n - 1, 0)] if n > 0 else []
        else:
            deps = [(kind - 1, r, n, 0)]
        for dep in deps:
            assert dep in pos and pos[dep] < p, f"{(kind, r, n, s)} listed before its dependency {dep}"
        assert need[kind, r, n, s] == n * (2 + tiles[r]) + kind


# The queue of k_rounds as a discrete-event model: BLOCKS blocks, each taking the
# next index at a cost of DQ, a task of a finished request being passed over at
# once; durations by kind; one round's picks of request r being per[r] at most.
# Prints: requests finished, whether the fault check fired, the largest number
# of macro-rounds the head ran past the oldest unfinished request's round.
MODEL = r"""
#include <algorithm>
#include <cstdio>
#include <queue>
#include <vector>
struct Wait { int block; int64_t need; int kind, sub; int64_t n; };
int main() {
  int R, BLOCKS; double DQ, dur[3];
  if (scanf("%d %d %lf %lf %lf %lf", &R, &BLOCKS, &DQ, dur, dur + 1, dur + 2) != 6) return 1;
  std::vector<int64_t> ft(R + 1, 0), K(R), per(R), t(R, 0), done(R, 0), round(R, 0), np(R, 0);
  for (int i = 0; i < R; ++i) {
    long a, b, c;
    if (scanf("%ld %ld %ld", &a, &b, &c) != 3) return 1;
    ft[i + 1] = ft[i] + a; K[i] = b; per[i] = c;
  }
  auto fta = [&](int64_t i) -> int64_t { return ft[i]; };
  int64_t Q = 0, head = 0, lead = 0; int live = R; bool abort_ = false;
  for (int i = 0; i < R; ++i) Q += tasks_a_round(ft[i + 1] - ft[i]);
  std::vector<char> fin(R, 0);
  std::vector<std::vector<Wait>> waits(R);
  struct Ev { double at; int block, r, kind; int64_t n; };
  auto later = [](const Ev &a, const Ev &b) { return a.at > b.at || (a.at == b.at && a.block > b.block); };
  std::priority_queue<Ev, std::vector<Ev>, decltype(later)> ev(later);
  for (int b = 0; b < BLOCKS; ++b) ev.push({0.0, b, -1, 0, 0});
  auto start = [&](double at, int b, int r, int kind, int64_t n) {
    if (past_last_round(n, K[r])) { abort_ = true; return; }
    if (kind == 0) round[r] = n;
    ev.push({at + dur[kind], b, r, kind, n});
  };
  long steps = 0;
  while (!ev.empty() && !abort_ && ++steps < 50000000) {
    Ev e = ev.top(); ev.pop();
    if (e.r >= 0) {   // the task's effects, then its count
      const int r = e.r;
      if (e.kind == 0) {
        if (e.n == 0) t[r] = 1; else if (t[r] >= K[r]) fin[r] = 1;
        if (e.n == 0 && K[r] == 1) fin[r] = 1;
        if (fin[r]) --live;
      }
      if (e.kind == 1 && e.n > 0) t[r] = std::min(K[r], t[r] + per[r]);
      ++done[r];
      for (size_t i = 0; i < waits[r].size();) {
        const Wait w = waits[r][i];
        if (!fin[r] && done[r] < w.need) { ++i; continue; }
        waits[r].erase(waits[r].begin() + i);
        if (fin[r]) ev.push({e.at + DQ, w.block, -1, 0, 0}); else start(e.at + 1.0, w.block, r, w.kind, w.n);
      }
      ev.push({e.at + DQ, e.block, -1, 0, 0});
      continue;
    }
    if (live == 0) continue;   // the block ends
    const int64_t q = head++, m = q / Q;
    int64_t oldest = INT64_MAX;
    for (int i = 0; i < R; ++i) if (!fin[i]) oldest = std::min(oldest, round[i]);
    lead = std::max(lead, m - oldest);
    int kind = 0, r = 0, sub = 0;
    const int64_t n = m + decode_task(q - m * Q, (int64_t)R, fta, kind, r, sub);
    if (n < 0 || fin[r]) { ev.push({e.at + DQ, e.block, -1, 0, 0}); continue; }
    const int64_t need = tasks_before(n, kind, ft[r + 1] - ft[r]);
    if (done[r] >= need) start(e.at + 1.0, e.block, r, kind, n);
    else waits[r].push_back({e.block, need, kind, sub, n});
  }
  printf("%d %d %ld\n", R - live, abort_ ? 1 : 0, (long)lead);
  return 0;
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    return _compile(tmp_path_factory, "queue", MODEL)


@pytest.mark.parametrize("dq", [0.5, 2.5, 5.5])
@pytest.mark.parametrize("R,N,K,slow", [
    (64, 1024, 16, 1),     # one request whose rounds make one pick each
    (32, 2880, 10, 1),
    (64, 1024, 32, 2),
    (128, 600, 24, 1),
    (256, 256, 8, 1),
    (8, 16384, 40, 1),
    (1, 5000, 60, 1),
    (33, 1500, 16, 33),    # every request slow
])
def test_queue_ends_every_request(model, R, N, K, slow, dq):
    exe, f_rows = model
    rng = np.random.default_rng(R + K)
    reqs = []
    for r in range(R):
        n = int(rng.integers(max(1, N // 2), N + 1)) if N < 1000 else N
        reqs.append(((n + f_rows - 1) // f_rows, 2 if K == 24 and r >= slow else K, 1 if r < slow else 128))
    for order in (reqs, reqs[::-1]):
        out = subprocess.run([exe], input=f"{R} 256 {dq} 23 89 70 " + " ".join("%d %d %d" % x for x in order),
                             capture_output=True, text=True, check=True, timeout=60).stdout.split()
        ended, aborted, lead = map(int, out)
        assert (ended, aborted) == (R, 0)
        if (R, N, K) == (64, 1024, 16) and order is reqs:
            # far past K rounds: nothing may be concluded from the head's position
            assert lead > K + 4, lead
