"""Host check of the bounded wait of a gang's exchange: the wait functions are taken from the device header, compiled
for the host against a memory whose slots carry their tag from a given tick on, and run as one lane.  Whatever is
missing, a gather gives up one time-out after its exchange began."""
import os
import re
import subprocess

import pytest

HDR = os.path.join(os.path.dirname(__file__), "..", "paper_1302_2073_amd", "csrc", "prost_frame.hpp")

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <cstddef>
#define __device__
#define __forceinline__ inline
#define __any(x) (x)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, o, s) (*(p))
#define __hip_atomic_fetch_or(p, v, o, s) (*(p) |= (v))
constexpr unsigned kErrTimeout = 1u;
struct FrameArgs { unsigned* sync; long long timeout; };
static long long ticks = 0;
static const double* memory;
static long long* arrives;       // tick from which a value carries the tag
static unsigned epoch;
inline long long now_ticks() { return ticks; }
inline double tagged(double v, unsigned t) {
  unsigned long long b; std::memcpy(&b, &v, 8); b = (b & ~0xFFull) | t; std::memcpy(&v, &b, 8); return v;
}
inline unsigned tag_of(double v) { unsigned long long b; std::memcpy(&b, &v, 8); return (unsigned)(b & 0xFF); }
inline double untag(double v) { return tagged(v, 0); }
inline double ld_tagged(const double* p) {
  ++ticks;
  return tagged(*p, ticks >= arrives[p - memory] ? epoch : (epoch + 1) & 0xFF);
}
%s
int main(int argc, char** argv) {
  // n stride q0 dq comp timeout raised-at-the-start, then n * stride arrival ticks on stdin
  const int n = std::atoi(argv[1]), stride = std::atoi(argv[2]), q0 = std::atoi(argv[3]), dq = std::atoi(argv[4]);
  const int comp = std::atoi(argv[5]);
  unsigned sync[8] = {0, 0, (unsigned)std::atoi(argv[7]), 0, 0, 0, 0, 0};
  FrameArgs a{sync, std::atoll(argv[6])};
  double* m = new double[n * stride];
  arrives = new long long[n * stride];
  for (int i = 0; i < n * stride; ++i) { m[i] = i + 1; if (std::scanf("%%lld", &arrives[i]) != 1) return 1; }
  memory = m;
  epoch = 7;
  double v = 0, vx = 0;
  GangWait w{now_ticks(), 0};
  poll_slots<17>(m, n, stride, q0, dq, comp, epoch, a, v, vx, w);
  std::printf("%%lld %%d %%u %%.17g %%.17g\n", ticks, w.bad, sync[2], v, vx);
}
"""

N, STRIDE, Q0, DQ, TIMEOUT = 90, 32, 3, 32, 100000
VALUES = 6                  # the lane's: slots 3, 35 and 67, two components each
SLACK = 64 * VALUES + 64    # a check every 64 polls of each, and the loads themselves


@pytest.fixture(scope="module")
def lane(tmp_path_factory):
    src = open(HDR).read()
    body = re.search(r"struct GangWait \{.*?(?=// Raises the gang's time-out bit)", src, re.S).group(0)
    d = tmp_path_factory.mktemp("wait")
    (d / "wait.cpp").write_text(HARNESS % body)
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", str(d / "wait"), str(d / "wait.cpp")], check=True)

    def run(arrival, comp=0, raised=0):
        out = subprocess.run([str(d / "wait")] + [str(x) for x in (N, STRIDE, Q0, DQ, comp, TIMEOUT, raised)],
                             input=" ".join(str(arrival(q, c)) for q in range(N) for c in range(STRIDE)),
                             capture_output=True, text=True, check=True, timeout=60).stdout.split()
        return int(out[0]), int(out[1]), int(out[2]), float(out[3]), float(out[4])
    return run


NEVER = 1 << 60


def _sums(comp):
    mine = range(Q0, N, DQ)
    return float(sum(q * STRIDE + comp + 1 for q in mine)), float(sum(q * STRIDE + 16 + comp + 1 for q in mine)
                                                                  if comp == 0 else 0)


@pytest.mark.parametrize("comp", [0, 1, 15])
def test_values_that_are_there_are_summed_without_a_wait(lane, comp):
    ticks, bad, word, v, vx = lane(lambda q, c: 0, comp)
    assert (bad, word) == (0, 0) and ticks <= 6 and (v, vx) == _sums(comp)


def test_late_values_are_waited_for(lane):
    ticks, bad, word, v, vx = lane(lambda q, c: (q * STRIDE + c) * TIMEOUT // (2 * N * STRIDE), 0)
    assert (bad, word) == (0, 0) and ticks <= TIMEOUT // 2 + SLACK and (v, vx) == _sums(0)


@pytest.mark.parametrize("missing", ["all", "one", "last", "second component"])
def test_missing_values_cost_one_time_out(lane, missing):
    def arrival(q, c):
        gone = {"all": True, "one": q == Q0, "last": q == Q0 + 2 * DQ, "second component": c == 16}[missing]
        return NEVER if gone else 0
    ticks, bad, word, _, _ = lane(arrival, 0)
    assert (bad, word) == (1, 0) and TIMEOUT < ticks <= TIMEOUT + SLACK


def test_values_that_come_one_by_one_share_the_clock(lane):
    """Each of them 0.9 of the time-out after the one before: no single wait is too long, the gather is."""
    order = {(q, c): i for i, (q, c) in enumerate((q, c) for q in range(Q0, N, DQ) for c in (0, 16))}
    ticks, bad, word, _, _ = lane(lambda q, c: (order.get((q, c), 0) + 1) * 9 * TIMEOUT // 10, 0)
    assert (bad, word) == (1, 0) and ticks <= TIMEOUT + SLACK


def test_a_gang_that_has_given_up_is_not_waited_for(lane):
    ticks, bad, word, _, _ = lane(lambda q, c: NEVER, 0, raised=1)
    assert (bad, word) == (1, 1) and ticks <= SLACK
