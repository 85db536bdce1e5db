"""CPU: the enrolment, the barrier and the end of a team (csrc/team.h) on a model of XCDs with their own L2.

The header is compiled for the CPU with stand-ins for the device builtins.  A
workgroup is a few threads; a store of workgroup scope and a plain one stay in
the L2 of their XCD until the launch ends, accesses of device scope go to
memory, and the L2s are written back one after the other (in both orders) when
a launch has ended.  Whatever XCDs
the candidates run on and in whatever order they leave, each launch has one
team, its ranks are 0..n-1, and no member passes a barrier that another member
has not reached.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TEAM_H = os.path.join(ROOT, "paper_2608_09102_amd", "csrc", "team.h")

MODEL = r"""
#pragma once
#include <pthread.h>
#include <stdint.h>
#include <string.h>
#include <unistd.h>
#include <map>
#include <mutex>
#define __HIPCC__ 1
#define __device__
#define __HIP_MEMORY_SCOPE_WORKGROUP 1
#define __HIP_MEMORY_SCOPE_AGENT 2
namespace sim {
constexpr int GROUPS = 4, LANES = 8, XCDS = 8;
struct Dim { unsigned x; };
inline std::mutex mu;
inline std::map<char*, std::pair<uint64_t, int>> dirty[XCDS];  // stores that wait in an XCD's L2
inline thread_local int group, xcd;
inline pthread_barrier_t bar[GROUPS];
inline unsigned votes[GROUPS];
template <typename T, int ID>
T& shared() {  // LDS: an object per workgroup
  static T v[GROUPS];
  return v[group];
}
template <typename X>
X load(const X* p) {
  usleep(50);
  std::lock_guard<std::mutex> lk(mu);
  X v = *p;
  auto it = dirty[xcd].find((char*)p);
  if (it != dirty[xcd].end()) memcpy(&v, &it->second.first, sizeof(X));
  return v;
}
template <typename X, typename Y>
void store(X* p, Y y, int scope) {
  std::lock_guard<std::mutex> lk(mu);
  const X v = (X)y;
  if (scope == __HIP_MEMORY_SCOPE_WORKGROUP) {
    uint64_t u = 0;
    memcpy(&u, &v, sizeof(X));
    dirty[xcd][(char*)p] = {u, (int)sizeof(X)};
  } else {
    dirty[xcd].erase((char*)p);
    *p = v;
  }
}
template <typename X, typename F>
X update(X* p, F f, int scope) {
  std::lock_guard<std::mutex> lk(mu);
  X old = *p;
  if (scope == __HIP_MEMORY_SCOPE_WORKGROUP) {
    auto& d = dirty[xcd];
    auto it = d.find((char*)p);
    if (it != d.end()) memcpy(&old, &it->second.first, sizeof(X));
    const X v = f(old);
    uint64_t u = 0;
    memcpy(&u, &v, sizeof(X));
    d[(char*)p] = {u, (int)sizeof(X)};
  } else {
    *p = f(old);
  }
  return old;
}
inline void write_back(bool up) {  // ascending or descending XCDs: the order is the hardware's own
  for (int k = 0; k < XCDS; ++k) {
    auto& d = dirty[up ? k : XCDS - 1 - k];
    for (auto& e : d) memcpy(e.first, &e.second.first, e.second.second);
    d.clear();
  }
}
inline void sync() { pthread_barrier_wait(&bar[group]); }
inline unsigned first(unsigned v, unsigned lane) {
  if (lane == 0) votes[group] = v;
  sync();
  const unsigned r = votes[group];
  sync();
  return r;
}
inline bool all(bool b, unsigned lane) {
  if (lane == 0) votes[group] = 0;
  sync();
  if (b) __atomic_fetch_add(&votes[group], 1u, __ATOMIC_SEQ_CST);
  sync();
  const bool r = votes[group] == LANES;
  sync();
  return r;
}
}  // namespace sim
inline thread_local sim::Dim threadIdx, blockIdx;
#define __builtin_amdgcn_s_getreg(r) ((unsigned)sim::xcd)
#define __builtin_amdgcn_readfirstlane(v) sim::first((v), threadIdx.x)
#define __syncthreads() sim::sync()
#define __all(pred) sim::all((pred), threadIdx.x)
#define __hip_atomic_load(p, o, sc) sim::load(p)
#define __hip_atomic_store(p, v, o, sc) sim::store(p, v, sc)
#define __hip_atomic_fetch_add(p, v, o, sc) sim::update(p, [&](auto q) { return q + (v); }, sc)
#define __hip_atomic_fetch_or(p, v, o, sc) sim::update(p, [&](auto q) { return q | (v); }, sc)
"""

MAIN = r"""
#include "team_model.h"
#include <stdio.h>
#include <stdlib.h>
#include <vector>
using namespace llg;
static TeamState state;
static int steps, arrived[64], ranks, members, teams, gone, bad;
static int polls;
struct Job { int group, lane, xcd, late, lag; };  // late 1: after the others have left, 2: after 30 ms

static void* run(void* a) {
  const Job j = *(Job*)a;
  sim::group = j.group;
  sim::xcd = j.xcd;
  threadIdx.x = j.lane;
  blockIdx.x = 8 * j.group + 3;
  if (j.late == 2) usleep(30000);
  if (j.late == 1)
    while (__atomic_load_n(&gone, __ATOMIC_SEQ_CST) < sim::GROUPS - 1) usleep(200);
  Team t;
  if (t.join(&state, 3, polls)) {
    if (j.lane == 0) {
      __atomic_fetch_add(&members, 1, __ATOMIC_SEQ_CST);
      if (__atomic_fetch_or(&ranks, 1 << t.rank, __ATOMIC_SEQ_CST) >> t.rank & 1) bad |= 1;
      if (t.rank == 0) __atomic_store_n(&teams, (int)t.n, __ATOMIC_SEQ_CST);
    }
    for (int k = 0; k < steps; ++k) {
      if (j.lane == 0) {
        if (j.lag) usleep(2000);
        __atomic_fetch_add(&arrived[k], 1, __ATOMIC_SEQ_CST);
      }
      t.barrier();
      if (__atomic_load_n(&arrived[k], __ATOMIC_SEQ_CST) < (int)t.n) bad |= 2;
    }
    t.leave();
  }
  if (j.lane == 0) __atomic_fetch_add(&gone, 1, __ATOMIC_SEQ_CST);
  return nullptr;
}

int main(int argc, char** argv) {  // order of write-back; per launch: barriers, polls, then xcd, late, lag of each workgroup
  for (int g = 0; g < sim::GROUPS; ++g) pthread_barrier_init(&sim::bar[g], nullptr, sim::LANES);
  const bool up = atoi(argv[1]) != 0;
  int a = 2;
  for (int launch = 0; a < argc; ++launch) {
    steps = atoi(argv[a++]);
    polls = atoi(argv[a++]);
    memset(arrived, 0, sizeof(arrived));
    ranks = members = teams = gone = bad = 0;
    std::vector<Job> jobs;
    for (int g = 0; g < sim::GROUPS; ++g, a += 3)
      for (int l = 0; l < sim::LANES; ++l) jobs.push_back({g, l, atoi(argv[a]), atoi(argv[a + 1]), atoi(argv[a + 2])});
    std::vector<pthread_t> th(jobs.size());
    for (size_t k = 0; k < jobs.size(); ++k) pthread_create(&th[k], nullptr, run, &jobs[k]);
    for (auto t : th) pthread_join(t, nullptr);
    sim::write_back(up);
    if (members < 1 || members != teams || ranks != (1 << members) - 1) bad |= 4;
    printf("launch %d: %d members, bad %d\n", launch, members, bad);
    fflush(stdout);
    if (bad) return 1;
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    d = tmp_path_factory.mktemp("team")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(MODEL)
    src, n = re.subn(r"TEAM_W = 32;", "TEAM_W = 4;", open(TEAM_H).read())
    assert n == 1
    src = re.sub(r'asm volatile\("s_waitcnt vmcnt\(0\)"[^;]*;', ";", src)  # the model's stores are done at once
    # a plain store stays in the XCD's L2 as one of workgroup scope does
    src = re.sub(r"\bs->(\w+(?:\[\w+\])?) = ([^;]+);", r"sim::store(&s->\1, \2, 1);", src)
    src, n = re.subn(r"__shared__ ([\w ]+?) (\w+)(\[\d+\])?;", r"auto& \2 = sim::shared<\1\3, __COUNTER__>();", src)
    assert n >= 1
    (d / "team_model.h").write_text('#include "hip/hip_runtime.h"\n' + src)
    (d / "main.cpp").write_text(MAIN)
    exe = d / "team"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", str(d), str(d / "main.cpp"), "-o", str(exe)],
                   check=True)
    return str(exe)


# per launch: barriers, and of four workgroups the XCD and L "starts when the
# others have left", S "starts late", 1 "is slow to each barrier"; the polls of
# the first and, where these suffice for all to join, the members
LAUNCHES = {
    "one XCD": [(3, "00 00 00 00"), (4, "00 01 00 00"), (2, "00 00 00 01")],
    "a late one on another XCD leaves last": [(3, "00 00 00 1L"), (3, "00 01 00 0L"), (3, "01 00 00 00")],
    "a late one on the team's XCD leaves last": [(3, "00 00 00 0L"), (3, "00 01 00 0L")],
    "teams on changing XCDs": [(2, "00 00 00 1L"), (3, "10 11 10 0L"), (4, "00 01 00 01"), (1, "10 11 11 10")],
    "no barrier": [(0, "00 00 00 1L"), (2, "00 01 00 00")],
    "a slow start": [(3, "00 0S 00 00", 4000, 4), (3, "00 0S 00 01"), (3, "00 01 00 0S", 4000, 4)],
    "a mixed start": [(3, "00 10 00 10"), (3, "00 01 00 11"), (3, "20 01 21 00"), (3, "00 01 00 01")],
}


@pytest.mark.parametrize("up", (1, 0), ids=("up", "down"))
@pytest.mark.parametrize("name", LAUNCHES)
def test_team_protocol(model, name, up):
    args = [str(up)]
    for steps, groups, *polls in LAUNCHES[name]:
        args += [str(steps), str(polls[0] if polls else 64)]
        for g in groups.split():
            args += [g[0], {"L": "1", "S": "2"}.get(g[1], "0"), "1" if g[1] == "1" else "0"]
    r = subprocess.run([model] + args, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    members = [int(x.split()[2]) for x in r.stdout.splitlines()]
    assert len(members) == len(LAUNCHES[name])
    for got, (_, _, *polls) in zip(members, LAUNCHES[name]):
        assert not polls or got == polls[1]
