"""The scalar words of the conjugate gradient launches, walked on the host: no
word that a launch writes is read by any thread of it (what the threads of a
launch see then does not depend on their order), and an ended solve stays
ended to the last launch."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2601_16911_amd", "csrc")

WALK = r"""
#include "cvw_pcg.h"
#include <cstdio>
#include <cstdlib>
#include <set>
using namespace cvw;

double words[8];
std::set<int> rd, wr;
struct Word {
  int k;
  operator double() const { rd.insert(k); return words[k]; }
  double operator=(double v) const { wr.insert(k); return words[k] = v; }
};
struct Scalars { Word operator[](int k) const { return Word{k}; } };
const Scalars S;

void launch(const char* name, int it) {       // the end of a launch: what it read and wrote
  for (int k : wr)
    if (rd.count(k)) { printf("%s of iteration %d reads and writes word %d\n", name, it, k); exit(1); }
  rd.clear();
  wr.clear();
}

// a launch that begins iteration it: the writer's and another thread's way through it
bool begin(int it, double rz, float& beta) {
  bool on[2] = {false, false};
  for (int w = 1; w >= 0; --w) {              // the writer first
    float b = 0.0f;
    on[w] = pcg_enter(S, it, w) && (it == 0 ? pcg_begin<true>(rz, S, it, w, b) : pcg_begin<false>(rz, S, it, w, b));
    if (on[w]) beta = b;
  }
  launch("the beginning", it);
  if (on[0] != on[1]) { printf("threads part in iteration %d\n", it); exit(1); }
  return on[0];
}

// iterations that run when r.z is rz[it] at the beginning of each, of at most maxit; the state after them
int solve(const double* rz, int maxit, double tol2, double& state) {
  for (double& w : words) w = 7.0;            // nothing is read before it is written
  pcg_setup(S, tol2);
  launch("the setup", -1);
  int ran = 0;
  for (int it = 0; it < maxit; ++it) {
    float beta = -1.0f;
    const bool on = begin(it, rz[it], beta);
    if (on) {
      ++ran;
      if (beta != (it == 0 ? 0.0f : static_cast<float>(rz[it] / rz[it - 1]))) { printf("beta\n"); exit(1); }
    }
    for (const char* k : {"the gather", "the update"}) {
      if (pcg_runs(S, it) != on) { printf("%s of iteration %d: another state\n", k, it); exit(1); }
      if (on && static_cast<double>(S[pcg_rz_word(it)]) != rz[it]) { printf("r.z\n"); exit(1); }
      launch(k, it);
    }
  }
  state = S[pcg_state_word(maxit - 1)];
  launch("the finish", maxit - 1);
  return ran;
}

int main() {
  double rz[12], st;
  for (int end = 0; end <= 12; ++end) {       // the tolerance met at the beginning of iteration `end` (12: never)
    for (int i = 0; i < 12; ++i) rz[i] = i < end ? 1.0 / (i + 1) : i == end ? 1e-9 : 0.5;   // later values are stale
    if (end == 0) rz[0] = 0.0;
    const int ran = solve(rz, 12, 1e-6, st);
    if (ran != end || st != (end == 0 ? PCG_NO_RHS : end < 12 ? PCG_ENDED : PCG_RUNS)) {
      printf("end %d: ran %d, state %g\n", end, ran, st);
      return 1;
    }
  }
  return 0;
}
"""


@pytest.mark.parametrize("opt", ["-O0", "-O2"])
def test_launches_read_no_word_they_write(tmp_path, opt):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run(["g++", "-std=c++17", opt, "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
