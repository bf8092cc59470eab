// The scalars of a conjugate gradient solve whose iterations are launches.
//
// Every block of a launch acts on them, and block 0 of some launches writes
// them, so no launch reads a word that it writes: r.z and the state are kept
// twice and alternate by iteration.  The launch that begins iteration `it`
// reads the words of it - 1 and writes those of it, also when the solve has
// ended before, and the later launches of the iteration only read them.  All
// threads of a block therefore take the same way at their barriers.
#pragma once

#ifdef __HIPCC__
#define CVW_PCG_FN __device__ __forceinline__
#else
#define CVW_PCG_FN inline      // host programs that walk the launches
#endif

namespace cvw {

enum { S_RZ = 0, S_RZ_ODD = 1, S_RZ0 = 2, S_ALPHA = 3, S_BETA = 4, S_STATE = 5, S_STATE_ODD = 6, S_TOL2 = 7 };
// the state: still running, tolerance met (or broken down), zero right-hand side (x = 0)
enum { PCG_RUNS = 0, PCG_ENDED = 1, PCG_NO_RHS = 2 };

CVW_PCG_FN int pcg_rz_word(int it) { return (it & 1) ? S_RZ_ODD : S_RZ; }
CVW_PCG_FN int pcg_state_word(int it) { return (it & 1) ? S_STATE_ODD : S_STATE; }

// before iteration 0 (a launch of its own)
template <typename SCALARS>
CVW_PCG_FN void pcg_setup(SCALARS S, double tol2) {
  S[pcg_state_word(-1)] = PCG_RUNS;
  S[S_TOL2] = tol2;
}

// whether iteration `it` runs, in its launches after the one that begins it
template <typename SCALARS>
CVW_PCG_FN bool pcg_runs(SCALARS S, int it) {
  return S[pcg_state_word(it)] == PCG_RUNS;
}

// On entry of the launch that begins iteration `it` (writer: one thread of the
// launch).  false: the solve has ended.
template <typename SCALARS>
CVW_PCG_FN bool pcg_enter(SCALARS S, int it, bool writer) {
  const double state = S[pcg_state_word(it - 1)];
  if (state == PCG_RUNS) return true;
  if (writer) S[pcg_state_word(it)] = state;
  return false;
}

// The recurrence at the start of iteration `it`, from rz = r.z: rz0, beta, the
// end of the solve (a zero right-hand side, or the tolerance met).  false: ended.
template <bool FIRST, typename SCALARS>
CVW_PCG_FN bool pcg_begin(double rz, SCALARS S, int it, bool writer, float& beta) {
  const double b = FIRST ? 0.0 : rz / S[pcg_rz_word(it - 1)];
  const bool ended = FIRST ? !(rz > 0.0) : !(rz > S[S_TOL2] * S[S_RZ0]);
  if (writer) {
    S[pcg_rz_word(it)] = rz;
    S[S_BETA] = b;
    if (FIRST) S[S_RZ0] = rz;
    S[pcg_state_word(it)] = !ended ? PCG_RUNS : (FIRST ? PCG_NO_RHS : PCG_ENDED);
  }
  beta = static_cast<float>(b);
  return !ended;
}

}  // namespace cvw
