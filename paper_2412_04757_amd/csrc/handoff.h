// A word by which one workgroup tells another that a result is in place. It is 0 before a launch and 0 again after it, also where
// the taker gave up waiting: it then leaves -1 behind, and the giver, who adds 1 whenever it comes, brings that back to 0. So a
// result that came too late is never taken for one of a later launch. Plain C++, so that the host tests can run every order of
// events. Word: load(), store(v), add(v) (returns the value before), pause(); each atomic at device scope.
#pragma once

#if defined(__HIPCC__)
#define LTRI_HANDOFF __device__ __forceinline__
#else
#define LTRI_HANDOFF inline
#endif

namespace ltri {

template <class Word>
LTRI_HANDOFF void handoff_give(Word w) { (void)w.add(1); }

// Waits for up to `polls` looks; false: it has not come. One taker for every giver.
template <class Word>
LTRI_HANDOFF bool handoff_take(Word w, int polls) {
  for (; polls > 0; --polls) {
    if (w.load() != 0) { w.store(0); return true; }
    w.pause();
  }
  return w.add(-1) != 0;             // it may have come since the last look: then it is there, and the word is 0
}

}  // namespace ltri
