// How the waves of a workgroup that walks over pairs hand its two slab buffers over (a host test compiles
// and runs this code too).
//
// A barrier per pair lets the waves of a SIMD start every pair together, with nothing in their pipelines, and makes
// all wait for the last one; what has to hold is less: a pair is walked when every wave's part of its slab has
// landed, and a buffer is filled when every wave has read it.  Two counters say so, and a wave may then run ahead of
// another by part of a pair:
//   the first slab is requested; slab_landed();
//   wait_landed(i); first steps of pair i; wait_read(i), request the slab of pair i + 1; more steps;
//   slab_landed(); last steps; slab_read().
// Every wave of the workgroup goes through the same number of pairs, and none waits for something that it
// has not itself done before: wait_landed(i) asks for what every wave does within pair i - 1 (the first
// slab: before the walk), wait_read(i) for the end of pair i - 1.  So the last wave never waits for long.
// No pairs at all: nobody requests, waits or counts anything.
#pragma once

#if defined(__HIP__)
#include <hip/hip_runtime.h>
#define LMKAN_GATE_FN __device__ __forceinline__
#else
#define LMKAN_GATE_FN inline
#endif

namespace lmkan {

// COUNTERS: arrive_landed(), arrive_read(): one more wave; until_landed(n), until_read(n): returns when as many have
// arrived; own_landed(): returns when what this wave has requested is there.
template <typename COUNTERS>
struct GateOrder : COUNTERS {
    // waits until this wave's part of the slab requested last is in LDS, and says so
    LMKAN_GATE_FN void slab_landed() const
    {
        COUNTERS::own_landed();
        COUNTERS::arrive_landed();
    }
    LMKAN_GATE_FN void slab_read() const { COUNTERS::arrive_read(); }
    // step = pairs this workgroup has walked before this one
    template <int WAVES>
    LMKAN_GATE_FN void wait_landed(int step) const
    {
        COUNTERS::until_landed(WAVES * (step + 1));
    }
    template <int WAVES>
    LMKAN_GATE_FN void wait_read(int step) const
    {
        COUNTERS::until_read(WAVES * step);
    }
    // The walk of a wave without samples: it fetches its part of every slab, as soon as there is room, and leaves the
    // SIMD to the others.  request(i, wanted): the slab of pair i.
    template <int WAVES, typename F>
    LMKAN_GATE_FN void feed_only(int n_pairs, F &&request) const
    {
        if (n_pairs <= 0) return;
        // (the first slab is in place before anyone reports the second: one count per wave and slab.  Later on
        // wait_read sees to that.)
        wait_landed<WAVES>(0);
        for (int i = 0; i < n_pairs; ++i) {
            wait_read<WAVES>(i);
            request(i + 1, i + 1 < n_pairs);
            slab_landed();
            slab_read();
        }
    }
};

}  // namespace lmkan
