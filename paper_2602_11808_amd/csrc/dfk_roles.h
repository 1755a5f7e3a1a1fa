// How the down workgroups of the launch that holds both kernels' workgroups (dfk_mfma_km.hip) wait for its gate/up workgroups.
// Free of device code, so that a host program can run it too: `Mem` supplies relaxed memory operations of device scope.
//
// A gate/up workgroup waits for nobody.  A down workgroup waits until the slices of its d_ff split have been published.  Alone on
// the device that wait ends by itself: each XCD takes a grid's workgroups in index order, gate/up first.  Two launches on two
// streams could block each other: one XCD takes the workgroups of the first launch first, another those of the second, and both
// fill up with down workgroups that wait for gate/up workgroups which find no room on the other XCD.  So a down workgroup that
// has waited for long parks: it leaves a note and ends, and makes room.  One per launch may not, the last that has neither passed
// its wait nor parked; it does the work of those that have when its own is done.  What waits for good is then one workgroup per
// launch in flight, and as long as these are fewer than the CUs of an XCD (a process has 4 hardware queues, 32 at most), every
// gate/up workgroup gets its turn.
#pragma once

#if defined(__HIPCC__)
#define DFK_HD __host__ __device__ __forceinline__
#else
#define DFK_HD inline
#endif

namespace dfk {

// Words in the counter area of the workspace, zero between launches (column block counters occupy [0, 512), the second reduction
// level word 512, the slice-local fused kernel word 1023).
constexpr int kRoleCount0 = 520;    // per d_ff split of the down projection: gate/up workgroups that have published
constexpr int kRoleCountEnd = 1020; //   A_2 rows of that split; RoleShape::stride words apart (spread over cache lines)
constexpr int kRoleNotes = 1021;    // notes left in the list of parked workgroups
constexpr int kRolePassed = 1022;   // down workgroups past their wait, plus 65536 times those parked

struct RoleShape {
    int n_down;     // down workgroups, at most 65535
    int splits;     // d_ff splits of the down projection
    int stride;
};

// Polls after which a down workgroup parks: far more than a healthy wait takes (tens of microseconds; a poll is about a third of
// one).
constexpr int kRoleParkPolls = 1024;

// Down workgroups that have neither passed nor parked.
DFK_HD unsigned role_left(const RoleShape& s, unsigned passed_word) {
    return (unsigned)s.n_down - (passed_word & 0xffffu) - (passed_word >> 16);
}

// True if workgroup `wg` has parked; false if all the others have passed or parked.  `list` has room for every down workgroup;
// each tries once.
template <typename Mem>
DFK_HD bool role_park(unsigned* t, const RoleShape& s, unsigned* list, int wg) {
    Mem::store(list + Mem::fetch_add(t + kRoleNotes, 1u), (unsigned)wg);
    Mem::settle();                                              // the note is there before it counts
    if (role_left(s, Mem::fetch_add(t + kRolePassed, 0x10000u)) > 1u) return true;
    Mem::fetch_add(t + kRolePassed, (unsigned)-0x10000);        // nobody else is left to see it meanwhile
    Mem::settle();
    return false;
}

// Waits for `expected` gate/up workgroups of split js.  list: nullptr where parking is out of the question.
enum RoleWait { kRoleReady, kRoleParked, kRoleGaveUp };
template <typename Mem>
DFK_HD int role_wait(unsigned* t, const RoleShape& s, int js, unsigned expected, int limit, unsigned* list, int wg) {
    int polls = 0;
    while (Mem::load(t + kRoleCount0 + js * s.stride) < expected) {
        if (++polls > limit) return kRoleGaveUp;
        if (list && polls == kRoleParkPolls && role_park<Mem>(t, s, list, wg)) return kRoleParked;
        Mem::pause();
    }
    return kRoleReady;
}

// Says that a down workgroup is past its wait; the answer is the word as it was (role_left of it is 1: the caller is the last).
template <typename Mem>
DFK_HD unsigned role_pass(unsigned* t) { return Mem::fetch_add(t + kRolePassed, 1u); }

// The words as the next launch needs them.  For the last workgroup, once it is past the waits of the parked ones too.
template <typename Mem>
DFK_HD void role_clear(unsigned* t, const RoleShape& s) {
    Mem::store(t + kRolePassed, 0u);
    Mem::store(t + kRoleNotes, 0u);
    for (int js = 0; js < s.splits; ++js) Mem::store(t + kRoleCount0 + js * s.stride, 0u);
}

}  // namespace dfk
