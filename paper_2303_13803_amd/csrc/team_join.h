// How the workgroups of a launch that work together find each other (core.hip).
//
// They wait for one another all through the launch, so all of them have to be on compute units at the
// same time.  A launch that has the device to itself gets that by its size, and the last workgroup to arrive
// closes the team.  With another context's launch of this kind beside it, each may hold compute units that the
// other's workgroups are still waiting for: then nobody else will arrive, and after `patience` looks
// whoever waits closes the team with those that are there.  A workgroup that comes later leaves at once.
// (Waiting for all of them instead ended both launches only when their bounded waits ran out, seconds
// later, and both solves went on without this kernel.)
//
// No dependence on the device: tests/team_join.cpp runs it on threads.
#pragma once

#if defined(__HIPCC__)
#define MF_TEAM_FN __host__ __device__ __forceinline__
#else
#define MF_TEAM_FN inline
#endif

constexpr unsigned TEAM_CLOSED = 0x80000000u;

struct TeamWords {
    int *die;                           // the die of the first to arrive, -1 before
    unsigned *joined;                   // members so far; the top bit: closed
    unsigned *arrived;                  // workgroups that have been here, members or not
    unsigned *size;                     // 0 until the team is closed
};

// Returns the workgroup's number in the team, -1 (not in it: the caller leaves), or -2 (the wait ran out:
// the caller has to tell the others); *size: members.
template <class Mem>
MF_TEAM_FN int join_team(const Mem &mem, const TeamWords &at, int die, bool any_die, unsigned launched, unsigned most,
                         unsigned patience, unsigned give_up, unsigned *number, unsigned *size)
{
    auto close = [&]() {
        const unsigned was = mem.set_bits(at.joined, TEAM_CLOSED);
        if (!(was & TEAM_CLOSED)) mem.store(at.size, was < most ? was : most);
    };
    const int first = mem.swap_if(at.die, -1, die);
    *number = any_die || first == -1 || first == die ? mem.add(at.joined, 1u) : TEAM_CLOSED;
    mem.settle();                                        // who has arrived has been counted
    if (mem.add(at.arrived, 1u) + 1u == launched) close();
    if (*number >= most) return -1;                      // (closed before: the top bit is set)
    for (unsigned looks = 0; (*size = mem.load(at.size)) == 0u;) {
        if (++looks > give_up) return -2;
        if (looks == patience) close();
    }
    return (int)*number;
}
