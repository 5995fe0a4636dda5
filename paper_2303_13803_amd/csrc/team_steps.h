// How the workgroups of a launch that work together come to the same decisions (core.hip).
//
// They go in steps, with a barrier over all of them after each, and every workgroup decides for
// itself, from counts they have all added to, what the next step is.  Some of those decisions lead
// to barriers of their own, so all have to decide alike.  A workgroup (or one wavefront of it) that is held up
// after a barrier reads those counts when the others are in the middle of the next step: nothing the next step
// does may change them.
//
// No dependence on the device: tests/team_steps.cpp runs this on threads, one of which is held up.
#pragma once

#if defined(__HIPCC__)
#define MF_STEPS_FN __host__ __device__ __forceinline__
#else
#define MF_STEPS_FN inline
#endif

// ---- counts kept from one step to the next: a ring of four ----
// Step e begins with reading its own count, adds to that of e + 1 and clears that of e + 2.  Whoever is late reading
// meets others in step e, none in e + 1: a barrier is in between.  Every stage of a launch is a step of the same
// ring, also those that do not bid, and steps are never counted from the start again; the rings are clear when the
// launch begins.  (Stages used to begin by clearing the whole ring, which could come before somebody's
// reading of what the stage before had left: bidders left over read as none, or as all of the next phase's.)
constexpr unsigned STEP_RING = 4;
MF_STEPS_FN unsigned step_reads(unsigned step) { return step % STEP_RING; }
MF_STEPS_FN unsigned step_fills(unsigned step) { return (step + 1u) % STEP_RING; }
MF_STEPS_FN unsigned step_clears(unsigned step) { return (step + 2u) % STEP_RING; }

// ---- new labels for the columns of a served tree ----
// The scanned rows offer them again: either every scanned row's list is looked through once more, or the lists are kept
// by column from here on (`make`, which has barriers of its own).  Which, is decided by how many rows all workgroups have
// looked at for the trees before this one.  What they added then ended at the barrier at the end; what they add for
// this tree comes after the one in the middle.  So the count is read before that one.  (Read behind it, it met
// the additions of those that had gone on, and some entered the barriers of `make` without the others.)
// clear(): the tree's columns lose their labels.  offer(by_column): returns the rows this workgroup has looked at.
// team.bidders_left(): is asked after `clear` and its barrier.  Returns false when a wait ran out.
template <class Team, class Clear, class Make, class Offer>
MF_STEPS_FN bool labels_of_served_tree(Team &team, bool &by_column, bool must, unsigned long long most, const Clear &clear,
                                       const Make &make, const Offer &offer)
{
    const bool now = !by_column && (must || team.rows_looked_at() > most);
    clear();
    if (!team.barrier()) return false;
    if (!team.bidders_left()) return true;
    if (now) {
        if (!make()) return false;
        by_column = true;
    }
    team.add_rows_looked_at(offer(by_column));
    return team.barrier();
}
