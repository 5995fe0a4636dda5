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
