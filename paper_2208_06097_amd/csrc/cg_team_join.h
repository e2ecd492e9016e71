// How the workgroups of a team CG launch (k_cg.hip) come together.
//
// The members of a team wait for each other, so a team may begin only when all
// of them run.  Which workgroups run at a time is not the launch's to say: other
// streams and processes hold CUs, and a stream may be restricted to a few.  So
// teams form in the order of arrival.  A workgroup that has begun to run takes
// the next place of its class; a team is complete when its last place is taken,
// and its members then keep their CUs until they end.  A team that is not
// complete when a member's patience ends closes the class: nobody takes a place
// there any more, and its members leave without having taken a pair.
//
// The class's word counts the places taken, with TEAM_CLOSED once it takes no
// more.  Places are taken by compare-and-swap, so a closed class's count is
// final and everyone who looks decides alike.
#pragma once

constexpr unsigned TEAM_CLOSED = 1u << 31;

// This workgroup's place (team place / size, member place % size), or -1.
// m: load() the word, cas(expected, desired) returning what was there,
// expired() whether patience has ended, pause() between two looks.
template <typename Word>
__host__ __device__ inline int team_join(Word& m, int size, int places) {
    unsigned w = m.load();
    for (;;) {
        if ((w & TEAM_CLOSED) || (int)w >= places) return -1;
        const unsigned seen = m.cas(w, w + 1);
        if (seen == w) break;
        w = seen;
    }
    const unsigned place = w, full = (place / size + 1) * size;
    for (;;) {
        w = m.load();
        if ((w & ~TEAM_CLOSED) >= full) return (int)place;
        if (w & TEAM_CLOSED) return -1;
        if (m.expired()) (void)m.cas(w, w | TEAM_CLOSED);   // (a late arrival may have been faster)
        else m.pause();
    }
}
