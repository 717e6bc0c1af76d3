// Whether a solver's next solve may take its cooperative form.  Plain C++.
#pragma once

namespace oasis {

// A halo that does not fit is the matrix's for good.  Launches that other work
// kept from coming together are not: the next solves then take the launched
// form, which needs nobody else's CUs, 16 at first and twice as many after
// each further failure up to 1024, so that a card that stays busy costs the
// waits (some 50 ms) only now and then, and one that is free again is used.
struct CoopUse {
    bool never = false;
    int rest = 0, failed = 0;
    // asked once a solve
    bool next() {
        if (never) return false;
        if (rest == 0) return true;
        --rest;
        return false;
    }
    void worked() { failed = 0; }
    void gave_up() {
        rest = 16 << (failed < 6 ? failed : 6);
        ++failed;
    }
};

}  // namespace oasis
