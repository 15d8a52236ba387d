// spare.h -- device structures that only make calls faster and that a call
// can do without when memory is short (host only, no HIP).
#pragma once

#include "error.h"

namespace gfr {

// Whether such a structure is there.  It counts as made only once everything
// that fills it has succeeded: a structure that was allocated when something
// failed is given back, and no later call finds it.
struct Spare {
    enum State { NONE, MADE, NO_ROOM } state = NONE;

    // True when it is there, made now if nothing was tried yet.  make() fails by
    // an exception; release() gives back whatever make() took.  Without room for
    // it: false, now and later; any other failure is the caller's, and the next
    // call tries again.
    template <class Make, class Release> bool get(Make make, Release release)
    {
        if (state != NONE) return state == MADE;
        try {
            make();
        } catch (const Error &e) {
            release();
            if (e.code != GFR_E_OOM) throw;
            state = NO_ROOM;
            return false;
        } catch (...) {
            release();
            throw;
        }
        state = MADE;
        return true;
    }
};

// call(), and once more if it ran out of device memory and give_back() freed some
template <class Call, class GiveBack> void with_room(Call call, GiveBack give_back)
{
    try {
        call();
        return;
    } catch (const Error &e) {
        if (e.code != GFR_E_OOM || !give_back()) throw;
    }
    call();
}

}  // namespace gfr
