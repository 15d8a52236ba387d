// error.h -- the failure that every internal function throws and the C entry
// points turn into a status (host only, no HIP).
#pragma once

#include <string>

#include "../../include/gfr.h"

namespace gfr {

struct Error {
    gfr_status code;
    std::string msg;
    bool crowded = false;   // a wait between work-groups ran out: something else held the device
};

[[noreturn]] void fail(gfr_status code, const std::string &msg);

[[noreturn]] inline void fail_crowded(const std::string &who)
{
    throw Error{GFR_E_DEVICE, who + ": frontier compaction look-back timed out", true};
}

// call(), and once more if it failed and mend(the failure) says that this makes sense
template <class Call, class Mend> void call_again_if(Call call, Mend mend)
{
    try {
        call();
        return;
    } catch (const Error &e) {
        if (!mend(e)) throw;
    }
    call();
}

}  // namespace gfr
