// error.h -- the failure that every internal function throws and the C entry
// points turn into a status (host only, no HIP).
#pragma once

#include <string>

#include "../../include/gfr.h"

namespace gfr {

struct Error {
    gfr_status code;
    std::string msg;
};

[[noreturn]] void fail(gfr_status code, const std::string &msg);

}  // namespace gfr
