// Launches noted instead of aborting, while launch_record points at a record.
#pragma once

#include <utility>
#include <vector>

#include "sf_launch.hpp"

namespace sf {
struct LaunchRecord {
    std::vector<std::pair<int, SegArgs>> seg;  // kernel kind, arguments
    std::vector<ConvArgs> conv;
};
extern LaunchRecord *launch_record;
}  // namespace sf
