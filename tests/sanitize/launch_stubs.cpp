// Launch stubs for the host-only sanitizer build of the ABI layer: every
// device launch aborts, so a validation failure that still reached a launch
// ends the run.  Only conv_channels_per_thread (a constant the validation
// reads) returns normally, and launches while a record is set (launch_stubs.hpp),
// which are noted there instead.
#include "launch_stubs.hpp"

#include <cstdio>
#include <cstdlib>

namespace sf {
LaunchRecord *launch_record = nullptr;
[[noreturn]] static void launched(const char *what) {
    std::fprintf(stderr, "unexpected launch: %s\n", what);
    std::abort();
}
hipError_t launch_kernel(int kind, int, int, const SegArgs &a, hipStream_t, hipEvent_t, hipEvent_t) {
    if (!launch_record) launched("launch_kernel");
    launch_record->seg.push_back({kind, a});
    return hipSuccess;
}
hipError_t launch_kernel_vg(int, int, int, const SegArgs &, hipStream_t, hipEvent_t, hipEvent_t) {
    launched("launch_kernel_vg");
}
hipError_t launch_state_copy(const float *, float *, int64_t, hipStream_t) { launched("launch_state_copy"); }
int conv_channels_per_thread() { return 8; }
hipError_t launch_conv(bool, const ConvArgs &a, hipStream_t, hipEvent_t, hipEvent_t) {
    if (!launch_record) launched("launch_conv");
    launch_record->conv.push_back(a);
    return hipSuccess;
}
hipError_t launch_gdn_phase(int, const GdnArgs &, int, hipStream_t, hipEvent_t, hipEvent_t) {
    launched("launch_gdn_phase");
}
}  // namespace sf
