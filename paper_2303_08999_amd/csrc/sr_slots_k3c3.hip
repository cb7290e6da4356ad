// k_assemble_slots for 3x3 atoms and two or three channels (sr_slots.h)
#include "sr_slots.h"

namespace srd {

hipError_t launch_slots_k3c3(const AssembleArgs& a, bool streamed, const LaunchTo& st) { return launch_slots_t<3, 3>(a, streamed, st); }

}  // namespace srd
