// k_assemble_slots for 7x7 atoms and two or three channels (sr_slots.h)
#include "sr_slots.h"

namespace srd {

hipError_t launch_slots_k7c3(const AssembleArgs& a, bool streamed, const LaunchTo& st) { return launch_slots_t<7, 3>(a, streamed, st); }

}  // namespace srd
