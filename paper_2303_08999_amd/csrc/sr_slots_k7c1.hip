// k_assemble_slots for 7x7 atoms and one channel (sr_slots.h)
#include "sr_slots.h"

namespace srd {

hipError_t launch_slots_k7c1(const AssembleArgs& a, bool streamed, const LaunchTo& st) { return launch_slots_t<7, 1>(a, streamed, st); }

}  // namespace srd
