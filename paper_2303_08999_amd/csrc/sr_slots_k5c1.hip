// k_assemble_slots for 5x5 atoms and one channel (sr_slots.h)
#include "sr_slots.h"

namespace srd {

hipError_t launch_slots_k5c1(const AssembleArgs& a, bool streamed, const LaunchTo& st) { return launch_slots_t<5, 1>(a, streamed, st); }

}  // namespace srd
