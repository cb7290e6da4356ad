// Host-side launch entry points of the individual kernel families.
#pragma once
#include <hip/hip_runtime.h>
#include "sr_device.h"

namespace srd {

// ---------------------------------------------------------------------------
// Host side: launch of one instantiation on a persistent grid.
// ---------------------------------------------------------------------------
// CUs of the current device (asked once per device and thread)
inline int compute_units() {
    static thread_local int known[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (known[dev] == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
        known[dev] = cus;
    }
    return known[dev];
}
inline int units_of(const AssembleArgs& a) { return a.cus ? a.cus : compute_units(); }

hipError_t launch_generic(const AssembleArgs& a, int k, bool io_f16, hipStream_t st);   // coefficient dtype: a.coeff_dtype
hipError_t launch_bicubic(const BicubicArgs& a, bool in_f16, bool out_f16, hipStream_t st);

// How a matrix-core launch walks the images: 1 = tiles, 2 = strips (0: not said); HR columns x rows of a tile or of a strip's segment;
// how many there are; workgroups, and wavefronts of each (a tile belongs to a workgroup, a segment to a wavefront).
struct Walk { int form, width, rows, pieces, workgroups, waves; };
// Where such a launch goes: to a stream, or (walk given) nowhere: the walk is written down instead.
struct LaunchTo {
    hipStream_t stream;
    Walk* walk;
    LaunchTo(hipStream_t st) : stream(st), walk(nullptr) {}
    explicit LaunchTo(Walk* w) : stream(nullptr), walk(w) {}
};

// Matrix-core kernel.  mfma_supported() is a pure host-side predicate.
bool mfma_supported(const AssembleArgs& a, int k, int coeff_dtype, int tile);
int mfma_capacity(const AssembleArgs& a, int k);        // of the instantiation that takes the call, in groups of 8 atoms
hipError_t launch_mfma(const AssembleArgs& a, int k, bool io_f16, int tile, const LaunchTo& st);
// Matrix-core kernel for calls the one above has no instantiation for (coefficient dtype: a.coeff_dtype); make_plan chooses
bool slots_supported(const AssembleArgs& a, int k);
bool generic_faster(const AssembleArgs& a, int k);     // ... but are faster on the generic kernel
bool slots_faster(const AssembleArgs& a, int k);       // ... and those that it has one for but serves slower
hipError_t launch_slots(const AssembleArgs& a, int k, bool streamed, const LaunchTo& st);      // streamed: with the streaming kernel's bits
// Per-pixel list form (sr_dict_assemble_list) on the matrix cores: a.coeff = values, a.index, a.T set; kept = identity.
bool mfma_list_supported(const AssembleArgs& a, int k, bool value_f16);
hipError_t launch_mfma_list(const AssembleArgs& a, const LaunchTo& st);
bool mfma_tile_shape(const AssembleArgs& a, int k, int coeff_dtype, int tile, int* tw, int* th, int* waves = nullptr,
                     int* groups = nullptr);

}  // namespace srd
