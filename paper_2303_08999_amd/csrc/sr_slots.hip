// Which calls k_assemble_slots (sr_slots.h) takes, and its instantiation for one.
#include "sr_launch.h"

namespace srd {

hipError_t launch_slots_k3c1(const AssembleArgs& a, hipStream_t st);
hipError_t launch_slots_k3c3(const AssembleArgs& a, hipStream_t st);
hipError_t launch_slots_k5c1(const AssembleArgs& a, hipStream_t st);
hipError_t launch_slots_k5c3(const AssembleArgs& a, hipStream_t st);
hipError_t launch_slots_k7c1(const AssembleArgs& a, hipStream_t st);
hipError_t launch_slots_k7c3(const AssembleArgs& a, hipStream_t st);

// Up to 128 folded atoms, one to three channels, every atom's coefficients of an image within 4 GB, rows of at least one word of
// coefficients; the generic kernel takes what is left.
bool slots_supported(const AssembleArgs& a, int k) {
    const int cb = a.coeff_dtype == SR_F32 ? 4 : (a.coeff_dtype == SR_F8E4M3 ? 1 : 2);
    if ((k != 3 && k != 5 && k != 7) || a.C < 1 || a.C > 3 || a.n_fold < 1 || a.n_fold > 128 || a.pixel_major || a.blocked) return false;
    // Few atoms: the generic kernel's time grows with them, this one's hardly below the 32 that its smallest instantiation
    // folds.  Before the pixel-shuffle, generic / this, us: 1060 x 1020 x1 fp32 5x5 14 atoms 34 / 39, 24 atoms 55 / 39; 7x7 24 atoms 64 / 65;
    // x3 fp8 5x5 24 atoms 52 / 54, 7x7 24 atoms 72 / 82, 3x3 14 atoms 33 / 34; bfloat16 5x5 6 atoms 29 / 36, 14 atoms 40 / 36.
    if (!a.logits && a.n_fold <= (a.coeff_dtype == SR_F32 ? (k == 7 ? 26 : 16)
                                  : a.coeff_dtype == SR_F8E4M3 ? (a.C == 1 ? 10 : k == 3 ? 14 : k == 5 ? 25 : 32) : 12)) return false;
    if (a.logits && (a.n_fold != a.L || a.coeff_dtype == SR_F8E4M3)) return false;
    if ((a.pre_shuffle ? a.w : a.W) < 4 / cb || a.H < 1) return false;
    if ((unsigned long long)a.L * a.H * a.W * cb >= (1ull << 32)) return false;
    if ((unsigned long long)a.C * a.H * a.W * 4ull > 0xffffffc0ull) return false;      // lanes outside the image store from there on
    return true;
}

hipError_t launch_slots(const AssembleArgs& a, int k, hipStream_t st) {
    switch (k) {
    case 3:  return a.C == 1 ? launch_slots_k3c1(a, st) : launch_slots_k3c3(a, st);
    case 5:  return a.C == 1 ? launch_slots_k5c1(a, st) : launch_slots_k5c3(a, st);
    case 7:  return a.C == 1 ? launch_slots_k7c1(a, st) : launch_slots_k7c3(a, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace srd
