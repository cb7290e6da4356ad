// Which calls k_assemble_slots (sr_slots.h) takes, and its instantiation for one.
#include "sr_launch.h"

namespace srd {

hipError_t launch_slots_k3c1(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k3c3(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k5c1(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k5c3(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k7c1(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k7c3(const AssembleArgs& a, bool streamed, const LaunchTo& st);

// Up to 128 folded atoms, one to three channels, every atom's coefficients of an image within 4 GB, rows of at least one word of
// coefficients; the generic kernel takes what is left.
bool slots_supported(const AssembleArgs& a, int k) {
    const int cb = a.coeff_dtype == SR_F32 ? 4 : (a.coeff_dtype == SR_F8E4M3 ? 1 : 2);
    if ((k != 3 && k != 5 && k != 7) || a.C < 1 || a.C > 3 || a.n_fold < 1 || a.n_fold > 128 || a.pixel_major || a.blocked) return false;
    // Few atoms: the generic kernel's time grows with them, this one's hardly below the 32 that its smallest instantiation
    // folds.  Before the pixel-shuffle, generic / this, us: 1060 x 1020 x1 fp32 5x5 14 atoms 34 / 39, 24 atoms 55 / 39; 7x7 24 atoms 64 / 65;
    // x3 fp8 5x5 24 atoms 52 / 54, 7x7 24 atoms 72 / 82, 3x3 14 atoms 33 / 34; bfloat16 5x5 6 atoms 29 / 36, 14 atoms 40 / 36.
    if (!a.logits && a.n_fold <= (a.coeff_dtype == SR_F32 ? (k == 7 ? 26 : k == 3 ? 22 : 16)
                                  : a.coeff_dtype == SR_F8E4M3 ? (a.C == 1 ? 10 : k == 3 ? 14 : k == 5 ? 25 : 32) : 12)) return false;
    // 7x7 atoms before the pixel-shuffle, beyond small frames: the two blocks of matrix instructions of every slot and the wide tiles
    // cost more than the generic kernel's fold until there are many atoms.  1350 thousand pixels x3 fp8 33 atoms 121 / 252, 60 atoms 189 /
    // 252, all of 128 390 / 279; fp32 33 atoms 124 / 165, 60 atoms 195 / 164, 80 atoms 255 / 266; but 103 thousand fp8 33 atoms 32 / 25.
    if (!a.logits && a.pre_shuffle && k == 7 && (long long)a.N * a.H * a.W > 150000) {
        if (a.coeff_dtype == SR_F8E4M3 && a.C != 1 && a.n_fold <= 90) return false;
        if (a.coeff_dtype == SR_F32 && (a.n_fold <= 48 || (a.C != 1 && a.n_fold > 72 && a.n_fold <= 84))) return false;
    }
    if (a.logits && (a.n_fold != a.L || a.coeff_dtype == SR_F8E4M3)) return false;
    if ((a.pre_shuffle ? a.w : a.W) < 4 / cb || a.H < 1) return false;
    if ((unsigned long long)a.L * a.H * a.W * cb >= (1ull << 32)) return false;
    if ((unsigned long long)a.C * a.H * a.W * 4ull > 0xffffffc0ull) return false;      // lanes outside the image store from there on
    return true;
}

// Planar coefficients that the streaming kernel has an instantiation for and this one is faster with.  Three reasons:
//   8-bit and fp32 coefficients of more than 72 atoms (and 8-bit ones of 7x7 atoms) fill the register file of a SIMD with one
//   wavefront there, in tiles of sixteen rows; here two or three share it and a small frame is cut finer.  Streaming / this, us: fp8 100
//   atoms 162 x 108 x3 21 / 10, 1548 x 1032 x3 86 / 58, 2112 x 1416 x3 125 / 102; fp32 100 atoms 162 x 108 x1 27 / 9, 1096 x 724 x3
//   114 / 97; fp8 7x7 164 x 108 x3 23 / 14, 824 x 548 x3 27 / 30; fp32 7x7 100 atoms 1096 x 724 x1 158 / 150, 1548 x 1032 x1
//   272 / 296.
//   fp32 coefficients of a few hundred units of sixteen rows, whose fullest SIMD has four and here two or three: 366 x 243 x3 18 /
//   14.5, 464 x 308 x3 21 / 18.5, but 548 x 364 x3 23 / 23.5; between 32 and 64 thousand pixels the streaming kernel's 64 x 4 tiles are as
//   good.
//   16-bit coefficients of one channel and of the smallest frames, for the same reason (few instantiations have tiles of four rows): 5x5
//   72 atoms fp16 546 x 363 x1 14 / 12.4, 162 x 108 x1 9 / 8, 3x3 162 x 108 x3 9 / 8.2; 128 atoms 456 x 327 x1 17 / 16, but at scale 4 516 x 384 x1 17 / 18; 7x7 363 x 243 x1
//   12 / 10, but 546 x 363 x1 14 / 14.7.
//   16-bit coefficients in rows that start on no multiple of 32 bytes (of 64 bytes: no difference): neighbouring pieces share memory lines, which the streaming
//   loads there take from memory twice and the ordinary ones here once: 3x3, 72 atoms, 822 x 548 x3
//   28 / 24, 5x5 669 x 441 x1 18 / 14.5; 128 atoms 1554 x 1030 x3 119 / 102; with whole lines 794 / 800 thousand pixels 32 / 35, 3 million 91 /
//   104.  3x3 atoms of 128 have no strips there: 540 x 360 x3 37 / 30.
bool slots_faster(const AssembleArgs& a, int k) {
    if (a.pre_shuffle || a.pixel_major || a.blocked || a.logits || a.C == 2 || !slots_supported(a, k)) return false;
    if (a.n_fold > 72 && k != 7 && (a.coeff_dtype == SR_F8E4M3 || a.coeff_dtype == SR_F32)) return true;      // (none is built there)
    if (a.W < 100) return false;                       // its planar tiles have 128 columns
    const long long px = (long long)a.N * a.H * a.W;
    const int n = a.n_fold;
    if (a.coeff_dtype == SR_F8E4M3) return k == 7 && (px <= 250000 || (a.C == 1 && n <= 72 && px > 700000));
    if (a.coeff_dtype == SR_F32) {
        if (n > 72) return px <= 700000;
        return px <= 32768 || (px > 65536 && px <= (k != 7 ? 170000 : a.C == 1 ? 150000 : 110000));
    }
    const bool f16 = a.coeff_dtype == SR_F16;
    if (a.C == 1 && (k == 3 ? n > 32 && px <= 320000 : k == 7 ? n > 16 && a.s != 4 && px <= 100000 : n > 72 ? a.s != 4 && px <= 160000 : n > 48 && f16 && px <= 320000)) return true;
    if (px <= 32768 && f16 && k == 3 && n > 32) return true;
    const bool shared_lines = (long long)a.W * 2 % 32 != 0;
    if (k == 3 && n > 72) return shared_lines || px <= 500000;
    if (k == 7 || !shared_lines) return false;
    if (n > 72) return px > 350000 || (px > 180000 && (a.s == 4 || px < 250000));
    // (5x5 atoms, three channels, up to 72 atoms: the streaming kernel takes them in several storage orders and gives the same bits in all)
    return (k == 3 ? n > 32 : a.C == 1 && n > 48 && f16) && px > 180000 && px <= 600000 && (a.s != 4 || px <= 320000);
}

hipError_t launch_slots(const AssembleArgs& a, int k, bool streamed, const LaunchTo& st) {
    switch (k) {
    case 3:  return a.C == 1 ? launch_slots_k3c1(a, streamed, st) : launch_slots_k3c3(a, streamed, st);
    case 5:  return a.C == 1 ? launch_slots_k5c1(a, streamed, st) : launch_slots_k5c3(a, streamed, st);
    case 7:  return a.C == 1 ? launch_slots_k7c1(a, streamed, st) : launch_slots_k7c3(a, streamed, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace srd
