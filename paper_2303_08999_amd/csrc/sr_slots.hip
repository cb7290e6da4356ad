// Which calls k_assemble_slots (sr_slots.h) takes, and its instantiation for one.
#include "sr_launch.h"
#include "sr_mfma_kernel.h"

namespace srd {

hipError_t launch_slots_k3c1(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k3c3(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k5c1(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k5c3(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k7c1(const AssembleArgs& a, bool streamed, const LaunchTo& st);
hipError_t launch_slots_k7c3(const AssembleArgs& a, bool streamed, const LaunchTo& st);

// Few atoms: the generic kernel's time grows with them, this one's hardly below the 32 that its smallest instantiation
// folds.  Before the pixel-shuffle, generic / this, us: 1060 x 1020 x1 fp32 5x5 14 atoms 34 / 39, 24 atoms 55 / 39; 7x7 24 atoms 64 / 65;
// planar 881 thousand x2 fp32 18 atoms 34 / 42; x3 fp8 5x5 24 atoms 52 / 54, 7x7 24 atoms 72 / 82, 3x3 248 thousand 16 atoms 10.7 / 14;
// bfloat16 x1 5x5 6 atoms 29 / 36, 14 atoms 40 / 36; fp16 x2 5x5 323 thousand 13 atoms 15 / 22.  Logits (800 drawn calls of 1 to 28
// atoms; generic over this): one channel up to 8 atoms 0.5 .. 1.07, 9 atoms 1.0 .. 1.33; two and three up to 11 atoms (3x3 12, 7x7 14)
// 0.5 .. 1.33, from there 0.9 .. 2.
static bool few_atoms(const AssembleArgs& a, int k) {
    const int n = a.n_fold;
    if (a.logits) return n <= (a.C == 1 ? 8 : k == 3 ? 12 : k == 5 ? 11 : 14);
    if (a.coeff_dtype == SR_F32) return n <= (k == 7 ? 26 : k == 3 ? 22 : a.C == 1 ? 16 : 20);
    if (a.coeff_dtype == SR_F8E4M3) return n <= (a.C == 1 ? (k == 3 ? 14 : 10) : k == 3 ? 24 : k == 5 ? 25 : 32);
    return n <= (a.C == 1 ? 12 : 16);
}

// Up to 128 folded atoms, one to three channels, every atom's coefficients of an image within 4 GB, rows of at least one word of
// coefficients; the generic kernel takes what is left.
bool slots_supported(const AssembleArgs& a, int k) {
    const int cb = a.coeff_dtype == SR_F32 ? 4 : (a.coeff_dtype == SR_F8E4M3 ? 1 : 2);
    if ((k != 3 && k != 5 && k != 7) || a.C < 1 || a.C > 3 || a.n_fold < 1 || a.n_fold > 128 || a.pixel_major || a.blocked) return false;
    if (a.logits && (a.n_fold != a.L || a.coeff_dtype == SR_F8E4M3)) return false;
    if ((a.pre_shuffle ? a.w : a.W) < 4 / cb || a.H < 1) return false;
    if ((unsigned long long)a.L * a.H * a.W * cb >= (1ull << 32)) return false;
    if ((unsigned long long)a.C * a.H * a.W * 4ull > 0xffffffc0ull) return false;      // lanes outside the image store from there on
    if ((long long)a.N * a.H * ((a.W + 31) / 32) > 0x3fffffffLL) return false;         // tiles are counted in 32 bits
    return !few_atoms(a, k);
}

// The calls among them that the generic kernel serves faster: its fold grows with the atoms, this kernel's in steps (32, 72, 128), and
// beyond small frames the filtering and the wide tiles weigh.  Generic / this, us:
//   7x7 before the pixel-shuffle, x3 fp8 1350 thousand pixels 33 atoms 121 / 252, 60 atoms 189 / 252, all of 128 390 / 279, 337 thousand
//   97 atoms 92 / 110, 95 thousand at scale 3 36 atoms 23 / 44, but 103 thousand 33 atoms 32 / 25; fp32 1350 thousand 33 atoms 124 / 165, 60 atoms
//   195 / 164, 80 atoms 255 / 266; planar 560 thousand x2 fp32 28 atoms 45 / 49; 319 thousand x2 bfloat16 33 atoms 33 / 36.
//   fp32 just above 32 atoms: 3x3 1615 thousand x3 37 atoms 74 / 108, 196 thousand x1 33 atoms 18 / 21, 924 thousand x3 40 atoms
//   0.96 of each other, but 63 thousand 40 atoms 1.07; 5x5 283 thousand x2 34 atoms 24 / 26, 1638 thousand x2 40 atoms 99 / 118.
bool generic_faster(const AssembleArgs& a, int k) {
    const long long px = (long long)a.N * a.H * a.W;
    const int n = a.n_fold;
    if (a.logits) return false;
    if (k == 7) {
        if (a.coeff_dtype == SR_F32) return px > 150000 && (n <= 48 || (a.pre_shuffle && a.C != 1 && n > 72 && n <= 84));
        if (!a.pre_shuffle || a.C == 1) return false;
        return a.coeff_dtype == SR_F8E4M3 ? n <= 100 && px > (a.s == 3 ? 25000 : 110000) : n > 32 && n <= 36 && px > 150000;
    }
    return a.coeff_dtype == SR_F32 && px > 120000 && n > 32 && n <= (k == 3 || a.C != 1 ? 42 : 36);
}

// Before the pixel-shuffle the streaming kernel's forms have tiles of 128 x 16 (scale 2), 384 x 8 (3) and 256 x 8 (4) only, so small frames leave most
// CUs idle, and where the LR width is no multiple of 4 (but the HR width is) it loads element by element.  `ratio` as in slots_faster, of whole tiles; limits from 160 drawn
// calls of 16 thousand to 2.2 million pixels (fp16 and bfloat16, 65 to 72 atoms, rotating inputs; same bits in all).  Streaming / this, us:
//   element by element, always: x2 102 thousand pixels 30.1 / 14.7, 659 thousand 90 / 38, x4 17 thousand 29.4 / 11.5, 751 thousand 104 / 45.
//   from a ratio of 1.6 on: x2 16 thousand 23.6 / 10.4, 161 thousand 25.2 / 18.1, 626 thousand 43.9 / 34.0; x3 20 thousand 19.4 / 10.5, 178 thousand 24.8 / 19.2,
//   344 thousand 24.3 / 24.1; x4 18 thousand 22.0 / 10.9, 126 thousand 24.0 / 15.2.  Below: x2 0.90 to 1.22 of each other, x3 0.78 to 1.03, x4 0.83 to 1.06,
//   but scales 2 and 4 in one tile for a CU at most from 1.33 on 1.08 to 1.27 (x4 337 thousand 22.7 / 21.0, x2 278 thousand 25.7 / 20.3).
static bool pre_shuffle_faster(const AssembleArgs& a, int k) {
    if (a.w % 4 != 0) return true;
    Walk s, t;
    if (launch_mfma(a, k, a.io_f16, 0, LaunchTo(&s)) != hipSuccess || launch_slots(a, k, true, LaunchTo(&t)) != hipSuccess) return false;
    const long long cus = units_of(a);
    const long long there = (s.pieces + cus - 1) / cus * s.width * s.rows, here = (t.pieces + cus - 1) / cus * t.width * t.rows;
    return 10 * there >= 16 * here || (a.s != 3 && s.pieces <= cus && 100 * there >= 133 * here);
}

// Coefficients that the streaming kernel has an instantiation for and this one is faster with (and gives the same bits).  Planar ones: both launches are
// known before either is made, and what decides is the work of the fullest CU.  Counted in pixels: those of its tiles or of its
// wavefronts' strip segments, plus 9 for each of the k - 1 rows that a tile, or each wavefront's segment, up-samples beyond its own
// (per 128 columns), plus 24 for what a tile costs whatever its size.  `ratio` is the streaming kernel's count over this one's.  The limits were
// read off 2401 drawn calls of 2 thousand to 4 million pixels, timed on both in turn with rotating inputs (in brackets: streaming us /
// this us of the calls from the limit on, smallest .. largest; with them the drawn calls take 0.84 of the streaming kernel's time, geometric mean):
//   tiles of one or two rows, in one round: 1.03 (0.91 .. 1.6), 3x3 0.97 (0.94 .. 1.4).  For more than 72 atoms, which take two pixels per lane there, 0.86
//   (0.96 .. 2.1); 7x7 in one channel 0.88 (1.0 .. 1.6), in three 1.06, 1.03 for more than 72 (0.96 .. 1.3).
//   tiles of four and eight rows: 1.13 (1.02 .. 1.4); from 0.9 to there 0.7 .. 1.15: strips win the large frames.
//   16-bit rows that start on no multiple of 32 bytes, whose shared lines the streaming kernel takes twice unless keep_lines holds: 3x3, launches of one round, 1.04 (0.97 ..
//   1.4), three channels at scales 2 and 3 0.97 (0.93 .. 1.4); more than 72 atoms of 5x5 0.855 (0.92 .. 1.5), but frames of few
//   tiles at scale 4, where the streaming tiles are larger: 1.05 (1.02 .. 1.3), against those of 24 rows and three channels 0.72 (0.97 .. 1.26).
//   Where keep_lines holds (three channels, 2 million pixels and more), up to 104 atoms against strips 1.0 (98 drawn calls from 0.86 to there: 0.80 .. 1.03, mean 0.95: 2080
//   thousand 77 atoms 83 / 103); more atoms 0.89 .. 1.06, mean 0.985, against tiles 0.99 .. 1.10, more than 72 of 3x3 1.01 .. 1.10: as without.
//   More than 72 atoms of 3x3 (no strips there), in tiles of four rows or such rows: 0.95 (0.97 .. 1.7); more than 72 of fp32 (one wavefront per
//   SIMD, tiles of sixteen rows): 0.925 in tiles of four and eight rows, 0.95 in lower ones (0.94 .. 3.2), 7x7 0.76 (0.95 .. 3.2).
//   fp32 atoms of 7x7, 27 to 32 of them, in the streaming kernel's capacity of 72: 0.85 (1.4 .. 1.9).
//   One tile for a CU at most: always (1.0 .. 3.2).  8-bit coefficients of 7x7, and of more than 72 atoms: always (0.96 .. 2.3).
//   5x5 atoms of three channels up to 72 in 16 bits (430 drawn calls of their own, the same bits in all; sr_dict_assemble_tile keeps saying the streaming
//   kernel's tile 0): against tiles of 128 x 4 1.1 (1.01 .. 1.27: 21 thousand pixels 10.5 / 8.2, 57 thousand 9.7 / 8.9, 175 thousand 14.2 / 12.3; 2 thousand 8.9 / 8.4,
//   below that 8.4 to 9.2 / 8.2 to 8.6, the launch alone: not taken), and in a
//   second round there 0.995 (1.05 .. 1.2: 298 thousand 19.4 / 16.2; in one round 512 x 512 13.2 / 15.0 from the memory-side cache, 17.9 / 16.1 from memory);
//   against taller tiles 1.2 (1.08 .. 1.28); against strips nowhere (0.78 .. 1.1).  8-bit ones gain 3 % there or lose.
// Left out otherwise: capacities that this kernel has not (5x5: 8, 16 and 48; 3x3: 8).
bool slots_faster(const AssembleArgs& a, int k) {
    if (a.pixel_major || a.blocked || a.logits || a.C == 2 || !slots_supported(a, k)) return false;
    if (a.pre_shuffle) return pre_shuffle_faster(a, k);
    const int n = a.n_fold, built = n <= 32 ? 4 : n <= 72 ? 9 : 16, streaming = mfma_capacity(a, k);
    if (a.coeff_dtype == SR_F8E4M3) return k == 7 || n > 72;               // (of more than 72 atoms of 3x3 and 5x5 none is built there)
    const bool f32 = a.coeff_dtype == SR_F32;
    const bool common = k == 5 && a.C == 3 && n <= 72 && !f32;
    const long long cus = units_of(a);
    if (!common && (a.W + 127ll) / 128 * a.H * a.N <= cus) return true;    // (single rows)
    if (!common && built > streaming) return false;
    Walk s, t;
    if (launch_mfma(a, k, a.io_f16, 0, LaunchTo(&s)) != hipSuccess || launch_slots(a, k, true, LaunchTo(&t)) != hipSuccess) return false;
    // in half pixels
    const long long halo = 18ll * (k - 1), fixed = 48, wide = 2ll * s.width * s.rows + halo * s.width / 128;
    const long long there = s.form == 1 ? (s.pieces + cus - 1) / cus * (wide + fixed)
                                        : ((s.pieces + s.waves - 1) / s.waves + cus - 1) / cus * s.waves * wide;
    const int width = f32 && t.rows >= 4 && a.W < 128 ? (a.W + 31) / 32 * 32 : 128;      // (a narrow image: its units only)
    const long long here = (t.pieces + cus - 1) / cus * (2ll * width * t.rows + halo * width / 128 + fixed);
    if (common) return s.form == 1 && (long long)a.N * a.H * a.W >= 2048 && 1000 * there >= (s.rows > 4 ? 1200 : t.rows == 4 && s.pieces > 2 * cus ? 995 : 1100) * here;
    const bool shared_lines = !f32 && a.W % 16 != 0, many = n > 72;
    const int limit = built < streaming                       ? 850         // thousandths
                      : many && f32                           ? (k == 7 ? 760 : t.rows >= 4 ? 925 : 950)
                      : t.rows <= 2 && (many || k == 7 || t.pieces <= 3 * cus) ? (k == 7 && a.C == 3 ? (many ? 1030 : 1060) : many ? 860 : k == 7 ? 880 : k == 3 ? 970 : 1030)
                      : many && k == 3 && (shared_lines || t.rows == 4) ? 950
                      : shared_lines && many && k == 5        ? (n <= 104 && s.form == 2 && keep_lines(a, k, false) ? 1000 : a.s == 4 && t.pieces <= 2 * cus ? (s.rows == 24 && a.C == 3 ? 720 : 1050) : 855)
                      : shared_lines && k == 3 && t.pieces <= 3 * cus ? (a.C == 3 && a.s != 4 && t.pieces <= 2 * cus ? 970 : 1040)
                                                              : 1130;
    return 1000 * there >= limit * here;
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
