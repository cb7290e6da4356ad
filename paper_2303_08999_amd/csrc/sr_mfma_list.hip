// Matrix-core kernel instantiations for coefficients given as per-pixel lists (CT_LIST8 / CT_LIST16 in
// sr_mfma_kernel.h; an extension beyond the paper, see sr_dict_assemble_list): 5x5 atoms, three
// channels, fp16 values, up to 72 or up to 128 atoms in the dictionary, up to 8 or up to 16 entries per pixel.
#include "sr_mfma_kernel.h"

namespace srd {

bool mfma_list_supported(const AssembleArgs& a, int k, bool value_f16) {
    if (k != 5 || a.C != 3 || !value_f16 || a.L > 128 || a.T < 1 || a.T > LIST_MAX_ENTRIES) return false;
    if (a.W < 4 || a.W % 4 != 0 || a.H < 1) return false;
    if ((unsigned long long)a.T * a.H * a.W >= (1ull << 32)) return false;             // 32-bit element offsets within an image
    if ((unsigned long long)a.C * a.H * a.W * 4ull >= (1ull << 32)) return false;
    return true;
}

// Up to 72 atoms: the dense form's operand steps (four of 16 atoms and one of 8); scale 4 in strips, scale 3 in strips or 128 x 8
// tiles, scale 2 in 128 x 8 tiles, but frames of at most one row for every SIMD in strips: rows of four wavefronts each instead of a few tiles of
// eight (tiles / strips, us, lists of 1 to 16: 16 thousand pixels 11.2 / 9.4, 101 thousand 11.5 / 9.7, 60 drawn calls 1.18 to 1.26 there).  Larger ones would need two of
// these workgroups on a CU, whose LDS (86 KB each) does not fit: 128 thousand pixels 11.5 / 17.2, 1905 thousand 49 / 55.  Up to 128: eight steps, 128 x 8 tiles at every scale (35 KB of scatter scratch).  Lists of up to 8
// entries keep half the registers.
// Scale 4 in one run of three forms, lists of 8 (us, 128 x 16 tiles with the scale-4 footprint / 128 x 8 / strips):
// 240 x 320 15.4 / - / 9.3, 480 x 640 16.3 / 14.4 / 13.7, 720 x 1280 22.0 / 25.4 / 21.1, 800 x 1200 22.7 / 25.5 /
// 21.4, 4K 142.2 / - / 107.5, 32 images of 128 x 192 21.5 / 24.8 / 21.0; no size was found where tiles are faster,
// also not where strips leave the fullest SIMD as many rows.
template <int CT>
static hipError_t launch_ct(const AssembleArgs& a, const LaunchTo& st) {
    if (a.L <= 72) {
        if (a.s == 4) return launch_one<5, 3, 9, 4, 1, 4, 1, 2, CT, 4, false, 0, 4>(a, st);
        if (a.s == 3 && strip_form(a, 0, 128, 128, 8)) return launch_one<5, 3, 9, 4, 1, 4, 1, 2, CT, 3, false, 0, 3>(a, st);
        if (a.s == 2 && (a.W + 127ll) / 128 * a.H * a.N <= 4ll * units_of(a)) return launch_one<5, 3, 9, 4, 1, 4, 1, 1, CT, 2, false, 0, 2>(a, st);
        return launch_one<5, 3, 9, 4, 1, 4, 2, 2, CT, 2>(a, st);
    }
    return launch_one<5, 3, 16, 4, 1, 4, 2, 2, CT, 2>(a, st);
}

hipError_t launch_mfma_list(const AssembleArgs& a, const LaunchTo& st) {
    return a.T <= 8 ? launch_ct<CT_LIST8>(a, st) : launch_ct<CT_LIST16>(a, st);
}

}  // namespace srd
