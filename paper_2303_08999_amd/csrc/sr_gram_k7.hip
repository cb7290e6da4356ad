// k_atom_gram_split for 7x7 atoms (sr_gram.h)
#include "sr_gram.h"

namespace gram {

hipError_t launch_split_k7(const GramArgs& a, int coeff_dtype, unsigned long long items, int grid, hipStream_t st) {
    return launch_split_k<7>(a, coeff_dtype, items, grid, st);
}

}  // namespace gram
