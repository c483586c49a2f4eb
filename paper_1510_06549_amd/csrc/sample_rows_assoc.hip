// sample_rows_assoc.hip -- the sampler over weight rows for the model with word
// associations: its instances of the kernel in sample_rows.hpp.
#include "sample_rows.hpp"

namespace spdp {

hipError_t launch_sample_rows_assoc(const RowArgs &A, int lanes, int kpl, hipStream_t st)
{
    switch (lanes) {
    case 16: return launch_rows_lanes<16, true>(A, kpl, st);
    case 32: return launch_rows_lanes<32, true>(A, kpl, st);
    default: return launch_rows_lanes<64, true>(A, kpl, st);
    }
}

}  // namespace spdp
