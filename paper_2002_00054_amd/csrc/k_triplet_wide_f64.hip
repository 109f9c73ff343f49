// Instantiation of the pair/triplet kernels for one arithmetic form, tables
// with wide angular functions.
#include "kernels.h"
#include "k_triplet.inc"

namespace nnp {
template void launch_triplet_wide<P_FP64>(int, int, const TripArgs<P_FP64>&, hipStream_t);
}  // namespace nnp
