// Instantiation of the pair/triplet kernels for one arithmetic form, tables
// with wide angular functions.
#include "kernels.h"
#include "k_triplet.inc"

namespace nnp {
template void launch_triplet_wide<P_FP32>(int, int, const TripArgs<P_FP32>&, hipStream_t);
}  // namespace nnp
