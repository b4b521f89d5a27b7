// Several levels in one launch, one direction (kInverse); see dwt2_pair.inl.
#include "dwt2_pair.inl"

namespace dwt2 {

hipError_t launch_pair_inv(Wavelet wav, Dtype dt, int levels, const PairParams& p, int planes, hipStream_t s) {
    return kern::pair::launch_dir<kInverse>(wav, dt, levels, p, planes, s);
}

}  // namespace dwt2
