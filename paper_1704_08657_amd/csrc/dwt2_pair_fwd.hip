// Several levels in one launch, one direction (kForward); see dwt2_pair.inl.
#include "dwt2_pair.inl"

namespace dwt2 {

hipError_t launch_pair_fwd(Wavelet wav, Dtype dt, int levels, const PairParams& p, int planes, hipStream_t s) {
    return kern::pair::launch_dir<kForward>(wav, dt, levels, p, planes, s);
}

}  // namespace dwt2
