// The reverse scan's instantiations for SNN_LEAKY.
#include "scan_bwd.hpp"

namespace snn {

void scan_bwd_leaky(int vec, int rs, int gm, int gt, const ScanArgs &a, const BwdBuffers &b,
                    hipStream_t s) {
    bwd_dispatch<SNN_LEAKY>(vec, rs, gm, gt, a, b, s);
}

}  // namespace snn
