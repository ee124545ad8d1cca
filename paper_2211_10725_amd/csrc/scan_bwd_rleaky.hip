// The reverse scan's instantiations for SNN_RLEAKY.
#include "scan_bwd.hpp"

namespace snn {

void scan_bwd_rleaky(int vec, int rs, int gm, int gt, const ScanArgs &a, const BwdBuffers &b,
                     hipStream_t s) {
    bwd_dispatch<SNN_RLEAKY>(vec, rs, gm, gt, a, b, s);
}

}  // namespace snn
