// The two-chunk kernels on ragged patches in 3-D (conv_mfma_pair_kernel.h, Ragged in conv_mfma_common.h), in a translation unit of
// their own for the build's sake.
#include "conv_mfma_pair_kernel.h"

namespace sp3d {

using namespace convk;

using PairKern = void (*)(ConvArgs);

const PairKern (&conv_mfma_pair_table_ragged())[4][2][5] {
    static const PairKern k[4][2][5] = SP3D_CONV_TABLE(wide::conv_mfma_pair_kernel, kRagged3, kMaskBits, kReluBits);
    return k;
}

}  // namespace sp3d
