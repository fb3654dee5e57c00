// Packing of bf16 3x3(x3) weights for the matrix-core convolutions: device code, launched by itself (conv_mfma.hip) or together
// with a halo exchange (index_kernels.hip).
#pragma once
#include "conv_mfma_common.h"

namespace sp3d {

struct PackArgs {
    const uint16_t *w;
    uint4 *wpack;
    int nci, nco, ntap, dgrad;
};

namespace convk {

// Pre-swizzle the weights into MFMA A-fragment order.  wpack[chunk i][block j][tap][half][lane] = the 8
// input channels k = 32i + 16*half + 8*(lane/32) + e of output channel m = 32j + lane%32.
// Forward reads w[tap][k][m]; data-grad reads w[26-tap][m][k] (taps mirrored, roles swapped), where
// the kernel's input channels are the layer's output channels.  ki / ko = channel counts as the
// kernel sees them (ki in, ko out).  The 2-D variant's nine taps w[3][3][..][..] sit in the slots 9 .. 17 (kd = 1);
// its other slots are never loaded and stay unwritten.
// A wave packs the two fragments of one (chunk, block, tap), a 32 x 32 square of w, neighbouring waves neighbouring
// blocks, so that the 64-byte rows of four waves are one run of memory.  In the data gradient's order a lane's eight
// values lie side by side; the forward order is transposed in LDS, rows 34 elements apart so that the eight reads of
// a lane and those of its 31 neighbours fall into different banks.  What bounds it: HBM for wide layers (one pass over
// w, one over wpack), the launch for narrow ones.  (One thread per element, 2-byte loads kilobytes apart, 27 slots
// also in 2-D, took four times as long: 1024 -> 1024 channels, 2-D, 39 -> 9.1 us (18.9 MB in, as much out: 4.1 TB/s), 512
// -> 512 12.8 -> 5.6 us; 3-D 1024 -> 1024 21.7 us (5.2 TB/s); a launch alone is 4 us.)
constexpr int kPackWaves = 4, kPackRow = 34;
using PackSquares = uint16_t[kPackWaves][C * kPackRow];
inline unsigned pack_blocks(const PackArgs &a) { return static_cast<unsigned>((a.nci * a.nco * a.ntap + kPackWaves - 1) / kPackWaves); }
__device__ __forceinline__ void pack_weights(const PackArgs &a, unsigned block, PackSquares &square) {
    const int nci = a.nci, nco = a.nco, ntap = a.ntap;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int id = block * kPackWaves + wave;
    const bool real = id < nci * nco * ntap;
    const int u = real ? id : 0;
    const int cj = u % nco, t = (u / nco) % ntap, ci = u / (nco * ntap);
    const int ki = C * nci, ko = C * nco;
    uint4 *dst = a.wpack + (static_cast<size_t>(ci * nco + cj) * NFRAG + 2 * (t + (ntap == 9 ? 9 : 0))) * 64 + lane;
    if (a.dgrad) {
        const uint16_t *src = a.w + (static_cast<size_t>(ntap - 1 - t) * ko + C * cj + (lane & 31)) * ki + C * ci + 8 * (lane >> 5);
        const uint4 v0 = *reinterpret_cast<const uint4 *>(src), v1 = *reinterpret_cast<const uint4 *>(src + 16);
        if (real) {
            dst[0] = v0;
            dst[64] = v1;
        }
        return;
    }
    const uint16_t *src = a.w + (static_cast<size_t>(t) * ki + C * ci + (lane >> 2)) * ko + C * cj + 8 * (lane & 3);
    uint16_t *sq = square[wave];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint4 v = *reinterpret_cast<const uint4 *>(src + static_cast<size_t>(16 * i) * ko);
        uint32_t *d = reinterpret_cast<uint32_t *>(sq + (16 * i + (lane >> 2)) * kPackRow + 8 * (lane & 3));
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    }
    __syncthreads();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const uint16_t *col = sq + (16 * half + 8 * (lane >> 5)) * kPackRow + (lane & 31);
        uint32_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = col[2 * e * kPackRow] | static_cast<uint32_t>(col[(2 * e + 1) * kPackRow]) << 16;
        if (real) dst[64 * half] = make_uint4(v[0], v[1], v[2], v[3]);
    }
}

}  // namespace convk
}  // namespace sp3d
