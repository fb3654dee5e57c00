// bf16 forward convolution of a first layer with 2 ... 8 input channels (a multi-phase scan, a slab of slices), kernel 3x3x3
// or 3x3 (2-D variant), output channels in multiples of 32, on v_mfma_f32_32x32x16_bf16.
//
// Padding the channels to 32 (chan_pad.hip) makes a copy of the input ten times its size and the matrix cores do as many
// products with zeros.  Here K runs over (kw, channel) of one kernel row: records of CS = 4 (up to four channels) or 8
// channels lie side by side in LDS, so that the three taps of a kernel row are one run of 12 or 24 values: one MFMA (CS = 4)
// or two (CS = 8) per kernel row and 32 voxels, their unused K slots zero in both operands.  A workgroup stages the records
// of a brick of 4 x 4 x 32 output voxels with its surround; wave w computes slice w, two rows at a time; the weight
// fragments of its 32 output channels stay in registers over all the bricks it visits.  Records are 8 or 16 bytes: 20 KB
// of LDS at most, several workgroups per compute unit hide each other's loads.
// What bounds it: the staging's 2-byte loads and their latency, then the stores of the result (HBM).
// Measured, zero-padded copies -> this kernel with the loads of a brick waited for in place: 3 -> 32 channels on 99 x 156 x
// 210 270 -> 144 us (its 227 MB: 35 us), 5 -> 32 on 16 slices of 512 x 512 320 -> 118 us.  With a brick's records on their
// way during the products of the one before it, that 3-D level (both layers, forward and backward) 1360 -> 1324 us.
#include "conv_mfma_common.h"

namespace sp3d {

using namespace convk;

namespace {

constexpr int kFewThreads = 256, BD = 4, BH = 4, BW = 32;

struct FewArgs {
    const uint16_t *in, *w;
    const float *bias;
    uint16_t *out;
    Geo g;
    int cout, relu;
    int nd, nh, nw, nbricks;     // bricks that cover the largest output box, per axis and over all tiles
};

template <int CS> struct Rec;
template <> struct Rec<4> { typedef uint32_t type __attribute__((ext_vector_type(2))); };
template <> struct Rec<8> { typedef uint32_t type __attribute__((ext_vector_type(4))); };
union FewFrag { uint32_t w[4]; bf16x8 v; };

template <int CIN, int KD>
__global__ __launch_bounds__(kFewThreads) void conv_few_kernel(FewArgs a) {
    constexpr int OD = KD / 2, RD = BD + 2 * OD, RH_ = BH + 2, RW = BW + 2, NREC = RD * RH_ * RW;
    constexpr int CS = CIN <= 4 ? 4 : 8, NR = 3 * KD, NM = CS / 4;      // channels of a record; kernel rows; MFMAs per row
    constexpr int PER = (NREC + kFewThreads - 1) / kFewThreads, NV = CIN % 2 ? CIN : CIN / 2;   // records per thread, loads per record
    typedef typename Rec<CS>::type rec_t;
    __shared__ rec_t recs[NREC];
    const Geo &g = a.g;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, hi = lane >> 5;
    const int co0 = C * blockIdx.y;

    // weight fragments: lane = output channel, K slot 8 hi + e of MFMA m = value 16 m + 8 hi + e of the kernel row's run
    FewFrag wf[NR][NM];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
                uint32_t v[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int k = 16 * m + 8 * hi + 2 * e2 + i, kw = k / CS, c = k % CS;
                    v[i] = 0;
                    if (kw < 3 && c < CIN) v[i] = a.w[(static_cast<size_t>(3 * r + kw) * CIN + c) * a.cout + co0 + col];
                }
                wf[r][m].w[e2] = v[0] | (v[1] << 16);
            }
    f32x16 init;
#pragma unroll
    for (int e = 0; e < 16; ++e) init[e] = a.bias ? a.bias[co0 + 8 * (e >> 2) + 4 * hi + (e & 3)] : 0.f;

    struct Pos { TileBox bx; long long base; int d0, h0, w0; };
    auto pos_of = [&](int brick) {
        Pos p;
        int t = brick;
        p.w0 = (t % a.nw) * BW; t /= a.nw;
        p.h0 = (t % a.nh) * BH; t /= a.nh;
        p.d0 = (t % a.nd) * BD; t /= a.nd;
        p.bx = tile_box(g, t);
        p.base = static_cast<long long>(t) * g.tile_vox + p.bx.org;
        return p;
    };
    // next brick of this workgroup that its tile's box reaches (nbricks: none)
    auto next = [&](int brick, Pos *p) {
        for (; brick < a.nbricks; brick += gridDim.x) {
            *p = pos_of(brick);
            if (p->d0 < p->bx.bd && p->h0 < p->bx.bh && p->w0 < p->bx.bw) break;
        }
        return brick;
    };
    // The records of a brick, on their way from memory while the brick before it is computed.  Even channel counts are
    // loaded two values at a time (a record starts at a multiple of four bytes).
    uint32_t raw[PER][NV];
    auto load = [&](const Pos &p) {
#pragma unroll
        for (int n = 0; n < PER; ++n) {
            // records beyond what the box's own voxels read are moved to the nearest one inside: they reach no result
            const int rec = min(static_cast<int>(threadIdx.x) + n * kFewThreads, NREC - 1);
            const int i = rec / (RH_ * RW), j = rec / RW % RH_, k = rec % RW;
            const int d = min(p.d0 + i - OD, p.bx.bd - 1 + OD), h = min(p.h0 + j - 1, p.bx.bh), w = min(p.w0 + k - 1, p.bx.bw);
            const uint16_t *src = a.in + (p.base + (1LL * (d + 1) * g.ph + h + 1) * g.pw + w + 1) * CIN;
#pragma unroll
            for (int v = 0; v < NV; ++v) raw[n][v] = CIN % 2 ? src[v] : reinterpret_cast<const uint32_t *>(src)[v];
        }
    };

    Pos p;
    int brick = next(blockIdx.x, &p);
    if (brick >= a.nbricks) return;
    load(p);
    while (brick < a.nbricks) {
        __syncthreads();                              // everybody is done with the previous brick
#pragma unroll
        for (int n = 0; n < PER; ++n) {
            rec_t v;
#pragma unroll
            for (int c = 0; c < CS; c += 2) {
                const uint32_t lo = c < CIN ? raw[n][c % NV] : 0u, hv = c + 1 < CIN ? raw[n][(c + 1) % NV] : 0u;
                v[c / 2] = CIN % 2 ? lo | (hv << 16) : (c < CIN ? raw[n][(c / 2) % NV] : 0u);
            }
            if (threadIdx.x + n * kFewThreads < NREC) recs[threadIdx.x + n * kFewThreads] = v;
        }
        const Pos now = p;
        brick = next(brick + gridDim.x, &p);
        const TileBox &bx = now.bx;
        const long long base = now.base;
        const int d0 = now.d0, h0 = now.h0, w0 = now.w0;
        __syncthreads();
        if (brick < a.nbricks) load(p);
        const int d = d0 + wave;
        if (d >= bx.bd) continue;                     // (wave-uniform; the barriers are at the top of the loop)
#pragma unroll
        for (int hp = 0; hp < BH; hp += 2) {
            f32x16 acc[2] = {init, init};
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int kd = r / 3, kh = r % 3;
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    const rec_t *p = recs + ((wave + kd) * RH_ + hp + s + kh) * RW + col;
                    if (CS == 4) {                    // records 0, 1 | 2, nothing
                        const rec_t x0 = p[2 * hi], x1 = p[1];
                        FewFrag b;
                        b.w[0] = x0[0]; b.w[1] = x0[1];
                        b.w[2] = hi ? 0u : x1[0]; b.w[3] = hi ? 0u : x1[1];
                        acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[r][0].v, b.v, acc[s], 0, 0, 0);
                    } else {                          // record 0 | 1, then 2 | nothing
                        const rec_t x0 = p[hi], x1 = p[2];
                        FewFrag b0, b1;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            b0.w[q] = x0[q % (CS / 2)];
                            b1.w[q] = hi ? 0u : x1[q % (CS / 2)];
                        }
                        acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[r][0].v, b0.v, acc[s], 0, 0, 0);
                        acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[r][NM - 1].v, b1.v, acc[s], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int h = h0 + hp + s, w = w0 + col;
                if (h >= bx.bh || w >= bx.bw) continue;
                uint16_t *o = a.out + (base + (1LL * (d + 1) * g.ph + h + 1) * g.pw + w + 1) * a.cout + co0 + 4 * hi;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = a.relu ? relu_f32(acc[s][4 * q + e]) : acc[s][4 * q + e];
                    *reinterpret_cast<uint2 *>(o + 8 * q) = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
                }
            }
        }
    }
}

}  // namespace

bool conv_few_supported(const Geo &g, int cin, int cout, sp_dtype_t dt) {
    const double vox = 1.0 * g.ntiles * (g.td + 2 * grow_d(g) + BD) * (g.th + 2 * g.grow + BH) * (g.tw + 2 * g.grow + BW);
    return dt == SP_BF16 && cin >= 2 && cin <= 8 && cout % C == 0 && vox / (BD * BH * BW) < 0x7fffffff;
}

int launch_conv_few(const void *Px, const void *w, const float *bias, void *Py, const Geo &g, int cin, int cout, bool relu,
                    hipStream_t s) {
    FewArgs a;
    a.in = static_cast<const uint16_t *>(Px);
    a.w = static_cast<const uint16_t *>(w);
    a.bias = bias;
    a.out = static_cast<uint16_t *>(Py);
    a.g = g;
    a.cout = cout; a.relu = relu;
    a.nd = (g.td + 2 * grow_d(g) + BD - 1) / BD;
    a.nh = (g.th + 2 * g.grow + BH - 1) / BH;
    a.nw = (g.tw + 2 * g.grow + BW - 1) / BW;
    a.nbricks = g.ntiles * a.nd * a.nh * a.nw;
    // four workgroups per compute unit, every one with the same number of bricks
    const int nco = cout / C, most = nco >= 1024 ? 1 : 1024 / nco, rounds = (a.nbricks + most - 1) / most;
    const dim3 grid((a.nbricks + rounds - 1) / rounds, nco);
    using Kern = void (*)(FewArgs);
    static const Kern kern[7][2] = {{conv_few_kernel<2, 3>, conv_few_kernel<2, 1>}, {conv_few_kernel<3, 3>, conv_few_kernel<3, 1>},
                                    {conv_few_kernel<4, 3>, conv_few_kernel<4, 1>}, {conv_few_kernel<5, 3>, conv_few_kernel<5, 1>},
                                    {conv_few_kernel<6, 3>, conv_few_kernel<6, 1>}, {conv_few_kernel<7, 3>, conv_few_kernel<7, 1>},
                                    {conv_few_kernel<8, 3>, conv_few_kernel<8, 1>}};
    hipLaunchKernelGGL(kern[cin - 2][g.flat], grid, dim3(kFewThreads), 0, s, a);
    return record_hip(hipGetLastError());
}

}  // namespace sp3d
