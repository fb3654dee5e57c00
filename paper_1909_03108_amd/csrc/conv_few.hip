// bf16 forward convolution and weight gradient of a first layer with 2 ... 8 input channels (a multi-phase scan, a slab of
// slices), kernel 3x3x3 or 3x3 (2-D variant), output channels in multiples of 32, on v_mfma_f32_32x32x16_bf16 (forward) and
// v_mfma_f32_16x16x32_bf16 (weight gradient, further down).
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

// ---- weight and bias gradient ------------------------------------------------------------------------------------------
// D[row][co] = sum over voxels X[row][voxel] dz[voxel][co], row = (kw, channel) of one kernel row: 3 CS of the 16 (CS = 4) or
// 32 (CS = 8) rows of one or two MFMAs, K = 32 voxels along W.  The records lie in LDS as above, so row m of voxel v is value
// v CS + m of a staged row of records whatever kw is, and the transposing LDS load reads A straight from there (the 16 voxels
// x 4 rows of a lane group overlap, which costs nothing: they are one run of LDS); B is dz, whose two halves of 16
// channels are kept apart in LDS as in wgrad_mfma.hip.  Rows past the last (kw, channel) multiply the record behind and are
// dropped.  A wave owns one slice of the brick and keeps the sums of all kernel rows (36 MB registers per three of them) over
// all bricks of its workgroup; the loads of the next brick are in flight during the products of this one.  Partial sums per
// workgroup, added in order by reduce_runs_kernel.
// What bounds it: dz from HBM (64 of 70 bytes per voxel and block of 32 output channels) and the staging's 2-byte loads.  On
// channels zero-padded to 32 it was a copy, ten times the products and a second pass over the result: 3 -> 32 on 99 x 156 x
// 210, both layers forward and backward, 1331 -> 1158 us; the 2-D network's training step on 16 slabs 21.88 -> 21.73 ms; error
// against 64 bits 5.5e-7 -> 2.1e-7 and 6.0e-7 -> 4.7e-7.
constexpr int wgrad_rows(int cin, int kd) { return cin > 4 && kd == 3 ? 2 : 4; }      // brick rows: what the registers hold
constexpr int wgrad_groups(int cin, int kd) { return cin > 4 && kd == 3 ? 2 : 3; }   // workgroups per compute unit, likewise

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
__device__ __forceinline__ s16x4 tr_read(const char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(__attribute__((address_space(3))) char *)(p));
}
union TrFrag { struct { s16x4 lo, hi; } s; uint32_t w[4]; bf16x8 v; };

struct FewWgradArgs {
    const uint16_t *x, *dz;
    float *part;                 // [workgroup along x][taps * cin * cout, then cout]
    Geo g;
    int cout, bias;
    int nd, nh, nw, nbricks;
};

template <int CIN, int KD>
__global__ __launch_bounds__(kFewThreads, wgrad_groups(CIN, KD)) void wgrad_few_kernel(FewWgradArgs a) {
    constexpr int BH = wgrad_rows(CIN, KD), OD = KD / 2, RD = BD + 2 * OD, RH_ = BH + 2, RW = BW + 2, NREC = RD * RH_ * RW;
    constexpr int CS = CIN <= 4 ? 4 : 8, NR = 3 * KD, MB = CS / 4;
    constexpr int PER = (NREC + kFewThreads - 1) / kFewThreads, NV = CIN % 2 ? CIN : CIN / 2;
    constexpr int ZVOX = BD * BH * BW, Z_HALF = ZVOX * 32 + 64;        // LDS bytes of one half of dz: 32-byte voxel records
    constexpr int ZLD = ZVOX * 4 / kFewThreads;                        // 16-byte pieces of dz per thread and brick
    constexpr int NSUM = NR * MB * 2 + 2;                              // accumulators per wave: dw, then the two halves of db
    typedef typename Rec<CS>::type rec_t;
    // (the reads of the rows past the last one reach four records past the end)
    constexpr int RECS_BYTES = ((NREC + 4) * CS * 2 + 15) / 16 * 16;
    constexpr int LDS_BYTES = RECS_BYTES + 2 * Z_HALF > NSUM * 1024 ? RECS_BYTES + 2 * Z_HALF : NSUM * 1024;
    __shared__ __align__(16) char lds[LDS_BYTES];
    rec_t *const recs = reinterpret_cast<rec_t *>(lds);
    char *const lz = lds + RECS_BYTES;
    const Geo &g = a.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int G = lane >> 4, p16 = lane & 15, c4 = threadIdx.x & 3;
    const int co0 = C * blockIdx.y;
    // workgroup ids go round the 8 XCDs; renumbered, an XCD holds a run of neighbouring bricks
    const int group = (gridDim.x & 7) == 0 ? (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3) : blockIdx.x;

    f32x4 acc[NR][MB][2], accb[2];
    const f32x4 zero{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        accb[n] = zero;
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int m = 0; m < MB; ++m) acc[r][m][n] = zero;
    }
    TrFrag ones;
#pragma unroll
    for (int i = 0; i < 4; ++i) ones.w[i] = 0x3f803f80u;

    uint32_t raw[PER][NV];
    uint4 zr[ZLD];
    struct Pos { int tile, d0, h0, w0; };
    auto pos_of = [&](int brick) {
        Pos p;
        int t = brick;
        p.w0 = (t % a.nw) * BW; t /= a.nw;
        p.h0 = (t % a.nh) * BH; t /= a.nh;
        p.d0 = (t % a.nd) * BD; p.tile = t / a.nd;
        return p;
    };
    auto load = [&](const Pos &p) {
        const long long base = p.tile * g.tile_vox;
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));                 // (coordinates are cheap; kept over the loop they push sums out of registers)
#pragma unroll
        for (int n = 0; n < PER; ++n) {
            // records beyond what the tile's own voxels read are moved to the nearest one inside: they reach no result
            const int rec = min(tid + n * kFewThreads, NREC - 1);
            const int i = rec / (RH_ * RW), j = rec / RW % RH_, k = rec % RW;
            const int d = min(p.d0 + i - OD, g.td - 1 + OD), h = min(p.h0 + j - 1, g.th), w = min(p.w0 + k - 1, g.tw);
            const uint16_t *src = a.x + (base + (1LL * (d + 1) * g.ph + h + 1) * g.pw + w + 1) * CIN;
#pragma unroll
            for (int v = 0; v < NV; ++v) raw[n][v] = CIN % 2 ? src[v] : reinterpret_cast<const uint32_t *>(src)[v];
        }
        const uint16_t *tz = a.dz + base * a.cout + co0 + 8 * c4;
#pragma unroll
        for (int i = 0; i < ZLD; ++i) {
            const int v = (tid + i * kFewThreads) >> 2;
            const int d = p.d0 + v / (BH * BW), h = p.h0 + v / BW % BH, w = p.w0 + v % BW;
            zr[i] = make_uint4(0, 0, 0, 0);
            if (d < g.td && h < g.th && w < g.tw)
                zr[i] = *reinterpret_cast<const uint4 *>(tz + ((1LL * (d + 1) * g.ph + h + 1) * g.pw + w + 1) * a.cout);
        }
    };

    // this lane's part of a transposing read: voxels 8 G + p16 / 4 (+ 4), rows or channels 4 (p16 % 4) ..
    const char *const xlane = lds + (8 * G + (p16 >> 2)) * (CS * 2) + (p16 & 3) * 8;
    const char *const zlane = lz + (8 * G + (p16 >> 2)) * 32 + (p16 & 3) * 8;

    int brick = group;
    Pos p = pos_of(brick);
    if (brick < a.nbricks) load(p);
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
#pragma unroll
        for (int i = 0; i < ZLD; ++i) {
            const int v = (threadIdx.x + i * kFewThreads) >> 2;
            *reinterpret_cast<uint4 *>(lz + (c4 >> 1) * Z_HALF + v * 32 + (c4 & 1) * 16) = zr[i];
        }
        const Pos now = p;
        brick += gridDim.x;
        __syncthreads();
        if (brick < a.nbricks) { p = pos_of(brick); load(p); }
        if (now.d0 + wave >= g.td) continue;          // (wave-uniform; the barriers are at the top of the loop)
        // voxels of the last, partial run of a row: their x counts as zero too (dz is zero there, but x may be infinite)
        const int left = g.tw - now.w0;
        uint32_t keep[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            keep[i] = (8 * G + 2 * i < left ? 0xffffu : 0u) | (8 * G + 2 * i + 1 < left ? 0xffff0000u : 0u);
#pragma unroll 1
        for (int h = 0; h < min(BH, g.th - now.h0); ++h) {
            TrFrag z[2];
            const char *const zp = zlane + (wave * BH + h) * BW * 32;
#pragma unroll
            for (int n = 0; n < 2; ++n) { z[n].s.lo = tr_read(zp + n * Z_HALF); z[n].s.hi = tr_read(zp + n * Z_HALF + 4 * 32); }
            // fragment i: kernel row i / MB, row block i % MB; the next one is read before the products of this one
            TrFrag x[2];
            auto read = [&](int i) {
                const int r = i / MB;
                const char *const xp = xlane + ((wave + r / 3) * RH_ + h + r % 3) * RW * (CS * 2) + (i % MB) * 32;
                x[i & 1].s.lo = tr_read(xp);
                x[i & 1].s.hi = tr_read(xp + 4 * CS * 2);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[i & 1].w[e] &= keep[e];
            };
            read(0);
#pragma unroll
            for (int i = 0; i < NR * MB; ++i) {
                if (i + 1 < NR * MB) read(i + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int n = 0; n < 2; ++n)
                    acc[i / MB][i % MB][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[i & 1].v, z[n].v, acc[i / MB][i % MB][n], 0, 0, 0);
            }
            if (a.bias) {
#pragma unroll
                for (int n = 0; n < 2; ++n) accb[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones.v, z[n].v, accb[n], 0, 0, 0);
            }
        }
    }
    // the four waves' sums, added in wave order
    __syncthreads();
    float *const red = reinterpret_cast<float *>(lds);
    for (int wv = 0; wv < kFewThreads / 64; ++wv) {
        if (wave == wv) {
#pragma unroll
            for (int n = 0; n < 2; ++n) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int r = 0; r < NR; ++r)
#pragma unroll
                        for (int m = 0; m < MB; ++m) {
                            float *q = red + (((r * MB + m) * 2 + n) * 4 + i) * 64 + lane;
                            *q = wv ? *q + acc[r][m][n][i] : acc[r][m][n][i];
                        }
                    float *q = red + ((NR * MB * 2 + n) * 4 + i) * 64 + lane;
                    *q = wv ? *q + accb[n][i] : accb[n][i];
                }
            }
        }
        __syncthreads();
    }
    const size_t ndw = static_cast<size_t>(3 * NR) * CIN * a.cout;
    float *const part = a.part + group * (ndw + a.cout);
    // element (row m, channel co) of a block: register m % 4 of lane 16 (m / 4) + co
    for (int e = threadIdx.x; e < 3 * NR * CIN * C; e += kFewThreads) {
        const int co = e % C, row = e / C, c = row % CIN, t = row / CIN, r = t / 3, m = (t % 3) * CS + c;
        part[static_cast<size_t>(row) * a.cout + co0 + co] =
            red[(((r * MB + m / 16) * 2 + co / 16) * 4 + m % 4) * 64 + (m % 16) / 4 * 16 + co % 16];
    }
    if (a.bias && threadIdx.x < C) {
        const int co = threadIdx.x;
        part[ndw + co0 + co] = red[(NR * MB * 2 + co / 16) * 4 * 64 + co % 16];
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

// ws_bytes: what the caller was asked for (chan_pad_wgrad_ws_bytes); at least one partial sum fits (a zero-padded layer keeps
// one of 32 channels there).
int launch_wgrad_few(const void *Px, const void *Pdz, float *dw, float *db, const Geo &g, int cin, int cout, void *ws,
                     size_t ws_bytes, hipStream_t s) {
    FewWgradArgs a;
    a.x = static_cast<const uint16_t *>(Px);
    a.dz = static_cast<const uint16_t *>(Pdz);
    a.part = static_cast<float *>(ws);
    a.g = g;
    a.cout = cout; a.bias = db != nullptr;
    a.nd = (g.td + BD - 1) / BD;
    const int kd = g.flat ? 1 : 3, bh = wgrad_rows(cin, kd);
    a.nh = (g.th + bh - 1) / bh;
    a.nw = (g.tw + BW - 1) / BW;
    a.nbricks = g.ntiles * a.nd * a.nh * a.nw;
    // as many workgroups as the compute units hold, every one with the same number of bricks; never more partial sums than
    // the workspace has room for
    const long long ndw = static_cast<long long>(taps_of(g)) * cin * cout, n = ndw + cout;
    const int nco = cout / C;
    long long most = 256 * wgrad_groups(cin, kd) / nco, room = static_cast<long long>(ws_bytes / (n * sizeof(float)));
    if (most > room) most = room;
    if (most < 1) most = 1;
    const long long rounds = (a.nbricks + most - 1) / most;
    const int groups = static_cast<int>((a.nbricks + rounds - 1) / rounds);
    using Kern = void (*)(FewWgradArgs);
    static const Kern kern[7][2] = {{wgrad_few_kernel<2, 3>, wgrad_few_kernel<2, 1>}, {wgrad_few_kernel<3, 3>, wgrad_few_kernel<3, 1>},
                                    {wgrad_few_kernel<4, 3>, wgrad_few_kernel<4, 1>}, {wgrad_few_kernel<5, 3>, wgrad_few_kernel<5, 1>},
                                    {wgrad_few_kernel<6, 3>, wgrad_few_kernel<6, 1>}, {wgrad_few_kernel<7, 3>, wgrad_few_kernel<7, 1>},
                                    {wgrad_few_kernel<8, 3>, wgrad_few_kernel<8, 1>}};
    hipLaunchKernelGGL(kern[cin - 2][g.flat], dim3(groups, nco), dim3(kFewThreads), 0, s, a);
    const int rc = record_hip(hipGetLastError());
    return rc == SP_OK ? launch_reduce_runs(a.part, dw, db, groups, ndw, n, s) : rc;
}

}  // namespace sp3d
