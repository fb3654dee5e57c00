// bf16 3x3 (2-D variant, geometry flag `flat`) and 3x3x3 convolution for layers on few voxels - the bottom levels of
// the 2-D U-Net (Sec. 3: 512 and 1024 filters on tiles of 16 x 16 voxels and less) and of the 3-D one, and every level
// of a network on a small patch - as an output-stationary implicit GEMM on the gfx950 matrix cores.  Serves conv3d_fwd
// and, on weights packed with mirrored taps and swapped channel roles, conv3d_dgrad, like the plane-marching kernels of
// conv_mfma.hip.
//
// Why a second kernel family.  The marching kernels keep the weights of ONE pair of input chunks in
// registers and stream voxels past them; a layer with 1024 input channels is 16 launches that hand fp32
// partial sums to each other through memory, and on tiles of 8 x 8 voxels each launch is a march of a few
// steps in a mostly empty patch.  Here the roles are swapped: a workgroup owns a tile of output voxels x output
// channels, keeps their sums in registers over a run of K (kernel rows x input chunks), and streams weights and
// voxels: voxels are numbered across rows, slices and tiles, so every MFMA column is a real voxel whatever the tile
// shape, and where tiles are fewer than compute units the K loop is split between `nsplit` workgroups, whose fp32 sums a
// second launch adds in order.
//
// A K step is one kernel row (three taps kw) x one 32-channel input chunk.
//   A (weights): the packed fragments of conv_mfma.hip, 1 KB each, lane-major, loaded into registers one or three steps ahead (the two
//     waves of an output block meet in the vector cache).
//   B (voxels): through LDS by direct loads, three stages: the records (32 channels, 64 bytes) of the padded rows that the
//     tile's voxels touch, each ONCE for the three taps of the row: voxel q of a box row of ew voxels is record (q / ew)
//     (ew + 2) + q % ew, and the taps read this record and the two after it.  The 16-byte pieces of a record sit in the order
//     piece ^ (record / 4 % 4), so that the 16-byte reads of 16 neighbouring voxels fall into 16 different bank groups.
// (v_mfma_f32_32x32x16_bf16, A = weights [32 output channels][16 input channels], B = voxels [16 input channels][32
// voxels]; four waves, two along output channels x two along voxels.)  One barrier per step, placed before the step's last
// MFMA group, so that the next step's first fragments are read behind it while that group runs; a step's loads are issued one per
// group, between its products.  Workgroups stay: as many as fit on the chip take one item (tile and range of K) after the
// other, and the loads run on into the next item while this one's sums are stored.
// What bounds it: long K loops the chip's power (512 -> 512 on 32^3 390 us = 1.19 PFLOP/s, what the vendor's GEMM reaches on the
// card), short ones the stores and index arithmetic between items.  With both operands in LDS and a workgroup per item, LDS
// reads and loads took as long as the products, the loads' addresses were computed while the matrix cores waited, and every
// item began and ended alone; before -> now: 2-D, 128 -> 128 on 16 x 128^2 145 -> 92 us, 256 -> 256 on 16 x 64^2 109 -> 88, 512 ->
// 512 on 16 x 32^2 98 -> 81, 64 -> 64 on 2 x 256^2 36 -> 23, 3-D, 256 -> 256 on 32^3 132 -> 110, 512 -> 512 on 16^3 84 -> 75 (with the
// packing of the weights; with both operands in LDS still, staying workgroups alone gave 145 -> 127).  Layers of one
// item per compute unit and few steps (1024 -> 1024 on 16 x 16, two slices: 31 us) wait for a launch, a pipeline of three stages and
// a second launch that adds the splits.
//
// Output box growth, two input tensors (concatenation without a copy), two output tensors, bias, ReLU, the ReLU mask
// of the data gradient, its one-bit forms and gathered halos behave as in conv_mfma.hip.  The order of the additions
// is fixed (kernel rows, then chunks, then taps within a split; then the splits), and the split depends on the layer's
// interior voxel count and channels only, so results are reproducible and depend neither on the voxel's position nor on
// the tile grid.
#include "conv_mfma_common.h"

#include <algorithm>

namespace sp3d {

using namespace convk;

namespace {

// (a plain vector type: arrays of the runtime's uint4 class stay in scratch memory)
constexpr int kGemmWaves = 4, kGemmThreads = 256;
constexpr int ROW = 3;                           // taps per K step (one row of the kernel)
constexpr int NTAP_PACK = 27;                    // packed weights: 27 tap slots per (chunk, block); the 3x3 kernel of the
                                                 // 2-D variant sits in 9 .. 17 (the taps with kd = 1)
constexpr int wg_vox(int vb) { return 128 * vb; }
// Cutting of a workgroup: CBW output blocks per wave (2 CBW per workgroup), VB x 128 voxels, BL wave loads of 16 records
// per wave and step.
constexpr int stage_bytes(int bl) { return 4 * bl * 1024; }
// LDS stages of voxels; the step loop is unrolled by as many, so that a stage and a register set have their place at compile
// time.  A whole K loop is a multiple of as many steps (kernel rows x chunks: 3 divides both 3 and 9); the part of one that a split
// has is any number from four up, so that items of split layers begin and end in any phase of the unrolled loop.
constexpr int NS = 3;
// steps that weight fragments are loaded ahead (128 channels x 128 voxels: one, so that two workgroups fit the registers)
constexpr int ahead(int cbw, int vb) { return cbw == 2 && vb == 1 ? 1 : NS; }
// workgroups per compute unit
constexpr int resident(int cbw, int vb) { return cbw == 2 && vb == 2 ? 1 : 2; }

struct GemmArgs {
    const uint16_t *in;      // input channels [0, in_ca): in_cs channels per voxel
    const uint16_t *in2;     // input channels [in_ca, ki): in2_cs channels per voxel (NULL: one tensor)
    int in_cs, in2_cs, in_ca;
    const uint4 *wpack;      // [nci][nco][27][2][64] x 16 bytes
    const float *bias;       // bias of all output channels or NULL
    uint16_t *out;           // output channels [0, out_ca): out_cs channels per voxel
    uint16_t *out2;          // output channels [out_ca, ko): out2_cs per voxel (NULL: one tensor)
    int out_cs, out2_cs, out_ca;
    const uint16_t *mask;    // kMask: tensor laid out like `out`; results are zeroed where it is not positive
    uint16_t *bits;          // kMaskBits (read) / kReluBits (written)
    float4 *part;            // nsplit > 1: fp32 sums in fragment order (see part_index)
    Geo g;
    int nci, nco;            // input chunks, output blocks
    int nrows;               // kernel rows (kd, kh): 3 in the 2-D variant, 9 in 3-D
    int nsplit;              // workgroups that share the K loop of a tile
    int nvg;                 // voxel groups of 128 VB
    int nblocks;             // tiles: nvg * nco / (2 CBW); times nsplit real workgroups (grid: rounded up to 8)
    int nvox;                // ntiles * ed * eh * ew: voxels of the largest output box, every tile
    int ed, eh, ew;          // largest output box of the grid (interior grown on both sides)
    int epi, gather;
    int relu_keeps_nan;      // ReLU: any NaN stays; otherwise one with the sign set becomes 0, as in the marching kernels
    FastDiv drow, drec, deh, ded;    // ew, ew + 2, eh, ed
};

// 16 bytes per lane from global memory straight into LDS: lane l's data lands at dst + 16 l (dst is wave-uniform and
// travels in M0).  Written as assembly because the compiler, when it knows of such a load, waits for ALL outstanding ones
// before every LDS read; the kernel waits for exactly the loads it needs.
__device__ __forceinline__ void dma16(const void *src, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(dst) : "memory");
}

// Source of input chunk i: tensor, channels per voxel, channel offset.
struct InSrc { const uint16_t *base; int cs, co; };
__device__ __forceinline__ InSrc in_src(const GemmArgs &a, int i) {
    const int c0 = C * i;
    if (a.in2 && c0 >= a.in_ca) return InSrc{a.in2, a.in2_cs, c0 - a.in_ca};
    return InSrc{a.in, a.in_cs, c0};
}

struct BoxPos { int tile, d, h, w; };
// box row index (over all tiles) -> tile, d, h
__device__ __forceinline__ BoxPos row_pos(const GemmArgs &a, uint32_t row) {
    BoxPos p;
    const uint32_t t = fdiv(row, a.deh), tile = fdiv(t, a.ded);
    p.h = static_cast<int>(fmod_(row, t, a.deh));
    p.d = static_cast<int>(fmod_(t, tile, a.ded));
    p.tile = static_cast<int>(tile);
    p.w = 0;
    return p;
}

// Output voxel q: whether it exists (past the end, or outside the box of a tile without a neighbour on that side: no) and
// its padded voxel index (0 where it does not: an address that can be loaded from).
struct OutVox { long long pv; bool ok; };
__device__ __forceinline__ OutVox out_vox(const GemmArgs &a, int q) {
    const uint32_t qq = static_cast<uint32_t>(min(q, a.nvox - 1)), row = fdiv(qq, a.drow);
    BoxPos p = row_pos(a, row);
    p.w = static_cast<int>(fmod_(qq, row, a.drow));
    const TileBox bx = tile_box(a.g, p.tile);
    OutVox o;
    o.ok = q < a.nvox && p.d < bx.bd && p.h < bx.bh && p.w < bx.bw;
    o.pv = o.ok ? static_cast<long long>(p.tile) * a.g.tile_vox + bx.org + (1LL * (p.d + 1) * a.g.ph + p.h + 1) * a.g.pw + p.w + 1 : 0;
    return o;
}

// What the epilogue of one voxel and output block reads: 16 bytes of the mask at channels 16 p + 8 hi, or the lane's word.
struct EpiIn { uint4 mask[2]; uint32_t word; };
template <int EPI>
__device__ __forceinline__ void epi_load(const GemmArgs &a, EpiIn &in, int cj, int hi, const OutVox &o) {
    if (EPI == kMask) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
            in.mask[p] = *reinterpret_cast<const uint4 *>(a.mask + o.pv * a.out_cs + C * cj + 16 * p + 8 * hi);
    }
    if (EPI == kMaskBits) in.word = a.bits[(o.pv * a.nco + cj) * 2 + hi];
}

// Finished sums of one voxel, 16 channels (8 q + 4 hi + i) of output block cj: ReLU / mask, convert, store.  The two lanes
// of a voxel (hi = 0, 1) exchange halves, so that each holds 8 consecutive channels: 16-byte stores, 32 consecutive bytes a
// voxel and instruction.
template <int EPI>
__device__ __forceinline__ void finish(const GemmArgs &a, const f32x16 &s, int cj, int hi, const OutVox &o, const EpiIn &in) {
    const int co = C * cj;
    uint16_t *obase = a.out;
    int ocs = a.out_cs, oco = co;
    if (a.out2 && co >= a.out_ca) { obase = a.out2; ocs = a.out2_cs; oco = co - a.out_ca; }
    uint4 *dst = reinterpret_cast<uint4 *>(obase + o.pv * ocs + oco + 8 * hi);
    uint32_t bits = 0;
    if (EPI == kMaskBits) bits = spread_word(in.word);
    uint2 pk[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = s[4 * q + i];
            if (is_relu(EPI)) v[i] = a.relu_keeps_nan ? (v[i] < 0.f ? 0.f : v[i]) : relu_f32(v[i]);
            if (EPI == kReluBits) bits = shift_in_positive(bits, v[i]);
        }
        pk[q] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        if (EPI == kMaskBits) {
            const uint2 mv = nibble_halves(bits, q);
            pk[q].x &= mv.x;
            pk[q].y &= mv.y;
        }
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const auto x = __builtin_amdgcn_permlane32_swap(pk[2 * p].x, pk[2 * p + 1].x, false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(pk[2 * p].y, pk[2 * p + 1].y, false, false);
        uint4 v = make_uint4(x[0], y[0], x[1], y[1]);
        if (EPI == kMask) {
            v.x &= positive_halves(in.mask[p].x);
            v.y &= positive_halves(in.mask[p].y);
            v.z &= positive_halves(in.mask[p].z);
            v.w &= positive_halves(in.mask[p].w);
        }
        if (o.ok) dst[2 * p] = v;
    }
    if (EPI == kReluBits && o.ok) a.bits[(o.pv * a.nco + cj) * 2 + hi] = row_word(bits);
}

// f(epilogue as a compile-time constant)
template <class F>
__device__ __forceinline__ void with_epilogue(int epi, F &&f) {
    switch (epi) {
    case kNone: f(std::integral_constant<int, kNone>{}); break;
    case kRelu: f(std::integral_constant<int, kRelu>{}); break;
    case kMask: f(std::integral_constant<int, kMask>{}); break;
    case kMaskBits: f(std::integral_constant<int, kMaskBits>{}); break;
    default: f(std::integral_constant<int, kReluBits>{}); break;
    }
}

// Sums of a split: unit (tile, wave, block of the wave, segment, q) x 64 lanes x 4 channels, 1 KB per unit.
template <int CBW, int VB>
__device__ __forceinline__ size_t part_index(const GemmArgs &a, int split, int blk, int wave, int c, int s, int lane) {
    return (((static_cast<size_t>(split) * a.nblocks + blk) * kGemmWaves + wave) * CBW * 2 * VB + c * 2 * VB + s) * 256 + lane;
}

// SPLIT: a.nsplit > 1.  Split s has the steps [s nk / nsplit, (s + 1) nk / nsplit), as plan_gemm prices them and in the order of the sums
// that a K loop cut by any kernel of this family has had; with splits in whole threes the longest of them ran up to half as
// many steps again: 128 -> 128 on 8^3 (nine splits of four steps) 17.2 -> 15.6 us, 256 -> 256 there 23.4 -> 21.9, 512 -> 512 on 4^3
// 29.1 -> 27.5; on 134 layers 0.94 of the time, where the splits are whole threes anyway up to 1.05 (an end to look for in every
// step).
template <int CBW, int VB, int BL, bool SPLIT>
__global__ __launch_bounds__(kGemmThreads, resident(CBW, VB)) void conv_gemm_kernel(GemmArgs a) {
    constexpr int NSEG = 2 * VB, CBT = 2 * CBW, NGRP = 2 * ROW, STAGE = stage_bytes(BL), AD = ahead(CBW, VB);
    extern __shared__ __align__(16) char lds[];
    // Workgroups of one XCD (blockIdx % 8) share a run of consecutive items (an item: a tile and a range of K) and take them
    // side by side: neighbours share output blocks and K range, i.e. weights.
    const int items = a.nblocks * a.nsplit, per_xcd = (items + 7) >> 3, nslots = gridDim.x >> 3;
    const int first = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3), end = min((static_cast<int>(blockIdx.x & 7) + 1) * per_xcd, items);
    if (first >= end) return;
    const Geo &g = a.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave & 1, wn = wave >> 1, hi = lane >> 5;
    // (voxel indices are unsigned and 32 bits wide: 2^32 voxels of at least 32 + 64 channels do not fit the memory)
    const uint32_t prow = g.pw, pplane = static_cast<uint32_t>(g.ph) * g.pw;
    const int nk = a.nci * a.nrows;
    struct Item { int vg, split, cg, k0, k1; };          // voxel group, split, group of output blocks, steps [k0, k1)
    auto item_at = [&](int i) __attribute__((always_inline)) {
        const int u = i / a.nvg;
        Item t;
        t.vg = i - u * a.nvg;
        t.cg = SPLIT ? u / a.nsplit : u;
        t.split = SPLIT ? u - t.cg * a.nsplit : 0;
        t.k0 = SPLIT ? t.split * nk / a.nsplit : 0;
        t.k1 = SPLIT ? (t.split + 1) * nk / a.nsplit : nk;
        return t;
    };
    auto record = [&](int q) __attribute__((always_inline)) {
        const uint32_t row = fdiv(static_cast<uint32_t>(q), a.drow);
        return row * (a.ew + 2) + fmod_(static_cast<uint32_t>(q), row, a.drow);
    };

    // The loads run ahead of the products, from one item into the next.  Voxels: NS - 1 steps.  This lane's share of them:
    // records 16 (BL wave + j) + lane / 4, piece lane % 4 of each (stored order).  Records past the last one repeat it;
    // records of rows that a tile's own box lacks are moved inside it (both only feed results that are dropped).
    int fitem = first, fleft = 0, fr = 0, fi = 0;               // item, steps left of it, next kernel row and chunk (chunks
                                                                // innermost: two neighbouring ones share a cache line)
    uint32_t rvox[BL];
    int rflag[BL];                   // gathered halos: bit 0 / 1 first / last row with a neighbour, 2 / 3 plane
    const uint32_t tvox = static_cast<uint32_t>(g.tile_vox);
    const uint32_t sw = tvox - g.tw, sh = tvox * g.gw - g.th * prow, sd = tvox * g.gw * g.gh - g.td * pplane;
    auto open_voxels = [&]() __attribute__((always_inline)) {
        const Item t = item_at(fitem);
        fleft = t.k1 - t.k0;
        fr = t.k0 / a.nci;
        fi = t.k0 - fr * a.nci;
        const int q0 = t.vg * wg_vox(VB);
        const uint32_t rec0 = record(q0), nrec = record(min(q0 + wg_vox(VB), a.nvox) - 1) + 3 - rec0;
#pragma unroll
        for (int j = 0; j < BL; ++j) {
            const uint32_t k = min(static_cast<uint32_t>(16 * (BL * wave + j) + (lane >> 2)), nrec - 1) + rec0;
            const uint32_t row = fdiv(k, a.drec);
            BoxPos p = row_pos(a, row);
            const TileBox bx = tile_box(g, p.tile);
            p.d = min(p.d, bx.bd - 1);
            p.h = min(p.h, bx.bh - 1);
            p.w = min(static_cast<int>(fmod_(k, row, a.drec)), bx.bw + 1);
            rvox[j] = p.tile * tvox + static_cast<uint32_t>(bx.org) + (p.d + 1) * pplane + (p.h + 1) * prow + p.w;
            rflag[j] = 0;
            if (a.gather) {          // (host: one-voxel margins, no grown box, 3-D)
                const int tc = p.tile % g.gw, t1 = p.tile / g.gw, tb = t1 % g.gh, ta = (t1 / g.gh) % g.gd;
                if (p.w == 0 && tc > 0) rvox[j] -= sw;
                if (p.w == g.tw + 1 && tc < g.gw - 1) rvox[j] += sw;
                rflag[j] = (p.h == 0 && tb > 0 ? 1 : 0) | (p.h == g.th - 1 && tb < g.gh - 1 ? 2 : 0) |
                           (p.d == 0 && ta > 0 ? 4 : 0) | (p.d == g.td - 1 && ta < g.gd - 1 ? 8 : 0);
            }
        }
    };
    const int piece = 8 * ((lane & 3) ^ (lane >> 4));
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char *)lds)) + BL * wave * 1024;
    // load j of the next step's records
    auto fetch_voxels = [&](int stage, int j) __attribute__((always_inline)) {
        const InSrc src = in_src(a, fi);
        const int kd = a.nrows == 3 ? 1 : fr / 3, kh = a.nrows == 3 ? fr : fr - 3 * (fr / 3);
        uint32_t at = rvox[j] + (kd - 1) * pplane + (kh - 1) * prow;
        if (a.gather) {
            const int mh = kh == 0 ? 1 : (kh == 2 ? 2 : 0), md = kd == 0 ? 4 : (kd == 2 ? 8 : 0);
            at += (rflag[j] & mh ? (kh == 0 ? -sh : sh) : 0) + (rflag[j] & md ? (kd == 0 ? -sd : sd) : 0);
        }
        const uint64_t base = reinterpret_cast<uint64_t>(src.base + src.co + piece);
        dma16(reinterpret_cast<const void *>(base + static_cast<uint64_t>(at) * static_cast<uint32_t>(2 * src.cs)),
              lds0 + stage * STAGE + j * 1024);
    };
    // may_end: the step just fetched may be an item's last one (its phase is NS - 1, or the items are splits)
    auto next_voxels = [&](bool may_end) __attribute__((always_inline)) {
        if (--fleft > 0) {
            if (++fi == a.nci) { fi = 0; ++fr; }
        } else if (may_end && fitem + nslots < end) {
            fitem += nslots;
            open_voxels();
        } else {
            fleft = 1;               // past the last step the loads repeat it (in bounds; what they fill is never used)
        }
    };

    // Weights: AD steps ahead, into registers, by ordinary loads (the two waves of an output block share them through the
    // vector cache).
    bf16x8 wf[AD][NGRP][CBW];
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint4 *>(a.wpack), 0, a.nci * a.nco * NTAP_PACK * 2048, 0x00027000);
    int witem = first, wleft = 0, wi = 0, wrow = 0, wat = 0;    // item, steps left, chunk, byte offset of (kernel row, block), with the chunk
    auto open_weights = [&]() __attribute__((always_inline)) {
        const Item t = item_at(witem);
        wleft = t.k1 - t.k0;
        const int r = t.k0 / a.nci;
        wi = t.k0 - r * a.nci;
        wrow = ((t.cg * CBT + wm * CBW) * NTAP_PACK + (a.nrows == 3 ? 9 : 0) + ROW * r) * 2048;
        wat = wrow + wi * a.nco * NTAP_PACK * 2048;
    };
    auto fetch_weights = [&](int set, int gi) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CBW; ++c) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(wres, lane * 16 + gi * 1024, wat + c * NTAP_PACK * 2048, 0);
            wf[set][gi][c] = __builtin_bit_cast(bf16x8, v);
        }
    };
    auto next_weights = [&](bool may_end) __attribute__((always_inline)) {
        if (--wleft > 0) {
            wat += a.nco * NTAP_PACK * 2048;
            if (++wi == a.nci) { wi = 0; wrow += ROW * 2048; wat = wrow; }
        } else if (may_end && witem + nslots < end) {
            witem += nslots;
            open_weights();
        } else {
            wleft = 1;
        }
    };

    // this lane's read offsets inside a stage: record of its voxel in segment s, one and two records on
    int boff[NSEG][ROW];
    auto read_offsets = [&](int q0) __attribute__((always_inline)) {
        const uint32_t rec0 = record(q0);
#pragma unroll
        for (int s = 0; s < NSEG; ++s) {
            const int q = min(q0 + wn * 64 * VB + s * 32 + (lane & 31), a.nvox - 1);
            const int r = static_cast<int>(record(q) - rec0);
#pragma unroll
            for (int kw = 0; kw < ROW; ++kw) boff[s][kw] = (r + kw) * 64 + ((hi ^ ((r + kw) >> 2)) & 3) * 16;
        }
    };

    f32x16 acc[CBW][NSEG];
    bf16x8 bf[2][NSEG];
    auto read_group = [&](int stage, int gi) __attribute__((always_inline)) {    // (kw, K-half) group gi -> fragment set gi % 2
#pragma unroll
        for (int s = 0; s < NSEG; ++s)
            bf[gi & 1][s] = *reinterpret_cast<const bf16x8 *>(lds + (boff[s][gi >> 1] ^ ((gi & 1) * 32)) + stage * STAGE);
    };
    // One step, in phase P of NS: its voxels are in stage P, the loads of the step NS - 1 on go to the stage that the step
    // before it left, one in each of the first BL groups; its weights are in set P (the only one if AD = 1).  TAIL: of the
    // workgroup's last NS - 1 steps at most, behind which there is nothing to load.
    int next_q0 = -1;                // first voxel of the next item, in an item's last step (-1: nothing to do)
    auto step = [&](auto phase, auto tail) __attribute__((always_inline)) {
        constexpr int P = decltype(phase)::value, SET = AD == 1 ? 0 : P;
        constexpr bool TAIL = decltype(tail)::value;
#pragma unroll
        for (int gi = 0; gi < NGRP; ++gi) {
            if (gi + 1 < NGRP) {
                read_group(P, gi + 1);
            } else {
                if (!TAIL && (SPLIT || P == NS - 1) && next_q0 >= 0) read_offsets(next_q0);
                // Every wave has read this step's last fragments (lgkmcnt) and the next step's records have landed: after
                // the last of their loads, in group BL - 1 of the step before, there were the weight loads of that group and the ones
                // behind it and this step's loads up to here.  Behind the barrier this step's stage is free.
                constexpr int NEWER = TAIL ? 0 : (NGRP + 1 - BL) * CBW + (BL < NGRP ? BL : NGRP - 1) + (NGRP - 1) * CBW;
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NEWER) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                read_group((P + 1) % NS, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < CBW * NSEG; ++m) {
                const int c = m / NSEG, s = m % NSEG;
                if (m == 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (!TAIL && gi < BL) fetch_voxels((P + NS - 1) % NS, gi);
                    // (where the next loads are from is found between products too)
                    if (SPLIT && !TAIL && gi == BL) next_voxels(true);
                    if (SPLIT && (!TAIL || AD == 1) && gi == 0) next_weights(true);
                    __builtin_amdgcn_sched_barrier(0);
                }
                acc[c][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[SET][gi][c], bf[gi & 1][s], acc[c][s], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!TAIL || AD == 1) fetch_weights(SET, gi);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!TAIL && (!SPLIT || BL == NGRP)) next_voxels(SPLIT || (P + NS - 1) % NS == NS - 1);
        if (!SPLIT) next_weights((P + AD) % NS == NS - 1);
    };

    open_voxels();
    open_weights();
#pragma unroll
    for (int st = 0; st < NS - 1; ++st) {
#pragma unroll
        for (int j = 0; j < BL; ++j) fetch_voxels(st, j);
        next_voxels(false);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int st = 0; st < AD; ++st) {
#pragma unroll
        for (int gi = 0; gi < NGRP; ++gi) fetch_weights(st, gi);
        if (!SPLIT || st + 1 < AD) next_weights(st == NS - 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    read_offsets(item_at(first).vg * wg_vox(VB));
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * BL + AD * NGRP * CBW) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_group(0, 0);
    int item = first, after = -1;    // first voxel of the item after this one
    Item t;
    // accumulators start from the bias (in the first split): lane l holds channels 8 (e / 4) + 4 (l / 32) + e % 4 of a block
    auto begin = [&]() __attribute__((always_inline)) {
        t = item_at(item);
        after = item + nslots < end ? item_at(item + nslots).vg * wg_vox(VB) : -1;
        const bool biased = a.bias && t.split == 0;
#pragma unroll
        for (int c = 0; c < CBW; ++c) {
            f32x16 v;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                v[e] = biased ? a.bias[C * (t.cg * CBT + wm * CBW + c) + 8 * (e >> 2) + 4 * hi + (e & 3)] : 0.f;
#pragma unroll
            for (int s = 0; s < NSEG; ++s) acc[c][s] = v;
        }
    };
    // The next item's loads are in flight meanwhile; the waits that the compiler puts behind the mask's loads are on the
    // same counter and only ask for more than they need.
    if constexpr (!SPLIT) {
#pragma unroll 1
        for (; item < end; item += nslots) {
            begin();
#pragma unroll 1
            for (int k = 0; k < nk; k += NS) {
                step(std::integral_constant<int, 0>{}, std::false_type{});
                step(std::integral_constant<int, 1>{}, std::false_type{});
                next_q0 = k + NS == nk ? after : -1;
                step(std::integral_constant<int, 2>{}, std::false_type{});
            }
            OutVox o[NSEG];
#pragma unroll
            for (int s = 0; s < NSEG; ++s) o[s] = out_vox(a, t.vg * wg_vox(VB) + wn * 64 * VB + s * 32 + (lane & 31));
            with_epilogue(a.epi, [&](auto epi) __attribute__((always_inline)) {
                constexpr int EPI = decltype(epi)::value;
                const int cj = t.cg * CBT + wm * CBW;
                constexpr int BATCH = NSEG < 2 ? NSEG : 2;       // segments whose mask values are loaded together
#pragma unroll
                for (int s0 = 0; s0 < NSEG; s0 += BATCH) {
                    EpiIn in[CBW][BATCH];
#pragma unroll
                    for (int s = 0; s < BATCH; ++s)
#pragma unroll
                        for (int c = 0; c < CBW; ++c) epi_load<EPI>(a, in[c][s], cj + c, hi, o[s0 + s]);
#pragma unroll
                    for (int s = 0; s < BATCH; ++s)
#pragma unroll
                        for (int c = 0; c < CBW; ++c) finish<EPI>(a, acc[c][s0 + s], cj + c, hi, o[s0 + s], in[c][s]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
        }
    } else {
        auto put = [&]() __attribute__((always_inline)) {
            const int blk = t.cg * a.nvg + t.vg;
#pragma unroll
            for (int s = 0; s < NSEG; ++s)
#pragma unroll
                for (int c = 0; c < CBW; ++c) {
                    float4 *p = a.part + part_index<CBW, VB>(a, t.split, blk, wave, c, s, lane);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        p[64 * q] = make_float4(acc[c][s][4 * q], acc[c][s][4 * q + 1], acc[c][s][4 * q + 2], acc[c][s][4 * q + 3]);
                }
        };
        int steps = 0;               // of all items
        for (int i = first; i < end; i += nslots) {
            const Item n = item_at(i);
            steps += n.k1 - n.k0;
        }
        begin();
        int left = t.k1 - t.k0;
        // (an item's end behind each of the three phases, the loop's only behind all: with a way from a phase to itself, though
        // it is never taken, the compiler waits for weights that are needed three steps later)
        auto turn = [&](auto phase) __attribute__((always_inline)) {
            next_q0 = left == 1 ? after : -1;
            step(phase, std::false_type{});
            if (--left == 0) {
                put();
                item += nslots;
                if (item < end) {
                    begin();
                    left = t.k1 - t.k0;
                }
            }
        };
        int rest = steps;
#pragma unroll 1
        do {                         // (an item has four steps or more)
            turn(std::integral_constant<int, 0>{});
            turn(std::integral_constant<int, 1>{});
            turn(std::integral_constant<int, 2>{});
            rest -= NS;
        } while (rest >= NS);
        if (rest > 0) {
            step(std::integral_constant<int, 0>{}, std::true_type{});
            if (rest > 1) step(std::integral_constant<int, 1>{}, std::true_type{});
            put();
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the repeated loads
}

// The splits' sums, added in order, and the epilogue: one thread per (unit of 16 channels, lane).
template <int CBW, int VB>
__global__ __launch_bounds__(kGemmThreads) void conv_gemm_join_kernel(GemmArgs a) {
    constexpr int NSEG = 2 * VB;
    const int lane = threadIdx.x & 63;
    const long long unit = 4LL * blockIdx.x + (threadIdx.x >> 6);
    if (unit >= 1LL * a.nblocks * kGemmWaves * CBW * NSEG) return;
    int t = static_cast<int>(unit);
    const int s = t % NSEG; t /= NSEG;
    const int c = t % CBW; t /= CBW;
    const int wave = t % kGemmWaves, blk = t / kGemmWaves;
    const int cg = blk / a.nvg, vg = blk - cg * a.nvg, wm = wave & 1, wn = wave >> 1;
    f32x16 sum;
#pragma unroll
    for (int e = 0; e < 16; ++e) sum[e] = 0.f;
#pragma unroll 4
    for (int sp = 0; sp < a.nsplit; ++sp) {
        const float4 *p = a.part + part_index<CBW, VB>(a, sp, blk, wave, c, s, lane);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = p[64 * q];
            sum[4 * q] += v.x; sum[4 * q + 1] += v.y; sum[4 * q + 2] += v.z; sum[4 * q + 3] += v.w;
        }
    }
    const OutVox o = out_vox(a, vg * wg_vox(VB) + wn * 64 * VB + s * 32 + (lane & 31));
    const int cj = cg * 2 * CBW + wm * CBW + c, hi = lane >> 5;
    with_epilogue(a.epi, [&](auto epi) {
        EpiIn in;
        epi_load<decltype(epi)::value>(a, in, cj, hi, o);
        finish<decltype(epi)::value>(a, sum, cj, hi, o, in);
    });
}

// largest output box of the grid
struct Box { int ed, eh, ew; };
Box max_box(const Geo &g) { return Box{g.td + 2 * grow_d(g), g.th + 2 * g.grow, g.tw + 2 * g.grow}; }

struct GemmPlan { int cbw, vb, bl, nsplit, nvg, nblocks; long long nvox; double us; };     // us: estimated time
// records that 128 vb consecutive voxels touch at most, in wave loads of 16 per wave
int record_loads(int vb, int ew) {
    const int n = wg_vox(vb), rows = n % ew == 0 ? n / ew - 1 : (n + ew - 2) / ew;
    return (n + 2 + 2 * rows + 63) / 64;
}
// Voxels per tile and splits of the K loop: what costs least in microseconds if 256 compute units take the items in rounds: a
// step lasts 0.41 us per 128 voxels x 64 channels, an item 10.7 us besides; splitting adds a second launch and a write and a
// read of every sum at about 6 TB/s.  The interior voxels alone decide, so that the order of the sums is the same for every
// output box growth and tile grid.  These constants, and those of the time that is then compared with the marching kernels'
// (fitted to 472 layers cut this way, 32 ... 1024 channels, 64 voxels ... 4 million, 2-D and 3-D; `shortk`, K loops of 3 or 6 steps:
// 354 layers), are of the kernel of one item per workgroup, and choose where a compute unit has one item: such layers have become
// 0.9 of the time that they had then, whatever their splits.  What several items in a row cost is cut_us below.
//
// cut_us: a compute unit works off its share of the items one after the other: per item `steps` steps and what its epilogue
// leaves uncovered.  Two workgroups on a compute unit cover each other's, so where there are several items of few steps
// tiles of 128 voxels are faster (2-D, 128 -> 128 on 16 x 128^2 91 against 106 us, 256 -> 256 on 16 x 64^2 81 against 88), and 256
// where the steps count (3-D, 512 -> 512 on 32^3 390 against 404).  Measured on 31 layers with every cut, 5 % rms.
constexpr struct { double step, item; } kCost[2][2] = {{{0.45, 1.8}, {0.72, 3.0}}, {{0.70, 2.2}, {1.36, 6.5}}};   // [CBW - 1][VB - 1]
double cut_us(int cbw, int vb, long long tiles, int steps) {
    const auto c = kCost[cbw - 1][vb - 1];
    return 7 + static_cast<double>((tiles + 255) / 256) * (steps * c.step + c.item);
}
GemmPlan plan_gemm(const Geo &g, int ki, int ko) {
    GemmPlan p;
    const Box b = max_box(g);
    p.nvox = 1LL * g.ntiles * b.ed * b.eh * b.ew;
    const int nco = ko / C, nk = ki / C * (g.flat ? 3 : 9);
    const long long nint = 1LL * g.ntiles * g.int_vox;
    p.cbw = nco % 4 == 0 ? 2 : 1;
    const bool shortk = g.flat && ki <= 2 * C;
    auto tiles_of = [&](int vb) { return (nint + wg_vox(vb) - 1) / wg_vox(vb) * (nco / (2 * p.cbw)); };
    double least = 0;
    for (int vb = 1; vb <= 2; ++vb) {
        const long long tiles = tiles_of(vb);
        for (int s = 1; s == 1 || (s <= nk / 4 && s <= 64 && tiles * s <= 1024); ++s) {
            const double rounds = static_cast<double>((tiles * s + 255) / 256), steps = (nk + s - 1) / s;
            const double sums = 8.0 * s * nint * ko / 1e6;
            const double us = 4 + rounds * (steps * 0.41 * vb * p.cbw + 10.7) + (s > 1 ? 2 + sums / 6 : 0);
            if ((vb == 1 && s == 1) || us < least) {
                least = us; p.vb = vb; p.nsplit = s;
                p.us = shortk ? 3 + rounds * (steps * 0.41 * (vb == 2 ? 2.66 : 1) * (p.cbw == 2 ? 2.39 : 1) + 9) + (s > 1 ? 1.6 + sums / 3.3 : 0)
                              : 4 + rounds * (steps * 0.44 * (vb == 2 ? 2.09 : 1) * (p.cbw == 2 ? 1.78 : 1) + 9.85) + (s > 1 ? 0.73 + sums / 3.74 : 0);
            }
        }
    }
    if (p.nsplit == 1 && p.cbw == 2 && p.vb == 2 && cut_us(2, 1, tiles_of(1), nk) < 0.97 * cut_us(2, 2, tiles_of(2), nk)) p.vb = 1;
    p.bl = record_loads(p.vb, b.ew);
    if (p.vb == 2 && p.bl > 6) { p.vb = 1; p.bl = record_loads(1, b.ew); }
    p.bl = p.vb == 2 ? (p.bl <= 5 ? 5 : 6) : (p.bl <= 3 ? 3 : (p.bl <= 4 ? 4 : 6));
    p.nvg = static_cast<int>((p.nvox + wg_vox(p.vb) - 1) / wg_vox(p.vb));
    p.nblocks = p.nvg * (nco / (2 * p.cbw));
    return p;
}

}  // namespace

bool conv_gemm_supported(const Geo &g, int ki, int ko) {
    const Box b = max_box(g);
    // (records are numbered in 32 bits: up to three per voxel)
    return ki % C == 0 && ko % (2 * C) == 0 && 1LL * g.ntiles * b.ed * b.eh * b.ew < (1LL << 28);
}

bool conv_gemm_tensor_forms(const Geo &g, int ki, int ko) {
    return conv_gemm_supported(g, ki, ko) && ki >= 512 && ki % (2 * C) == 0 && ko % (4 * C) == 0 &&
           1LL * g.ntiles * g.int_vox <= (g.flat ? (1 << 16) : (1 << 13));
}

double conv_gemm_us(const Geo &g, int ki, int ko) { return plan_gemm(g, ki, ko).us; }

void conv_gemm_detail(const Geo &g, int ki, int ko, int *detail) {
    const GemmPlan p = plan_gemm(g, ki, ko);
    detail[0] = p.cbw; detail[1] = p.vb; detail[2] = p.bl; detail[3] = p.nsplit;
}

size_t conv_gemm_ws_bytes(const Geo &g, int ki, int ko) {
    const GemmPlan p = plan_gemm(g, ki, ko);
    return p.nsplit == 1 ? 0 : static_cast<size_t>(p.nsplit) * p.nvg * wg_vox(p.vb) * ko * sizeof(float);
}

// wpack: the layer's weights in the fragment order of conv_mfma.hip (already packed, in the workspace); part: the
// conv_gemm_ws_bytes behind them.
int launch_conv_gemm(const void *Pin, const void *wpack, void *part, const float *bias, void *Pout, const Geo &g, int ki, int ko,
                     bool relu, bool dgrad, hipStream_t s, const void *mask, const ConvSplit *split, bool gather, void *bits) {
    GemmArgs a;
    a.in = static_cast<const uint16_t *>(Pin);
    a.in2 = nullptr;
    a.in_cs = ki;
    a.in2_cs = 0;
    a.in_ca = ki;
    if (split && split->in2) {
        a.in2 = static_cast<const uint16_t *>(split->in2);
        a.in_ca = split->in_ca;
        a.in_cs = split->in_ca;
        a.in2_cs = ki - split->in_ca;
    }
    a.out = static_cast<uint16_t *>(Pout);
    a.out2 = nullptr;
    a.out_cs = ko;
    a.out2_cs = 0;
    a.out_ca = ko;
    if (split && split->out2) {
        a.out2 = static_cast<uint16_t *>(split->out2);
        a.out_ca = split->out_ca;
        a.out_cs = split->out_ca;
        a.out2_cs = ko - split->out_ca;
    }
    a.wpack = static_cast<const uint4 *>(wpack);
    a.bias = bias;
    a.mask = static_cast<const uint16_t *>(mask);
    a.bits = static_cast<uint16_t *>(bits);
    a.part = static_cast<float4 *>(part);
    a.g = g;
    a.nci = ki / C;
    a.nco = ko / C;
    a.nrows = g.flat ? 3 : 9;
    const Box b = max_box(g);
    a.ed = b.ed;
    a.eh = b.eh;
    a.ew = b.ew;
    const GemmPlan p = plan_gemm(g, ki, ko);
    a.nvox = static_cast<int>(p.nvox);
    a.nsplit = p.nsplit;
    a.nvg = p.nvg;
    a.nblocks = p.nblocks;
    a.epi = bits ? (dgrad ? kMaskBits : kReluBits) : (mask ? kMask : (relu ? kRelu : kNone));
    a.gather = gather ? 1 : 0;
    a.relu_keeps_nan = conv_gemm_tensor_forms(g, ki, ko) ? 1 : 0;
    a.drow = make_fastdiv(static_cast<uint32_t>(b.ew));
    a.drec = make_fastdiv(static_cast<uint32_t>(b.ew + 2));
    a.deh = make_fastdiv(static_cast<uint32_t>(b.eh));
    a.ded = make_fastdiv(static_cast<uint32_t>(b.ed));
    using Kern = void (*)(GemmArgs);
    // [split][output blocks per wave - 1][(voxels, record loads)]
#define SP3D_GEMM_SHAPES(CBW, SPLIT)                                                                                             \
    {conv_gemm_kernel<CBW, 1, 3, SPLIT>, conv_gemm_kernel<CBW, 1, 4, SPLIT>, conv_gemm_kernel<CBW, 1, 6, SPLIT>,                  \
     conv_gemm_kernel<CBW, 2, 5, SPLIT>, conv_gemm_kernel<CBW, 2, 6, SPLIT>}
    static const Kern kern[2][2][5] = {{SP3D_GEMM_SHAPES(1, false), SP3D_GEMM_SHAPES(2, false)},
                                       {SP3D_GEMM_SHAPES(1, true), SP3D_GEMM_SHAPES(2, true)}};
#undef SP3D_GEMM_SHAPES
    static const Kern join[2][2] = {{conv_gemm_join_kernel<1, 1>, conv_gemm_join_kernel<1, 2>},
                                    {conv_gemm_join_kernel<2, 1>, conv_gemm_join_kernel<2, 2>}};
    static const int bls[5] = {3, 4, 6, 5, 6};
    // more than 64 KB of dynamic LDS has to be requested explicitly
    static const hipError_t attr = [] {
        for (int i = 0; i < 20; ++i) {
            const int bl = bls[i % 5];
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern[i / 10][i / 5 % 2][i % 5]),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, NS * stage_bytes(bl));
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (attr != hipSuccess) return record_hip(attr);
    const int shape = p.vb == 2 ? (p.bl == 5 ? 3 : 4) : (p.bl == 3 ? 0 : (p.bl == 4 ? 1 : 2));
    // as many workgroups as fit on the 256 compute units at once
    const unsigned grid = static_cast<unsigned>((std::min(256LL * resident(p.cbw, p.vb), 1LL * a.nblocks * a.nsplit) + 7) / 8 * 8);
    hipLaunchKernelGGL(kern[a.nsplit > 1 ? 1 : 0][p.cbw - 1][shape], dim3(grid), dim3(kGemmThreads), NS * stage_bytes(p.bl), s, a);
    int rc = record_hip(hipGetLastError());
    if (rc != SP_OK || a.nsplit == 1) return rc;
    const unsigned units = static_cast<unsigned>(a.nblocks) * kGemmWaves * p.cbw * 2 * p.vb;
    hipLaunchKernelGGL(join[p.cbw - 1][p.vb - 1], dim3((units + 3) / 4), dim3(kGemmThreads), 0, s, a);
    return record_hip(hipGetLastError());
}

}  // namespace sp3d
