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
// A K step is one kernel row (three taps kw) x one 32-channel input chunk.  Both operands come through LDS by
// direct loads, NS stages deep (one barrier per step, placed before the step's last MFMA group, so that the next
// step's first fragments are read behind it while that group runs):
//   A (weights): the packed fragments of conv_mfma.hip, 1 KB each, lane-major.
//   B (voxels): the records (32 channels, 64 bytes) of the padded rows that the tile's voxels touch, each ONCE for the
//     three taps of the row: voxel q of a box row of ew voxels is record (q / ew) (ew + 2) + q % ew, and the taps read
//     this record and the two after it.  The 16-byte pieces of a record sit in the order piece ^ (record / 4 % 4), so
//     that the 16-byte reads of 16 neighbouring voxels fall into 16 different bank groups.
// (v_mfma_f32_32x32x16_bf16, A = weights [32 output channels][16 input channels], B = voxels [16 input channels][32
// voxels]; four waves, two along output channels x two along voxels.)
// What bounds it: in its first form the B fragments were fetched by the lanes themselves, 16 bytes of 64 different
// lines per load, and the vector cache's one line per clock held the step at 0.9 (128 voxels) and 2.1 us (256 voxels),
// three times its MFMAs; with up to 32 workgroups and no split the bottom level of the 3-D network took 250 us a layer.
// Now, first form -> this one: 1024 -> 1024 on 8^3 voxels (3-D) 250 -> 31 + 9 us (its 57 MB of weights: 7 us of HBM), 512 ->
// 512 on 16^3 150 -> 64 + 9 us (0.9 PFLOP/s), 2-D on two slices 1024 -> 1024 on 16 x 16 88 -> 22 + 6 us (a launch, a pipeline
// of three stages and 12 steps: latency), 512 -> 512 on 16 slices of 32 x 32 115 -> 100 us.
//
// Output box growth, two input tensors (concatenation without a copy), two output tensors, bias, ReLU, the ReLU mask
// of the data gradient, its one-bit forms and gathered halos behave as in conv_mfma.hip.  The order of the additions
// is fixed (kernel rows, then chunks, then taps within a split; then the splits), and the split depends on the layer's
// interior voxel count and channels only, so results are reproducible and depend neither on the voxel's position nor on
// the tile grid.
#include "conv_mfma_common.h"

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
constexpr int stage_bytes(int cbw, int bl) { return (2 * cbw * ROW * 2 + 4 * bl) * 1024; }
// LDS stages: four for wide workgroups, one per compute unit; three where two workgroups then share one
constexpr int stages(int cbw, int bl) { return cbw == 2 && 4 * stage_bytes(2, bl) <= 160 * 1024 ? 4 : 3; }

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

// Output voxel q: padded voxel index, and whether it exists (past the end, or outside the box of a tile without a
// neighbour on that side: no).
struct OutVox { long long pv; bool ok; };
__device__ __forceinline__ OutVox out_vox(const GemmArgs &a, int q) {
    const uint32_t qq = static_cast<uint32_t>(min(q, a.nvox - 1)), row = fdiv(qq, a.drow);
    BoxPos p = row_pos(a, row);
    p.w = static_cast<int>(fmod_(qq, row, a.drow));
    const TileBox bx = tile_box(a.g, p.tile);
    OutVox o;
    o.ok = q < a.nvox && p.d < bx.bd && p.h < bx.bh && p.w < bx.bw;
    o.pv = static_cast<long long>(p.tile) * a.g.tile_vox + bx.org + (1LL * (p.d + 1) * a.g.ph + p.h + 1) * a.g.pw + p.w + 1;
    return o;
}

// Finished sums of one voxel, 16 channels (8 q + 4 hi + i) of output block cj: ReLU / mask, convert, 8-byte stores.
__device__ __forceinline__ void finish(const GemmArgs &a, const f32x16 &s, int cj, int hi, const OutVox &o) {
    if (!o.ok) return;
    const int co = C * cj;
    uint16_t *obase = a.out;
    int ocs = a.out_cs, oco = co;
    if (a.out2 && co >= a.out_ca) { obase = a.out2; ocs = a.out2_cs; oco = co - a.out_ca; }
    uint16_t *dst = obase + o.pv * ocs + oco + 4 * hi;
    const uint16_t *m = a.mask + o.pv * a.out_cs + co + 4 * hi;
    uint16_t *word = a.bits + (o.pv * a.nco + cj) * 2 + hi;
    uint32_t bits = 0;
    if (a.epi == kMaskBits) bits = spread_word(*word);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = s[4 * q + i];
            if (is_relu(a.epi)) v[i] = a.relu_keeps_nan ? (v[i] < 0.f ? 0.f : v[i]) : relu_f32(v[i]);
        }
        uint2 pk = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        if (a.epi == kMask) {
            const uint2 mv = *reinterpret_cast<const uint2 *>(m + 8 * q);
            pk.x &= positive_halves(mv.x);
            pk.y &= positive_halves(mv.y);
        }
        if (a.epi == kMaskBits) {
            const uint2 mv = nibble_halves(bits, q);
            pk.x &= mv.x;
            pk.y &= mv.y;
        }
        if (a.epi == kReluBits) {
#pragma unroll
            for (int i = 0; i < 4; ++i) bits = shift_in_positive(bits, v[i]);
        }
        *reinterpret_cast<uint2 *>(dst + 8 * q) = pk;
    }
    if (a.epi == kReluBits) *word = row_word(bits);
}

// Sums of a split: unit (tile, wave, block of the wave, segment, q) x 64 lanes x 4 channels, 1 KB per unit.
template <int CBW, int VB>
__device__ __forceinline__ size_t part_index(const GemmArgs &a, int split, int blk, int wave, int c, int s, int lane) {
    return (((static_cast<size_t>(split) * a.nblocks + blk) * kGemmWaves + wave) * CBW * 2 * VB + c * 2 * VB + s) * 256 + lane;
}

template <int CBW, int VB, int BL>
__global__ __launch_bounds__(kGemmThreads, 1) void conv_gemm_kernel(GemmArgs a) {
    constexpr int NSEG = 2 * VB, CBT = 2 * CBW, AFRAGS = CBT * ROW * 2, AL = AFRAGS / kGemmWaves, L = AL + BL;
    constexpr int STAGE = stage_bytes(CBW, BL), NS = stages(CBW, BL);
    static_assert((NS - 1) * L < 64, "vmcnt");
    extern __shared__ __align__(16) char lds[];
    // workgroups of one XCD (blockIdx % 8) get consecutive logical ids: they share output blocks and K range, i.e. weights
    const int per_xcd = gridDim.x >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= a.nblocks * a.nsplit) return;
    const Geo &g = a.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave & 1, wn = wave >> 1, hi = lane >> 5;
    const int vg = logical % a.nvg, u = logical / a.nvg, split = u % a.nsplit, cg = u / a.nsplit;
    const long long prow = g.pw, pplane = static_cast<long long>(g.ph) * g.pw;
    const int q0 = vg * wg_vox(VB);
    auto record = [&](int q) {
        const uint32_t row = fdiv(static_cast<uint32_t>(q), a.drow);
        return row * (a.ew + 2) + fmod_(static_cast<uint32_t>(q), row, a.drow);
    };
    const uint32_t rec0 = record(q0), nrec = record(min(q0 + wg_vox(VB), a.nvox) - 1) + 3 - rec0;

    // This lane's share of the record loads: records 16 (BL wave + j) + lane / 4, piece lane % 4 of each (stored order).
    // Records past the last one repeat it; records of rows that a tile's own box lacks are moved inside it (both only
    // feed results that are dropped).
    long long rpos[BL];
    int rflag[BL];                   // gathered halos: bit 0 / 1 first / last row with a neighbour, 2 / 3 plane
    const long long sw = g.tile_vox - g.tw, sh = g.tile_vox * g.gw - g.th * prow, sd = g.tile_vox * g.gw * g.gh - g.td * pplane;
#pragma unroll
    for (int j = 0; j < BL; ++j) {
        const uint32_t k = min(static_cast<uint32_t>(16 * (BL * wave + j) + (lane >> 2)), nrec - 1) + rec0;
        const uint32_t row = fdiv(k, a.drec);
        BoxPos p = row_pos(a, row);
        const TileBox bx = tile_box(g, p.tile);
        p.d = min(p.d, bx.bd - 1);
        p.h = min(p.h, bx.bh - 1);
        p.w = min(static_cast<int>(fmod_(k, row, a.drec)), bx.bw + 1);
        rpos[j] = static_cast<long long>(p.tile) * g.tile_vox + bx.org + (p.d + 1) * pplane + (p.h + 1) * prow + p.w;
        rflag[j] = 0;
        if (a.gather) {              // (host: one-voxel margins, no grown box, 3-D)
            const int tc = p.tile % g.gw, t1 = p.tile / g.gw, tb = t1 % g.gh, ta = (t1 / g.gh) % g.gd;
            if (p.w == 0 && tc > 0) rpos[j] -= sw;
            if (p.w == g.tw + 1 && tc < g.gw - 1) rpos[j] += sw;
            rflag[j] = (p.h == 0 && tb > 0 ? 1 : 0) | (p.h == g.th - 1 && tb < g.gh - 1 ? 2 : 0) |
                       (p.d == 0 && ta > 0 ? 4 : 0) | (p.d == g.td - 1 && ta < g.gd - 1 ? 8 : 0);
        }
    }
    const int piece = 8 * ((lane & 3) ^ (lane >> 4));
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char *)lds));

    // K range of this split
    const int nk = a.nci * a.nrows;
    const int k0 = static_cast<int>(1LL * split * nk / a.nsplit), k1 = static_cast<int>(1LL * (split + 1) * nk / a.nsplit);
    int fk = k0, fr = k0 / a.nci, fi = k0 - fr * a.nci;         // next step to fetch: kernel row fr, chunk fi (innermost: the
                                                                // record of two neighbouring chunks is one cache line)
    auto fetch = [&](int stage) {
        const int tap0 = (a.nrows == 3 ? 9 : 0) + ROW * fr;
        const uint32_t dst = lds0 + stage * STAGE;
#pragma unroll
        for (int n = 0; n < AL; ++n) {
            const int m = wave * AL + n, cb = m / (ROW * 2), x = m - cb * (ROW * 2);
            const size_t frag = (static_cast<size_t>(fi * a.nco + cg * CBT + cb) * NTAP_PACK + tap0) * 2 + x;
            dma16(a.wpack + frag * 64 + lane, dst + m * 1024);
        }
        const InSrc src = in_src(a, fi);
        const int kd = a.nrows == 3 ? 1 : fr / 3, kh = a.nrows == 3 ? fr : fr - 3 * (fr / 3);
        const long long ro = (kd - 1) * pplane + (kh - 1) * prow;
        const long long gh = kh == 0 ? -sh : sh, gd = kd == 0 ? -sd : sd;
        const int mh = kh == 0 ? 1 : (kh == 2 ? 2 : 0), md = kd == 0 ? 4 : (kd == 2 ? 8 : 0);
        const uint16_t *base = src.base + src.co + piece;
#pragma unroll
        for (int j = 0; j < BL; ++j) {
            long long at = rpos[j] + ro;
            if (a.gather) at += (rflag[j] & mh ? gh : 0) + (rflag[j] & md ? gd : 0);
            dma16(base + at * src.cs, dst + (AFRAGS + BL * wave + j) * 1024);
        }
        if (fk + 1 < k1) {           // past the last step the loads repeat it: what they fill is never used
            ++fk;
            if (++fi == a.nci) { fi = 0; ++fr; }
        }
    };

    // this lane's read offsets inside a stage: record of its voxel in segment s, one and two records on
    int boff[NSEG][ROW];
#pragma unroll
    for (int s = 0; s < NSEG; ++s) {
        const int q = min(q0 + wn * 64 * VB + s * 32 + (lane & 31), a.nvox - 1);
        const int r = static_cast<int>(record(q) - rec0);
#pragma unroll
        for (int kw = 0; kw < ROW; ++kw) boff[s][kw] = AFRAGS * 1024 + (r + kw) * 64 + ((hi ^ ((r + kw) >> 2)) & 3) * 16;
    }

    // accumulators start from the bias (in the first split): lane l holds channels 8 (e / 4) + 4 (l / 32) + e % 4 of a block
    f32x16 acc[CBW][NSEG];
    const bool biased = a.bias && split == 0;
#pragma unroll
    for (int c = 0; c < CBW; ++c) {
        f32x16 v;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            v[e] = biased ? a.bias[C * (cg * CBT + wm * CBW + c) + 8 * (e >> 2) + 4 * hi + (e & 3)] : 0.f;
#pragma unroll
        for (int s = 0; s < NSEG; ++s) acc[c][s] = v;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // (the bias: from here on only the staged loads are counted)

    bf16x8 wf[2][CBW], bf[2][NSEG];
    auto read_group = [&](const char *stage, int gi) {          // (kw, K-half) group gi -> fragment set gi % 2
        const int kw = gi >> 1, half = gi & 1;
#pragma unroll
        for (int c = 0; c < CBW; ++c)
            wf[gi & 1][c] = *reinterpret_cast<const bf16x8 *>(stage + (((wm * CBW + c) * ROW + kw) * 2 + half) * 1024 + lane * 16);
#pragma unroll
        for (int s = 0; s < NSEG; ++s) bf[gi & 1][s] = *reinterpret_cast<const bf16x8 *>(stage + (boff[s][kw] ^ (half * 32)));
    };

#pragma unroll
    for (int i = 0; i < NS; ++i) fetch(i);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * L) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_group(lds, 0);
    int cur = 0;
    for (int k = k0; k < k1; ++k) {
        const int nxt = cur + 1 == NS ? 0 : cur + 1;
        const char *const stage = lds + cur * STAGE;
#pragma unroll
        for (int gi = 0; gi < 2 * ROW; ++gi) {
            if (gi + 1 < 2 * ROW) {
                read_group(stage, gi + 1);
            } else {
                // every wave has read this step's last fragments (lgkmcnt) and the next step's loads have landed: those
                // of the NS - 2 steps after it may stay in flight.  Behind the barrier this step's stage is free.
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * L) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                read_group(lds + nxt * STAGE, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (gi + 1 == 2 * ROW) fetch(cur);
#pragma unroll
            for (int c = 0; c < CBW; ++c)
#pragma unroll
                for (int s = 0; s < NSEG; ++s)
                    acc[c][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[gi & 1][c], bf[gi & 1][s], acc[c][s], 0, 0, 0);
        }
        cur = nxt;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the repeated loads

    const int blk = cg * a.nvg + vg;
#pragma unroll
    for (int s = 0; s < NSEG; ++s) {
        const OutVox o = out_vox(a, q0 + wn * 64 * VB + s * 32 + (lane & 31));
#pragma unroll
        for (int c = 0; c < CBW; ++c) {
            if (a.nsplit == 1) {
                finish(a, acc[c][s], cg * CBT + wm * CBW + c, hi, o);
            } else {
                float4 *p = a.part + part_index<CBW, VB>(a, split, blk, wave, c, s, lane);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    p[64 * q] = make_float4(acc[c][s][4 * q], acc[c][s][4 * q + 1], acc[c][s][4 * q + 2], acc[c][s][4 * q + 3]);
            }
        }
    }
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
    finish(a, sum, cg * 2 * CBW + wm * CBW + c, lane >> 5, out_vox(a, vg * wg_vox(VB) + wn * 64 * VB + s * 32 + (lane & 31)));
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
// Voxels per workgroup and splits of the K loop: what costs least in microseconds if 256 compute units take the workgroups
// in rounds: a step lasts 0.41 us per 128 voxels x 64 channels, a workgroup 10.7 us besides (launch, first loads, stores);
// splitting adds a second launch and a write and a read of every sum at about 6 TB/s.  The interior voxels alone decide, so
// that the order of the sums is the same for every output box growth and tile grid.  The time that is then compared with the
// marching kernels' has constants of its own, fitted to 472 layers cut this way (32 ... 1024 channels, 64 voxels ... 4 million,
// 2-D and 3-D; 11 % rms; `shortk`, K loops of 3 or 6 steps: 354 layers, 6 % rms): the layers of 64 channels a workgroup
// take 7 % longer than the first constants say, and short loops do not reach the rate of a step.
GemmPlan plan_gemm(const Geo &g, int ki, int ko) {
    GemmPlan p;
    const Box b = max_box(g);
    p.nvox = 1LL * g.ntiles * b.ed * b.eh * b.ew;
    const int nco = ko / C, nk = ki / C * (g.flat ? 3 : 9);
    const long long nint = 1LL * g.ntiles * g.int_vox;
    p.cbw = nco % 4 == 0 ? 2 : 1;
    const bool shortk = g.flat && ki <= 2 * C;
    double least = 0;
    for (int vb = 1; vb <= 2; ++vb) {
        const long long tiles = (nint + wg_vox(vb) - 1) / wg_vox(vb) * (nco / (2 * p.cbw));
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
    // [output blocks per wave - 1][(voxels, record loads)]
    static const Kern kern[2][5] = {{conv_gemm_kernel<1, 1, 3>, conv_gemm_kernel<1, 1, 4>, conv_gemm_kernel<1, 1, 6>,
                                     conv_gemm_kernel<1, 2, 5>, conv_gemm_kernel<1, 2, 6>},
                                    {conv_gemm_kernel<2, 1, 3>, conv_gemm_kernel<2, 1, 4>, conv_gemm_kernel<2, 1, 6>,
                                     conv_gemm_kernel<2, 2, 5>, conv_gemm_kernel<2, 2, 6>}};
    static const Kern join[2][2] = {{conv_gemm_join_kernel<1, 1>, conv_gemm_join_kernel<1, 2>},
                                    {conv_gemm_join_kernel<2, 1>, conv_gemm_join_kernel<2, 2>}};
    static const int bls[5] = {3, 4, 6, 5, 6};
    // more than 64 KB of dynamic LDS has to be requested explicitly
    static const hipError_t attr = [] {
        for (int i = 0; i < 10; ++i) {
            const int cbw = i / 5 + 1, bl = bls[i % 5];
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern[i / 5][i % 5]),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, stages(cbw, bl) * stage_bytes(cbw, bl));
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (attr != hipSuccess) return record_hip(attr);
    const int shape = p.vb == 2 ? (p.bl == 5 ? 3 : 4) : (p.bl == 3 ? 0 : (p.bl == 4 ? 1 : 2));
    const unsigned grid = static_cast<unsigned>((1LL * a.nblocks * a.nsplit + 7) / 8 * 8);
    hipLaunchKernelGGL(kern[p.cbw - 1][shape], dim3(grid), dim3(kGemmThreads), stages(p.cbw, p.bl) * stage_bytes(p.cbw, p.bl), s, a);
    int rc = record_hip(hipGetLastError());
    if (rc != SP_OK || a.nsplit == 1) return rc;
    const unsigned units = static_cast<unsigned>(a.nblocks) * kGemmWaves * p.cbw * 2 * p.vb;
    hipLaunchKernelGGL(join[p.cbw - 1][p.vb - 1], dim3((units + 3) / 4), dim3(kGemmThreads), 0, s, a);
    return record_hip(hipGetLastError());
}

}  // namespace sp3d
