// bf16 3x3 convolution of the 2-D variant (geometry flag `flat`) with 32 or 64 input channels: forward and, on mirrored weights,
// data gradient of the two finest levels of the paper's 2-D network (Sec. 3), whose layers move 128 or 256 bytes a voxel for 18
// or 74 kFLOP.
//
// A wave owns 32 columns of one slice and marches along H by itself: no barrier, no hand-over.  The weights of its 32 output
// channels (18 fragments an input chunk of 32 channels) stay in registers, as do the fragments of the last three input rows: a
// row is staged once, read from LDS once (six fragments a chunk, each into the registers of the row that falls out of the
// window, behind the products that used them last) and meets three output rows.  An output row is one chain of 18 products a
// chunk in the order (kw, K half, kh), and two chunks' chains are added at the end: the order of conv_mfma_kernel and
// conv_mfma_pair_kernel, so that a layer's bits do not depend on which of them serves it (narrow tiles, several slices side
// by side in a patch, stay there).  A row's conversion and stores stand between the products of the next one.
// v_mfma_f32_32x32x16_bf16, A = weights, B = voxels.
//
// Rows go from memory straight into the wave's ring in LDS, 34 records (32 channels, 64 bytes) a chunk of which 16 a load, R rows
// in flight or in use; the mask of the data gradient (kMask) has a ring of its own.  The 16-byte pieces of a record sit in
// the order piece ^ (column / 4 % 4) as in the other kernels.  Two workgroups of four waves on a compute unit with one chunk,
// one with two (512 registers a wave).
//
// What bounds it: HBM (32 input channels, large stacks), products (64), the first rows' way (small ones).  The patch marches, one
// workgroup per compute unit, stage 10 rows for 8 (6 for 4) and wait at a barrier every 36 products, and every march of
// theirs starts with an idle compute unit.  Figures of both: at launch_conv_rows2d.
#include "conv_mfma_common.h"

#include <algorithm>

namespace sp3d {

using namespace convk;

namespace {

constexpr int NTAP2 = 9, NWF = NTAP2 * 2, NGROUP = 6;         // weight fragments of a chunk; (kw, K half) groups
constexpr int ROW_REC = PW + 2;                               // records of a staged row
constexpr int ROW_LDS = ROW_REC * REC, MASK_LDS = PW * REC;   // of a chunk's row; of a mask row
constexpr int IN_LOADS = 3, MASK_LOADS = 2;                   // wave loads of 16 records (the third one: the last two records)
// NC input chunks of 32 channels: waves per SIMD, input rows and mask rows in the rings
constexpr int occupancy(int nc) { return nc == 1 ? 2 : 1; }
constexpr int ring(int nc, bool mask) { return mask ? (nc == 1 ? 5 : 6) : 8; }
constexpr int mask_ring(int nc, bool mask) { return mask ? ring(nc, mask) - 1 : 0; }
constexpr int wave_lds(int nc, bool mask) { return ring(nc, mask) * nc * ROW_LDS + mask_ring(nc, mask) * MASK_LDS; }
constexpr bool fits(int nc, bool mask) { return occupancy(nc) * kWaves * wave_lds(nc, mask) <= 160 * 1024; }
static_assert(fits(1, false) && fits(1, true) && fits(2, false) && fits(2, true), "LDS of a compute unit");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct RowArgs {
    const uint16_t *in[2];   // input chunk c: 32 channels at in[c], in_cs[c] channels per voxel
    int in_cs[2];
    const uint4 *wpack;      // [chunk][nco][27][2][64] x 16 bytes; the nine taps in slots 9 .. 17
    const float *bias;
    uint16_t *out, *out2;    // output channels [0, out_ca), out_cs per voxel / the rest (NULL: one tensor), out2_cs
    const uint16_t *mask;    // kMask: laid out like `out`
    int out_cs, out2_cs, out_ca;
    Geo g;
    int nco, nstrip, nchunk, rows;      // output blocks, strips of 32 columns, chunks of `rows` output rows
    int nwaves;
};

// 16 bytes per lane into LDS at dst + 16 lane: uniform base, 32-bit byte offset per lane.  (Assembly: the compiler, when it
// knows of such a load, waits for all outstanding ones before every LDS read.)
__device__ __forceinline__ void dma_row(const uint16_t *base, uint32_t off, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(dst) : "memory");
}

template <int NC, int EPI, bool HAS_BIAS>
__global__ __launch_bounds__(kThreads, occupancy(NC)) void conv_rows2d_kernel(RowArgs a) {
    constexpr bool MASK = EPI == kMask;
    constexpr int R = ring(NC, MASK), M = mask_ring(NC, MASK), LEAD_LOADS = NC * IN_LOADS + (MASK ? MASK_LOADS : 0);
    extern __shared__ __align__(128) char lds[];
    const int per_xcd = gridDim.x >> 3;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 31, hi = lane >> 5;
    int t = ((blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3)) * kWaves + wave;     // neighbours on one XCD
    if (t >= a.nwaves) return;
    const Geo &g = a.g;
    const int cj = t % a.nco; t /= a.nco;            // blocks of output channels first: they share the input rows
    const int strip = t % a.nstrip; t /= a.nstrip;
    const int chunk = t % a.nchunk; t /= a.nchunk;
    const int slice = t % g.td, tile = t / g.td;
    const TileBox bx = tile_box(g, tile);
    const int h0 = chunk * a.rows, w0 = strip * PW, n = min(a.rows, bx.bh - h0);
    if (n <= 0 || w0 >= bx.bw) return;

    bf16x8 wf[NC][NWF];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int f = 0; f < NWF; ++f) wf[c][f] = __builtin_bit_cast(bf16x8, a.wpack[((c * a.nco + cj) * NFRAG + 18 + f) * 64 + lane]);

    // the corner of the chunk's input rows; input row r (0 .. n + 1) is r rows further down
    const size_t vox0 = static_cast<size_t>(tile) * g.tile_vox + bx.org + (static_cast<size_t>(slice + 1) * g.ph + h0) * g.pw + w0;
    // columns outside the box and its surround repeat the last one (they only feed results that are not stored)
    const uint16_t *in0[NC];
    size_t irow[NC];
    uint32_t ioff[NC][IN_LOADS], moff[MASK_LOADS];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        in0[c] = a.in[c] + vox0 * a.in_cs[c];
        irow[c] = static_cast<size_t>(g.pw) * a.in_cs[c];
#pragma unroll
        for (int j = 0; j < IN_LOADS; ++j) {
            const int k = min(16 * j + (lane >> 2), ROW_REC - 1);
            ioff[c][j] = min(k, bx.bw + 1 - w0) * a.in_cs[c] * 2 + 16 * piece_at(k, lane & 3);
        }
    }
    const bool second = a.out2 && C * cj >= a.out_ca;
    const int ocs = second ? a.out2_cs : a.out_cs;
    const size_t oat = (vox0 + g.pw + 1) * ocs + C * cj - (second ? a.out_ca : 0), orow = static_cast<size_t>(g.pw) * ocs;
    const uint16_t *const mask0 = a.mask + oat;
    if (MASK) {
#pragma unroll
        for (int j = 0; j < MASK_LOADS; ++j) {
            const int k = 16 * j + (lane >> 2);
            moff[j] = min(k, bx.bw - 1 - w0) * ocs * 2 + 16 * piece_at(k, lane & 3);
        }
    }
    const uint32_t lds_in = lds_addr(lds) + wave * wave_lds(NC, MASK), lds_mask = lds_in + R * NC * ROW_LDS;
    int rin = 0, sin = 0, rmask = 0, smask = 0;      // next input row to fetch and its slot; next mask row and its slot
    // rows past the last one repeat it, so that every step issues the same loads
    auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint16_t *src = in0[c] + min(rin, n + 1) * irow[c];
            const uint32_t dst = lds_in + (sin * NC + c) * ROW_LDS;
            dma_row(src, ioff[c][0], dst);
            dma_row(src, ioff[c][1], dst + 1024);
            if (lane < 4 * (ROW_REC - 32)) dma_row(src, ioff[c][2], dst + 2048);
        }
        ++rin;
        sin = sin + 1 == R ? 0 : sin + 1;
    };
    auto fetch_mask = [&]() __attribute__((always_inline)) {
        if (!MASK) return;
        const uint16_t *src = mask0 + min(rmask, n - 1) * orow;
        const uint32_t dst = lds_mask + smask * MASK_LDS;
        dma_row(src, moff[0], dst);
        dma_row(src, moff[1], dst + 1024);
        ++rmask;
        smask = smask + 1 == M ? 0 : smask + 1;
    };

    char *const in_lds = lds + wave * wave_lds(NC, MASK), *const mask_lds = in_lds + R * NC * ROW_LDS;
    int boff[3];                                     // column lane % 32 + kw, piece lane / 32; the second K half's is 32 bytes away
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) boff[kw] = lds_off(col + kw, hi);
    bf16x8 bf[3][NC][NGROUP];                        // input row r in set r % 3
    int sread = 0;                                   // slot of the next row to read
    auto read_group = [&](int set, int gi) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            bf[set][c][gi] = *reinterpret_cast<const bf16x8 *>(in_lds + (sread * NC + c) * ROW_LDS + (boff[gi >> 1] ^ ((gi & 1) * 32)));
    };
    float bv[HAS_BIAS ? 16 : 1];
    if (HAS_BIAS) {
#pragma unroll
        for (int e = 0; e < 16; ++e) bv[HAS_BIAS ? e : 0] = a.bias[C * cj + 8 * (e >> 2) + 4 * hi + (e & 3)];
    }
    // Output rows leave as whole records: store j of a row writes columns 16 j + lane / 4, four lanes to a record.
    bool ok[2];
    uint32_t vo[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int k = 16 * j + (lane >> 2);
        ok[j] = w0 + k < bx.bw;
        vo[j] = k * ocs + 8 * piece_at(k, lane & 3);
    }
    uint16_t *out = (second ? a.out2 : a.out) + oat;
    int srmask = 0;

    // Output row i - 1, whose sums were completed a step ago, in three parts that stand between the products of step i.
    f32x16 sums[NC];                                 // of output row i - 1
    char *turn;
    uint4 mv[2];
    // Parts 0 and 1: convert 16 channels; the two lanes of a voxel exchange halves, so that each has 8 consecutive ones.  The row is
    // turned into whole records in a slot that the loads at the step's end fill: the mask row's, or that of input row i + 1, whose
    // fragments are in registers (sin is its number).
    auto convert = [&](int p) __attribute__((always_inline)) {
        if (p == 0) {
            turn = MASK ? mask_lds + srmask * MASK_LDS : in_lds + sin * NC * ROW_LDS;
            if (MASK) {
#pragma unroll
                for (int k = 0; k < 2; ++k) mv[k] = *reinterpret_cast<const uint4 *>(turn + lds_off(col, 2 * k + hi));
                srmask = srmask + 1 == M ? 0 : srmask + 1;
            }
        }
        uint2 pk[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = sums[0][8 * p + 4 * q + e];
                if (NC == 2) v[e] += sums[NC - 1][8 * p + 4 * q + e];
                if (is_relu(EPI)) v[e] = relu_f32(v[e]);
            }
            pk[q] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        }
        const auto x = __builtin_amdgcn_permlane32_swap(pk[0].x, pk[1].x, false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(pk[0].y, pk[1].y, false, false);
        uint4 v = make_uint4(x[0], y[0], x[1], y[1]);
        if (MASK) {
            v.x &= positive_halves(mv[p].x);
            v.y &= positive_halves(mv[p].y);
            v.z &= positive_halves(mv[p].z);
            v.w &= positive_halves(mv[p].w);
        }
        *reinterpret_cast<uint4 *>(turn + lds_off(col, 2 * p + hi)) = v;
    };
    // Part 2, a group or more behind part 1: store.
    auto store = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(turn + j * 1024 + lane * 16);
            if (ok[j]) __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(out + vo[j]));
        }
        out += orow;
    };

    // Step i, phase i mod 3: products of output row i, whose input rows i, i + 1, i + 2 are in sets i, i + 1, i + 2 (mod 3), and the end of
    // output row i - 1 (DONE).
    auto step = [&](auto phase, auto done_tag) __attribute__((always_inline)) {
        constexpr int SET = decltype(phase)::value;
        constexpr bool DONE = decltype(done_tag)::value;
        // Row i + 3 (and the mask of row i - 1) have landed: the loads issued after them are those of R - 3 later steps; the
        // stores among them only ask for more.
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R - 3) * LEAD_LOADS) : "memory");
        f32x16 acc[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[c][e] = HAS_BIAS && c == 0 ? bv[HAS_BIAS ? e : 0] : 0.f;
#pragma unroll
        for (int gi = 0; gi < NGROUP; ++gi) {
#pragma unroll
            for (int kh = 0; kh < 3; ++kh)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[c][(kh * 3 + (gi >> 1)) * 2 + (gi & 1)],
                                                                     bf[(SET + kh) % 3][c][gi], acc[c], 0, 0, 0);
            read_group(SET, gi);
            if (DONE && (gi == 1 || gi == 2)) convert(gi - 1);
            if (DONE && gi == 4) store();
            __builtin_amdgcn_sched_barrier(0);
        }
        sread = sread + 1 == R ? 0 : sread + 1;
        // behind the last reads of the slots that the next loads fill (newer than the row's: this step's last group)
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(NC) : "memory");
        fetch();
        fetch_mask();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < NC; ++c) sums[c] = acc[c];
    };

    // Loads in the order of the steps -(R - 2) ... -1: input row i + R + 1 and mask row i + R - 2 together.
#pragma unroll
    for (int r = 0; r < 3; ++r) fetch();
#pragma unroll
    for (int r = 3; r < R; ++r) { fetch(); fetch_mask(); }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R - 3) * LEAD_LOADS) : "memory");
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int gi = 0; gi < NGROUP; ++gi) read_group(r, gi);
        ++sread;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // slot 0 is free
    __builtin_amdgcn_sched_barrier(0);
    fetch();
    fetch_mask();
    __builtin_amdgcn_sched_barrier(0);
    // (the first step stands before the loop: the compiler's waits for the weights, which know nothing of the rows on their
    // way and so wait for those too, are in it)
    step(std::integral_constant<int, 0>{}, std::false_type{});
    for (int left = n - 1; left > 0;) {
        step(std::integral_constant<int, 1>{}, std::true_type{});
        if (--left == 0) break;
        step(std::integral_constant<int, 2>{}, std::true_type{});
        if (--left == 0) break;
        step(std::integral_constant<int, 0>{}, std::true_type{});
        --left;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the last row's mask; the repeated rows
    convert(0);
    convert(1);
    store();
}

}  // namespace

// Chunks of rows: a march costs its rows, the two of the surround and about six rows' time before its first product, and 2048
// waves (1024 with two chunks) fit on the chip at once.  Where the tensors do not fit the 256 MB of memory-side cache, half as many waves on marches
// twice as long touch memory in fewer places and are faster, as eight waves of a compute unit are no longer what its memory
// share is waiting for (16 x 512^2 in 1 x 2 x 2 tiles, 64 -> 128 rows: 32 -> 32 122 -> 113 us, 32 -> 64 241 (128 rows) -> 201 (256);
// but 32 -> 64 on 16 x 256^2, 201 MB, 64 -> 32 rows 49 -> 43).
// Measured with the packing of the weights, patch march -> this: 32 -> 32 on 16 x 512^2 in 1 x 2 x 2 tiles forward 158 -> 102 us (5.3
// TB/s), masked data gradient 191 -> 158 (5.1), 32 -> 64 397 -> 255, 64 -> 32 255 -> 167; 64 -> 64 on 16 x 256^2 124 -> 76 (1.0 PFLOP/s),
// masked 167 -> 106, on 11 x 390 x 410 253 -> 136, on 9 x 64 x 96 14.7 -> 12.2; 32 -> 32 on 2 x 512^2 36 -> 15, on 480^2 29 -> 10, on 7 x
// 64^2 8.1 -> 5.9.  Copies of such tensors reach 6.4 TB/s; stores of 32 bytes a voxel instead of whole records cost 5 to 20 %.
int launch_conv_rows2d(const void *Pin, const void *wpack, const float *bias, void *Pout, const Geo &g, int ki, int ko, bool relu,
                       hipStream_t s, const void *mask, const ConvSplit *split) {
    RowArgs a;
    const int nc = ki / C;
    a.in[0] = static_cast<const uint16_t *>(Pin);
    a.in[1] = a.in[0] + C;
    a.in_cs[0] = a.in_cs[1] = ki;
    if (split && split->in2) {
        a.in[1] = static_cast<const uint16_t *>(split->in2);
        a.in_cs[0] = a.in_cs[1] = C;
    }
    a.wpack = static_cast<const uint4 *>(wpack);
    a.bias = bias;
    a.out = static_cast<uint16_t *>(Pout);
    a.out2 = nullptr;
    a.out_cs = a.out_ca = ko;
    a.out2_cs = 0;
    if (split && split->out2) {
        a.out2 = static_cast<uint16_t *>(split->out2);
        a.out_cs = a.out_ca = split->out_ca;
        a.out2_cs = ko - split->out_ca;
    }
    a.mask = static_cast<const uint16_t *>(mask);
    a.g = g;
    a.nco = ko / C;
    const int eh = g.th + 2 * g.grow, ew = g.tw + 2 * g.grow;
    a.nstrip = (ew + PW - 1) / PW;
    const long long marches = 1LL * g.ntiles * g.td * a.nstrip * a.nco;
    a.nchunk = 1;
    const long long vox = 1LL * g.ntiles * g.td * eh * ew;
    const long long fit = 1024 * (occupancy(nc) == 2 && vox * 2 * (ki + ko * (mask ? 2 : 1)) <= (256LL << 20) ? 2 : 1);
    double least = 0;
    for (int k = 1; k <= eh && (k == 1 || marches * k <= 16384); ++k) {
        const double cost = static_cast<double>((marches * k + fit - 1) / fit) * ((eh + k - 1) / k + 8);
        if (k == 1 || cost < least) { least = cost; a.nchunk = k; }
    }
    a.rows = (eh + a.nchunk - 1) / a.nchunk;
    const long long nw = marches * a.nchunk;
    if (nw > 0x7fffffc0LL) return SP_EGEOM;
    a.nwaves = static_cast<int>(nw);
    const unsigned grid = static_cast<unsigned>(((nw + kWaves - 1) / kWaves + 7) / 8 * 8);
    const int epi = mask ? kMask : (relu ? kRelu : kNone);
    using Kern = void (*)(RowArgs);
    // [chunks - 1][bias][epilogue]
    static const Kern kern[2][2][3] = {
        {{conv_rows2d_kernel<1, kNone, false>, conv_rows2d_kernel<1, kRelu, false>, conv_rows2d_kernel<1, kMask, false>},
         {conv_rows2d_kernel<1, kNone, true>, conv_rows2d_kernel<1, kRelu, true>, conv_rows2d_kernel<1, kMask, false>}},
        {{conv_rows2d_kernel<2, kNone, false>, conv_rows2d_kernel<2, kRelu, false>, conv_rows2d_kernel<2, kMask, false>},
         {conv_rows2d_kernel<2, kNone, true>, conv_rows2d_kernel<2, kRelu, true>, conv_rows2d_kernel<2, kMask, false>}}};
    // more than 64 KB of dynamic LDS has to be requested explicitly
    static const hipError_t attr = [] {
        for (int i = 0; i < 12; ++i) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern[i / 6][(i / 3) % 2][i % 3]),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kWaves * wave_lds(i / 6 + 1, i % 3 == kMask));
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (attr != hipSuccess) return record_hip(attr);
    hipLaunchKernelGGL(kern[nc - 1][bias ? 1 : 0][epi], dim3(grid), dim3(kThreads), kWaves * wave_lds(nc, epi == kMask), s, a);
    return record_hip(hipGetLastError());
}

}  // namespace sp3d
