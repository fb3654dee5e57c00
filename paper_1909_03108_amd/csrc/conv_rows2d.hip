// bf16 3x3 convolution of the 2-D variant (geometry flag `flat`) with 32 input channels: forward and, on mirrored weights, data
// gradient of the finest level of the paper's 2-D network (Sec. 3), whose layers move 128 bytes a voxel for 18 kFLOP and are
// bound by memory.
//
// A wave owns 32 columns of one slice and marches along H by itself: no barrier, no hand-over.  The nine taps' weights (18
// fragments) stay in registers, as do the fragments of the last three input rows: a row is staged once, read from LDS once
// (six fragments, each into the registers of the row that falls out of the window, behind the products that used them
// last) and meets three output rows.  An output row is one chain of 18 products in the order (kw, K half, kh), the order of
// conv_mfma_kernel, so that a layer's bits do not depend on which of the two serves it (narrow tiles, several slices side by
// side in a patch, stay there).  v_mfma_f32_32x32x16_bf16, A = weights, B = voxels.
//
// Rows go from memory straight into the wave's ring in LDS, 34 records (32 channels, 64 bytes) of which 16 a load, R rows in
// flight or in use; the mask of the data gradient (kMask) has a ring of its own.  The 16-byte pieces of a record sit in the
// order piece ^ (column / 4 % 4) as in the other kernels.  Two workgroups of four waves on a compute unit.
//
// What bounds it: HBM (large stacks), the first rows' way (small ones).  The patch march, one workgroup per compute unit, stages
// 10 rows for 8, waits at a barrier every 36 products and starts every march with an idle chip.  Figures of both: at
// launch_conv_rows2d.
#include "conv_mfma_common.h"

#include <algorithm>

namespace sp3d {

using namespace convk;

namespace {

constexpr int NTAP2 = 9, NWF = NTAP2 * 2, NGROUP = 6;         // weight fragments; (kw, K half) groups
constexpr int ROW_REC = PW + 2;                               // records of a staged row
constexpr int ROW_LDS = ROW_REC * REC, MASK_LDS = PW * REC;
constexpr int IN_LOADS = 3, MASK_LOADS = 2;                   // wave loads of 16 records (the third one: the last two records)
constexpr int ring(bool mask) { return mask ? 5 : 8; }        // input rows
constexpr int mask_ring(bool mask) { return mask ? 4 : 0; }
constexpr int wave_lds(bool mask) { return ring(mask) * ROW_LDS + mask_ring(mask) * MASK_LDS; }
static_assert(2 * kWaves * wave_lds(false) <= 160 * 1024 && 2 * kWaves * wave_lds(true) <= 160 * 1024, "two workgroups");

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct RowArgs {
    const uint16_t *in;
    const uint4 *wpack;      // [1][nco][27][2][64] x 16 bytes; the nine taps in slots 9 .. 17
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

template <int EPI, bool HAS_BIAS>
__global__ __launch_bounds__(kThreads, 2) void conv_rows2d_kernel(RowArgs a) {
    constexpr bool MASK = EPI == kMask;
    constexpr int R = ring(MASK), M = mask_ring(MASK), LEAD_LOADS = IN_LOADS + (MASK ? MASK_LOADS : 0);
    static_assert(!MASK || M == R - 1, "mask row i and input row i + 3 are fetched together, R - 1 steps before step i");
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

    bf16x8 wf[NWF];
#pragma unroll
    for (int f = 0; f < NWF; ++f) wf[f] = __builtin_bit_cast(bf16x8, a.wpack[(cj * NFRAG + 18 + f) * 64 + lane]);

    // the corner of the chunk's input rows; input row r (0 .. n + 1) is r rows further down
    const size_t vox0 = static_cast<size_t>(tile) * g.tile_vox + bx.org + (static_cast<size_t>(slice + 1) * g.ph + h0) * g.pw + w0;
    const uint16_t *in0 = a.in + vox0 * C;
    const size_t irow = static_cast<size_t>(g.pw) * C;
    // columns outside the box and its surround repeat the last one (they only feed results that are not stored)
    uint32_t ioff[IN_LOADS], moff[MASK_LOADS];
#pragma unroll
    for (int j = 0; j < IN_LOADS; ++j) {
        const int c = min(16 * j + (lane >> 2), ROW_REC - 1);
        ioff[j] = min(c, bx.bw + 1 - w0) * REC + 16 * piece_at(c, lane & 3);
    }
    const bool second = a.out2 && C * cj >= a.out_ca;
    const int ocs = second ? a.out2_cs : a.out_cs;
    const size_t oat = (vox0 + g.pw + 1) * ocs + C * cj - (second ? a.out_ca : 0), orow = static_cast<size_t>(g.pw) * ocs;
    uint16_t *const out0 = (second ? a.out2 : a.out) + oat;
    const uint16_t *const mask0 = a.mask + oat;
    if (MASK) {
#pragma unroll
        for (int j = 0; j < MASK_LOADS; ++j) {
            const int c = 16 * j + (lane >> 2);
            moff[j] = min(c, bx.bw - 1 - w0) * ocs * 2 + 16 * piece_at(c, lane & 3);
        }
    }
    const uint32_t lds_in = lds_addr(lds) + wave * wave_lds(MASK), lds_mask = lds_in + R * ROW_LDS;
    int rin = 0, sin = 0, rmask = 0, smask = 0;      // next input row to fetch and its slot; next mask row and its slot
    // rows past the last one repeat it, so that every step issues the same loads
    auto fetch = [&]() __attribute__((always_inline)) {
        const uint16_t *src = in0 + min(rin, n + 1) * irow;
        const uint32_t dst = lds_in + sin * ROW_LDS;
        dma_row(src, ioff[0], dst);
        dma_row(src, ioff[1], dst + 1024);
        if (lane < 4 * (ROW_REC - 32)) dma_row(src, ioff[2], dst + 2048);
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

    char *const in_lds = lds + wave * wave_lds(MASK), *const mask_lds = in_lds + R * ROW_LDS;
    int boff[3];                                     // column lane % 32 + kw, piece lane / 32; the second K half's is 32 bytes away
#pragma unroll
    for (int kw = 0; kw < 3; ++kw) boff[kw] = lds_off(col + kw, hi);
    bf16x8 bf[3][NGROUP];                            // input row r in set r % 3
    int sread = 0;                                   // slot of the next row to read
    auto read_group = [&](int set, int gi) __attribute__((always_inline)) {
        bf[set][gi] = *reinterpret_cast<const bf16x8 *>(in_lds + sread * ROW_LDS + (boff[gi >> 1] ^ ((gi & 1) * 32)));
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
        const int c = 16 * j + (lane >> 2);
        ok[j] = w0 + c < bx.bw;
        vo[j] = c * ocs + 8 * piece_at(c, lane & 3);
    }
    uint16_t *out = out0;
    int srmask = 0;

    // Output row i: input rows i, i + 1, i + 2 are in sets SET, SET + 1, SET + 2 (mod 3).
    auto step = [&](auto set_tag) __attribute__((always_inline)) {
        constexpr int SET = decltype(set_tag)::value;
        // Row i + 3 (and the mask of row i) have landed: the loads issued after them are those of R - 2 later steps; the
        // stores among them only ask for more.
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R - 2) * LEAD_LOADS) : "memory");
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = HAS_BIAS ? bv[HAS_BIAS ? e : 0] : 0.f;
#pragma unroll
        for (int gi = 0; gi < NGROUP; ++gi) {
#pragma unroll
            for (int kh = 0; kh < 3; ++kh)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[(kh * 3 + (gi >> 1)) * 2 + (gi & 1)], bf[(SET + kh) % 3][gi], acc, 0, 0, 0);
            read_group(SET, gi);
        }
        uint4 mv[2];
        // The row is turned into whole records in the slot that the loads at the step's end fill next: the mask row's, or that of
        // input row i + 2, whose fragments are in registers (sin is its number).
        char *const turn = MASK ? mask_lds + srmask * MASK_LDS : in_lds + sin * ROW_LDS;
        if (MASK) {
#pragma unroll
            for (int p = 0; p < 2; ++p) mv[p] = *reinterpret_cast<const uint4 *>(turn + lds_off(col, 2 * p + hi));
            srmask = srmask + 1 == M ? 0 : srmask + 1;
        }
        sread = sread + 1 == R ? 0 : sread + 1;
        // convert; the two lanes of a voxel exchange halves, so that each has twice 8 consecutive channels
        uint2 pk[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = is_relu(EPI) ? relu_f32(acc[4 * q + e]) : acc[4 * q + e];
            pk[q] = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
        }
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const auto x = __builtin_amdgcn_permlane32_swap(pk[2 * p].x, pk[2 * p + 1].x, false, false);
            const auto y = __builtin_amdgcn_permlane32_swap(pk[2 * p].y, pk[2 * p + 1].y, false, false);
            uint4 v = make_uint4(x[0], y[0], x[1], y[1]);
            if (MASK) {
                v.x &= positive_halves(mv[p].x);
                v.y &= positive_halves(mv[p].y);
                v.z &= positive_halves(mv[p].z);
                v.w &= positive_halves(mv[p].w);
            }
            *reinterpret_cast<uint4 *>(turn + lds_off(col, 2 * p + hi)) = v;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(turn + j * 1024 + lane * 16);
            if (ok[j]) __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(out + vo[j]));
        }
        out += orow;
        // behind the last reads of the slot that the next loads fill (the stores wait for them: lgkmcnt(0) makes it formal)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        fetch();
        fetch_mask();
        __builtin_amdgcn_sched_barrier(0);
    };

    // Loads in the order of the steps -(R - 2) ... -1: input row i + R + 2 and mask row i + R - 1 together.
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
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // slots 0 and 1 are free
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = R; r < R + 2; ++r) { fetch(); fetch_mask(); }
    __builtin_amdgcn_sched_barrier(0);
    // (the first step stands before the loop: the compiler's waits for the weights, which know nothing of the rows on their
    // way and so wait for those too, are in it)
    step(std::integral_constant<int, 0>{});
    for (int left = n - 1; left > 0;) {
        step(std::integral_constant<int, 1>{});
        if (--left == 0) break;
        step(std::integral_constant<int, 2>{});
        if (--left == 0) break;
        step(std::integral_constant<int, 0>{});
        --left;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the repeated rows
}

}  // namespace

// Chunks of rows: a march costs its rows, the two of the surround and about six rows' time before its first product, and 2048
// waves fit on the chip at once.  Where the tensors do not fit the 256 MB of memory-side cache, half as many waves on marches
// twice as long touch memory in fewer places and are faster, as eight waves of a compute unit are no longer what its memory
// share is waiting for (16 x 512^2 in 1 x 2 x 2 tiles, 64 -> 128 rows: 32 -> 32 122 -> 113 us, 32 -> 64 241 (128 rows) -> 201 (256);
// but 32 -> 64 on 16 x 256^2, 201 MB, 64 -> 32 rows 49 -> 43).
// Measured with the packing of the weights, patch march -> this: 32 -> 32 on 16 x 512^2 in 1 x 2 x 2 tiles forward 158 -> 104 us (5.2
// TB/s), masked data gradient 191 -> 160 (5.0), 32 -> 64 397 -> 258; 32 -> 64 on 16 x 256^2 69 -> 43, 32 -> 32 on 2 x 512^2 36 -> 15, on 11
// x 390 x 410 70 -> 42, on 480^2 29 -> 10, on 7 x 64^2 8.1 -> 5.9.  Copies of such tensors reach 6.4 TB/s; stores of 32 bytes a voxel
// instead of whole records cost 5 to 20 %.
int launch_conv_rows2d(const void *Pin, const void *wpack, const float *bias, void *Pout, const Geo &g, int ko, bool relu,
                       hipStream_t s, const void *mask, const ConvSplit *split) {
    RowArgs a;
    a.in = static_cast<const uint16_t *>(Pin);
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
    const long long vox = 1LL * g.ntiles * g.td * eh * ew, fit = vox * 2 * (C + ko * (mask ? 2 : 1)) > (256LL << 20) ? 1024 : 2048;
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
    static const Kern kern[2][3] = {{conv_rows2d_kernel<kNone, false>, conv_rows2d_kernel<kRelu, false>, conv_rows2d_kernel<kMask, false>},
                                    {conv_rows2d_kernel<kNone, true>, conv_rows2d_kernel<kRelu, true>, conv_rows2d_kernel<kMask, false>}};
    // more than 64 KB of dynamic LDS has to be requested explicitly
    static const hipError_t attr = [] {
        for (int i = 0; i < 6; ++i) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern[i / 3][i % 3]),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kWaves * wave_lds(i % 3 == kMask));
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (attr != hipSuccess) return record_hip(attr);
    hipLaunchKernelGGL(kern[bias ? 1 : 0][epi], dim3(grid), dim3(kThreads), kWaves * wave_lds(epi == kMask), s, a);
    return record_hip(hipGetLastError());
}

}  // namespace sp3d
