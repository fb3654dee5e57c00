// bf16 implicit-GEMM 3x3x3 convolution on padded tiles for channel counts that are multiples of 32,
// on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulation).  Serves conv3d_fwd and,
// with mirrored taps and swapped channel roles, conv3d_dgrad.
//
// The kernel proper contracts ONE 32-channel input chunk into one 32-channel output block.  Wider
// layers run it once per input chunk (one launch each, every output block in the same launch): the
// first chunk writes fp32 partial sums to the workspace, later chunks add to them, the last one adds,
// applies ReLU and stores bf16.  The order of the additions is fixed, so results are reproducible.
//
// Work decomposition.  A workgroup (4 waves, one per SIMD) owns an output patch of 8 rows (H) x 32
// columns (W) of one tile and marches along D.  Each input plane (10 x 34 voxels x 32 channels) is
// staged once in LDS by direct global->LDS loads, three planes ahead of the plane being consumed
// (ring of four).  A wave owns 2 of the 8 rows and keeps the accumulators of consecutive output
// planes in registers: input plane D feeds output planes D, D-1, D-2 through taps kd = 0, 1, 2, so an
// input fragment read from LDS once is used by up to 3 (kd) x 2 (kh) MFMAs.  A fourth accumulator
// slot holds the plane finished in the previous step, whose conversion and stores are spread over
// the MFMA stream of the current step.  All 27 x 2 weight fragments (32 x 16 each) live in
// registers for the whole march.
//
// 2-D variant (template parameter KD = 1; geometry flag `flat`): the kernel has extent 1 along D, so a staged
// plane feeds only its own output plane (tap kd = 1 of the scheme above; the MFMAs of kd = 0, 2 and their
// weight fragments are left out).  The march, the ring and the epilogue timing are unchanged.
//
// MFMA operand roles: A = weights [M = Cout][K = 16 input channels], B = voxels [K][N = 32 voxels
// along W], D[M = Cout][N = voxel].  Lane l of B supplies voxel l%32, channels 8*(l/32)..+7 of the
// 16-channel half; lane l of D holds voxel l%32, channels 8*(i/4) + 4*(l/32) + i%4 for i = 0..15.
#include "pack_weights.h"

namespace sp3d {

using namespace convk;

namespace {

__global__ __launch_bounds__(64 * kPackWaves) void pack_weights_kernel(PackArgs a) {
    __shared__ __align__(16) PackSquares square;
    pack_weights(a, blockIdx.x, square);
}

// Per-wave state of the march that the side work of a step needs.
template <bool HAS_BIAS>
struct Ctx {
    const uint16_t *tin0;       // first padded input plane of this workgroup's D chunk (at the chunk's channels)
    size_t plane_elems;         // input elements per padded plane of the tile
    int nplanes;                // input planes of the chunk (output planes + 2)
    int plo, phi;               // staged planes are clamped to [plo, phi] (slices side by side: the outer two are not real)
    ptrdiff_t dlo, dhi;         // gathered halos: what to add for staged plane 0 / the last one (else 0)
    int goff[LOADS];            // per-lane source offsets of the staging loads (elements)
    char *lds_stage;            // where this wave's first load goes (ring slot 0)
    int last;                   // ... and its last one, further on: waves that have one less repeat the one before
    uint16_t *obase;            // output address of (plane 0, first row of the wave, this lane)
    const uint16_t *mbase;      // same position in the mask tensor
    uint16_t *bbase;            // this lane's word of that voxel in the one-bit mask (see relu_bit)
    float *pbase;               // this lane's slot in the wave's region of the fp32 partial-sum buffer
    size_t oplane, orow;        // output elements per padded plane / per padded row
    size_t mrow;                // from the row that the mask of the wave's first row is read from to that of the second
    Ragged rag;                 // 3-D, ragged patches
    RaggedPart rpart;
    bool okrow[RH];             // row/column of this lane lies inside the tile interior
    float bv[HAS_BIAS ? 16 : 1];
};

// Staging load j of padded plane `dplane` of the chunk -> ring slot dplane % NBUF.  global_load_lds:
// lane l supplies its own global address and the 16 bytes land at LDS base + 16*l.  Planes past the last
// one needed are clamped (their ring slot is never read), so every step issues exactly LOADS loads.
template <bool HAS_BIAS>
__device__ __forceinline__ void stage(const Ctx<HAS_BIAS> &c, int dplane, int j) {
    const int dpl = min(max(dplane, c.plo), c.phi);
    const uint16_t *p = c.tin0 + static_cast<ptrdiff_t>(dpl) * static_cast<ptrdiff_t>(c.plane_elems) +
                        (dpl == 0 ? c.dlo : 0) + (dpl == c.nplanes - 1 ? c.dhi : 0);
    char *dst = c.lds_stage + (dplane % NBUF) * PLANE_BYTES + (j == LOADS - 1 ? c.last : j * kWaves * 1024);
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(p + c.goff[j]),
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// Partial sums of 4 channels of row h of plane d written by the previous input chunk.
template <Edge EDGE, bool HAS_BIAS>
__device__ __forceinline__ pin_t load_partial(const Ctx<HAS_BIAS> &c, int d, int h, int q) {
    pin_t v = pin_t{0.f, 0.f, 0.f, 0.f};
    if (EDGE != kBranches || c.okrow[h]) v = *reinterpret_cast<const pin_t *>(c.pbase + part_from<EDGE>(c, d, h, q));
    return v;
}

// The 4 mask values that belong to one store unit (fetched at the start of the step, like the partial sums).
template <Edge EDGE, bool BITS, bool HAS_BIAS>
__device__ __forceinline__ mask_t load_mask(const Ctx<HAS_BIAS> &c, int d, int h, int q) {
    mask_t v = mask_t{0u, 0u};
    if (BITS) {         // the row's word, kept in unit 0
        if (q == 0 && (EDGE != kBranches || c.okrow[h])) v.x = c.bbase[mask_off<EDGE>(c, d, h) >> 4];
        return v;
    }
    if (EDGE != kBranches || c.okrow[h]) v = *reinterpret_cast<const mask_t *>(c.mbase + mask_off<EDGE>(c, d, h) + 8 * q);
    return v;
}

// Finish 4 channels of row h of a finished plane (channels 8q + 4*(lane/32) .. +3 of this output block):
// add the earlier chunks' partial sums if there are any, then either store the new partial (fp32) or
// apply ReLU, convert and store bf16 (8 bytes).
template <int MODE, int RELU, Edge EDGE, bool HAS_BIAS>
__device__ __forceinline__ void store_unit(const Ctx<HAS_BIAS> &c, int d, const f32x16 (&s)[RH],
                                           const pin_t (&pin)[RH][4], mask_t (&mk)[RH][4], int h, int q) {
    float v0 = s[h][4 * q], v1 = s[h][4 * q + 1], v2 = s[h][4 * q + 2], v3 = s[h][4 * q + 3];
    if (MODE == kMiddle || MODE == kLast) {
        v0 += pin[h][q].x; v1 += pin[h][q].y; v2 += pin[h][q].z; v3 += pin[h][q].w;
    }
    const size_t at = d * c.oplane + h * c.orow + 8 * q;
    if (MODE == kFirst || MODE == kMiddle) {
        if (EDGE == kDrops) drop_store<0>(c.rpart, d, h, q, pin_t{v0, v1, v2, v3});
        else if (EDGE == kInside || c.okrow[h]) *reinterpret_cast<float4 *>(c.pbase + part_unit(d, h, q)) = make_float4(v0, v1, v2, v3);
        return;
    }
    if (is_relu(RELU)) {
        v0 = relu_f32(v0); v1 = relu_f32(v1); v2 = relu_f32(v2); v3 = relu_f32(v3);
    }
    uint2 pk = make_uint2(pack2(v0, v1), pack2(v2, v3));
    if (RELU == kMask) {
        pk.x &= positive_halves(mk[h][q].x);
        pk.y &= positive_halves(mk[h][q].y);
    }
    if (RELU == kMaskBits) {
        if (q == 0) mk[h][0].x = spread_word(mk[h][0].x);
        const uint2 m = nibble_halves(mk[h][0].x, q);
        pk.x &= m.x;
        pk.y &= m.y;
    }
    if (EDGE == kDrops) drop_store(c.rag.out + d * c.oplane, c.rag.vo[h] + 16 * q, pk);
    else if (EDGE == kInside || c.okrow[h]) *reinterpret_cast<uint2 *>(c.obase + at) = pk;
    if (RELU == kReluBits) {
        // the row's word collects in the (otherwise unused) mask register of unit 0 and leaves with the last unit
        uint32_t n = mk[h][0].x;
        n = shift_in_positive(n, v0); n = shift_in_positive(n, v1);
        n = shift_in_positive(n, v2); n = shift_in_positive(n, v3);
        mk[h][0].x = n;
        if (q == 3) store_bits<EDGE>(c, d, mk, h);
    }
}

// All MFMAs of one staged input plane Dp, with the step's side work spread over the six MFMA groups:
// the staging loads of plane Dp+DIST and (EPI) the conversion and stores of output plane Dp-3, which
// received its last contribution in step Dp-1, after which its accumulator slot returns to the bias.
// lcol[kw]: this lane's read base in ring slot 0: first row of the wave, column lane % 32 + kw, piece lane / 32 (the second K
// half's piece is 32 bytes away, up or down).  Fragments are fetched one (kw, K-half) group of RH+2 rows ahead of the MFMAs that
// consume them.  P = Dp mod 4: output plane Dp-kd lives in slot (P-kd) mod 4, plane Dp-3 in slot (P+1) mod 4.
// EDGE: a patch that lies completely inside the tile interior needs no mask for its stores (no branches in
// the step, which lets the scheduler weave the side work between the MFMAs; in 3-D others have none either, see Ragged).
// SIDE (see side_load): kSideNone - the step loads its own partial sums / mask values (pin, mk) the ordinary
// way; otherwise it uses the ones the previous step fetched (kSideUse) and first of all fetches those of the
// plane that the next step finishes, Dp - 2, into the other set (npin, nmk), which the caller passes through
// the wait that ends the step.
template <int P, bool EPI, int MODE, int RELU, Edge EDGE, int KD, int SIDE, int NV, bool HAS_BIAS>
__device__ __forceinline__ void plane_step(const Ctx<HAS_BIAS> &c, int Dp, const uint32_t (&lcol)[3],
                                           const bf16x8 (&wf)[NFRAG], f32x16 (&acc)[4][RH],
                                           pin_t (&pin)[RH][4], mask_t (&mk)[RH][4],
                                           pin_t (&npin)[RH][4], mask_t (&nmk)[RH][4], bf16x8 (&b0)[RH + 2]) {
    constexpr int NR = RH + 2;
    constexpr int DONE = (P + 1) & 3;
    using S = Side<MODE, RELU, KD, false>;
    // ring slots of plane Dp and of plane Dp + 1: two of them are within reach of the instruction's 16-bit offset field
    constexpr int PN = (P + 1) & 3;
    constexpr int HIGH = (P >> 1) * 2 * PLANE_BYTES, HIGHN = (PN >> 1) * 2 * PLANE_BYTES;
    constexpr int OFF = (P & 1) * PLANE_BYTES, OFFN = (PN & 1) * PLANE_BYTES;
    static_assert(PLANE_BYTES + (RH + 1) * ROW_BYTES < 65536, "offset field");
    bf16x8 b[2][NR];
    if (SIDE != kSideNone) {
#pragma unroll
        for (int h = 0; h < RH; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const size_t at = mask_off<EDGE>(c, Dp - 2, h);
                if (S::PINS) side_load(npin[h][q], c.pbase + part_from<EDGE>(c, Dp - 2, h, q));
                if (S::MASK && !S::BITS) side_load(nmk[h][q], c.mbase + at + 8 * q);
                if (S::BITS && q == 0) SP3D_SIDE_LOAD_BITS(nmk[h][0].x, c.bbase + (at >> 4));
            }
    }
    if (SIDE == kSideNone && EPI && S::PINS) {
#pragma unroll
        for (int h = 0; h < RH; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) pin[h][q] = load_partial<EDGE>(c, Dp - 3, h, q);
    }
    if (SIDE == kSideNone && EPI && S::MASK) {
#pragma unroll
        for (int h = 0; h < RH; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) mk[h][q] = load_mask<EDGE, S::BITS>(c, Dp - 3, h, q);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) b[0][r] = b0[r];       // group 0's fragments: read, and waited for, by the previous step
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
        const int kw = gi >> 1, half = gi & 1;
        if (gi + 1 < NG) {
            const int kw2 = (gi + 1) >> 1, half2 = (gi + 1) & 1;
            const uint32_t at = (lcol[kw2] ^ (half2 * 32)) + HIGH;
#pragma unroll
            for (int r = 0; r < NR; ++r) frag_read(b[(gi + 1) & 1][r], at, OFF + r * ROW_BYTES);
        } else {
            // The step's one synchronisation sits here, before its last group, not at its end: plane Dp + 1
            // must be complete (every wave's staging loads of it, issued two steps ago: loads complete in issue
            // order and the only ones issued after them are those of plane Dp + 2 and the NG - 1 of this step,
            // so "at most NV outstanding" implies it; stores share the counter and only make the wait more
            // conservative), and every wave must have finished reading plane Dp, this step's own (its last
            // fragment reads were issued a group ago; lgkmcnt(0) makes that formal), whose ring slot the next
            // step's staging loads overwrite.  Behind the barrier the first group of the NEXT step is read
            // already, while this step's last 18 MFMAs run: the step boundary itself has no wait, no barrier and
            // no exposed LDS latency.  (With the synchronisation at the end of the step the matrix cores idled
            // there for the barrier, the reads of two groups and their latency.)
            side_fence<NV, true, SIDE != kSideNone && S::PINS, SIDE != kSideNone && S::MASK,
                       SIDE != kSideNone && S::BITS>(npin, nmk);
            __builtin_amdgcn_s_barrier();
#pragma unroll
            for (int r = 0; r < NR; ++r) frag_read(b[0][r], lcol[0] + HIGHN, OFFN + r * ROW_BYTES);
        }
        // this group's fragments were read a group ago; the NR reads issued just now may stay in flight
        frag_wait<NR>(b[gi & 1]);
        // keep the reads of the next group ahead of this group's MFMAs (the scheduler would
        // otherwise sink every read to just before its first use and expose the LDS latency)
        __builtin_amdgcn_sched_barrier(0);
        stage(c, Dp + DIST, gi);
        if (gi < 4) {
            if (EPI) {
                // (the copies of the finished plane's sums out of the accumulation registers have no operand that
                // is computed in the step, so the compiler emits all 32 at the top of the step, in front of its
                // first MFMA; passing the plane through an empty statement here makes each group's eight depend
                // on a point inside the group, where they are woven between the MFMAs like the rest)
                asm volatile("" : "+a"(acc[DONE][0]), "+a"(acc[DONE][1]));
                store_unit<MODE, RELU, EDGE>(c, Dp - 3, acc[DONE], pin, mk, 0, gi);
                store_unit<MODE, RELU, EDGE>(c, Dp - 3, acc[DONE], pin, mk, 1, gi);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[DONE][gi - 4][i] = HAS_BIAS ? c.bv[HAS_BIAS ? i : 0] : 0.f;
        }
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int kh = 0; kh < 3; ++kh) {
                const int h = r - kh;
                if (h < 0 || h >= RH) continue;
#pragma unroll
                for (int kd = 0; kd < 3; ++kd) {
                    if (KD == 1 && kd != 1) continue;
                    const int slot = (P - kd + 4) & 3;
                    acc[slot][h] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        wf[((kd * 3 + kh) * 3 + kw) * 2 + half], b[gi & 1][r], acc[slot][h], 0, 0, 0);
                }
            }
        // weave: after each MFMA let a few of the side-work instructions issue while it executes
#pragma unroll
        for (int i = 0; i < KD * (RH + 1) * 2; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
            __builtin_amdgcn_sched_group_barrier(0x006, 3, 0);   // up to three VALU / SALU
            if (i % 6 == 2) __builtin_amdgcn_sched_group_barrier(0x060, 1, 0);   // a vector memory op
        }
    }
    // the next step's first fragments, read 18 MFMAs ago: complete before they leave the step (beyond it the
    // compiler may copy the registers at a block boundary, which it must not do while data is on its way)
    frag_wait<0>(b[0]);
#pragma unroll
    for (int r = 0; r < NR; ++r) b0[r] = b[0][r];
}

template <int MODE, bool HAS_BIAS, int RELU, int PATCHES>
__global__ __launch_bounds__(kThreads, 1) void conv_mfma_kernel(ConvArgs a) {
    constexpr int KD = kd_of(PATCHES);
    extern __shared__ __attribute__((aligned(128))) char lds[];  // NBUF planes of PLANE_BYTES
    const Geo &g = a.g;
    // Consecutive hardware workgroup ids rotate over the 8 XCDs; give each XCD a contiguous range of
    // logical ids so that patches sharing halo rows/columns meet in the same L2.
    const int per_xcd = gridDim.x >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= a.nblocks) return;
    int t = logical;
    const int cj = t % a.nco; t /= a.nco;          // output block: fastest, so that the workgroups that
                                                    // share an input patch run together
    const int pw_i = t % a.nw; t /= a.nw;
    const int ph_i = t % a.nh; t /= a.nh;
    const int pd_i = t % a.nd; t /= a.nd;
    const int tile = t;
    const int d0 = pd_i * a.dchunk, h0 = ph_i * PH, w0 = pw_i * PW;      // coordinates inside the output box
    const TileBox bx = tile_box(g, tile);
    int dn = min(a.dchunk, bx.bd - d0);                                 // output planes (slices) to produce
    // the patches are laid out for the largest box of the grid; a tile at the volume border has a smaller one
    if (dn <= 0 || h0 >= bx.bh || w0 >= bx.bw) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hi = lane >> 5;

    // weight fragments: 54 x 16 bytes per lane, resident for the whole march
    bf16x8 wf[NFRAG];
#pragma unroll
    for (int f = 0; f < NFRAG; ++f) {
        if (KD == 1 && f / 18 != 1) continue;        // 2-D variant: only the taps with kd = 1 exist
        const uint4 q = a.wpack[(cj * NFRAG + f) * 64 + lane];
        wf[f] = *reinterpret_cast<const bf16x8 *>(&q);
        if (KD == 3 && SP3D_PARKED(f)) park(wf[f]);
    }

    Ctx<HAS_BIAS> c;
    const int F = KD == 1 ? a.fold : 1;         // slices side by side (see fold_col); dn is a multiple of F
    const size_t plane_real = static_cast<size_t>(g.ph) * g.pw * a.in_cs;
    c.plane_elems = plane_real * F;
    c.tin0 = a.in + (static_cast<size_t>(tile) * g.tile_vox + bx.org) * a.in_cs + d0 * plane_real + a.in_co -
             static_cast<ptrdiff_t>(F - 1) * static_cast<ptrdiff_t>(plane_real);
    dn /= F;                                    // from here on: output steps
    c.nplanes = dn + 2;
    c.plo = F > 1 ? 1 : 0;
    c.phi = F > 1 ? c.nplanes - 2 : c.nplanes - 1;
    // Load j of wave w covers patch-local voxels 16 (w + 4 j) .. + 15, four lanes to a voxel, each the piece whose place is its
    // own (see piece_at).  Voxels beyond the box and its one-voxel surround (ragged patches) are clamped to a valid
    // address; they only feed outputs that are never stored.  Places past the last voxel take that voxel again.
    const bool less = wave + kWaves * (LOADS - 1) >= PLANE_LOADS;
    c.last = (LOADS - 1 - (less ? 1 : 0)) * kWaves * 1024;
    const auto staged_voxel = [&](int j) {
        return min(16 * (wave + kWaves * (j == LOADS - 1 && less ? j - 1 : j)) + (lane >> 2), PLANE_VOX - 1);
    };
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
        const int v = staged_voxel(j);
        const FoldCol fc = fold_col(v % LCOLS, F, a.fold_w);
        const int row = min(h0 + v / LCOLS, bx.bh + 1), colv = min(w0 + fc.c, bx.bw + 1);
        c.goff[j] = ((min(fc.s, F - 1) * g.ph + row) * g.pw + colv) * a.in_cs + 8 * piece_at(v % LCOLS, lane & 3);
    }
    c.dlo = c.dhi = 0;
    if (a.gather) {          // (host: one-voxel margins, no grown box, 3-D)
        const GatherShift gs = gather_shift(g, tile, a.in_cs);
#pragma unroll
        for (int j = 0; j < LOADS; ++j) {
            const int v = staged_voxel(j);
            const int row = min(h0 + v / LCOLS, bx.bh + 1), colv = min(w0 + v % LCOLS, bx.bw + 1);
            c.goff[j] += (row == 0 ? gs.hm : 0) + (row == g.th + 1 ? gs.hp : 0) + (colv == 0 ? gs.wm : 0) +
                         (colv == g.tw + 1 ? gs.wp : 0);
        }
        if (d0 == 0) c.dlo = gs.dm;
        if (d0 + dn == g.td) c.dhi = gs.dp;
    }
    c.lds_stage = lds + wave * 1024;
    const OutDst od = out_dest(a, cj);
    const FoldCol oc = fold_col(col, F, a.fold_w);
    c.orow = static_cast<size_t>(g.pw) * od.cs;
    c.oplane = static_cast<size_t>(g.ph) * c.orow * F;
    const size_t ovox = static_cast<size_t>(tile) * g.tile_vox + bx.org +
                        (static_cast<size_t>(d0 + 1 + min(oc.s, F - 1)) * g.ph + h0 + wave * RH + 1) * g.pw + w0 +
                        oc.c + 1;
    const size_t opos = ovox * od.cs + od.co + 4 * hi;
    c.obase = od.base + opos;
    c.mbase = a.mask + opos;
    c.bbase = a.bits + (ovox * a.nco + cj) * 2 + hi;
    c.mrow = c.orow;
    if (PATCHES == kRagged3) {
        const size_t voxel0 = static_cast<size_t>(tile) * g.tile_vox + bx.org +
                              (static_cast<size_t>(d0 + 1) * g.ph + h0 + wave * RH + 1) * g.pw + w0 + 1;
        c.rag = ragged(g, bx, h0, w0, wave * RH, col, hi, voxel0, od.base, od.cs, od.co, a.bits, a.nco, cj);
        // the mask's row and column nearest to the lane's inside the box
        const int up = max(h0 + wave * RH - (bx.bh - 1), 0), left = max(w0 + col - (bx.bw - 1), 0);
        c.mbase -= up * c.orow + static_cast<size_t>(left) * od.cs;
        if (RELU == kMaskBits) c.bbase -= (up * c.orow + static_cast<size_t>(left) * od.cs) >> 4;
        if (h0 + wave * RH + 1 >= bx.bh) c.mrow = 0;
    }
    // wave `wave` of workgroup `logical`: a region of dchunk planes x RH rows x 4 units x 1 KB
    float *const region = a.part + (static_cast<size_t>(logical) * kWaves + wave) * a.dchunk * (RH * 4 * 256);
    c.pbase = region + lane * 4;
    if (PATCHES == kRagged3 && MODE != kSingle) {
        c.rpart = ragged_part(bx, h0, w0, wave * RH, col, lane, region);
        if (c.rpart.off[0] == kDrop) c.pbase = region;
    }
#pragma unroll
    for (int h = 0; h < RH; ++h) c.okrow[h] = h0 + wave * RH + h < bx.bh && w0 + oc.c < bx.bw && oc.s < F;
    // the bias is folded into the accumulators: a slot starts from the bias instead of zero
    // (without a bias the slots start from the constant zero and no registers are spent on it)
    if (HAS_BIAS) {
#pragma unroll
        for (int i = 0; i < 16; ++i) c.bv[HAS_BIAS ? i : 0] = a.bias[C * cj + 8 * (i >> 2) + 4 * hi + (i & 3)];
    }
    f32x16 acc[4][RH];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int h = 0; h < RH; ++h)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[s][h][i] = HAS_BIAS ? c.bv[HAS_BIAS ? i : 0] : 0.f;

    const char *lbase = lds + wave * RH * ROW_BYTES;
    const int nplanes = c.nplanes;

    // Prologue: planes 0 .. DIST-1 in flight; plane 0 must have landed before the first MFMA.
#pragma unroll
    for (int i = 0; i < DIST; ++i)
#pragma unroll
        for (int j = 0; j < LOADS; ++j) stage(c, i, j);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    // (the synchronisation of a step sits inside it, before its last MFMA group: see plane_step)
    constexpr int NV_STEP = (DIST - 1) * LOADS - 1;     // plane Dp + 2's loads and the step's first NG - 1
    static_assert(NG == LOADS, "one staging load per MFMA group");
    const uint32_t lcol[3] = {lds_addr(lbase + lds_off(col, hi)), lds_addr(lbase + lds_off(col + 1, hi)),
                        lds_addr(lbase + lds_off(col + 2, hi))};
    bf16x8 b0[RH + 2];
#pragma unroll
    for (int r = 0; r < RH + 2; ++r) b0[r] = *reinterpret_cast<const bf16x8 *>(lbase + lds_off(col, hi) + r * ROW_BYTES);

    auto march = [&](auto edge_tag) {
        constexpr Edge EDGE = decltype(edge_tag)::value;
        using S = Side<MODE, RELU, KD, false>;
        // whole patches, and in 3-D all, fetch their partial sums / mask values one step ahead (see side_load): steps with an even
        // plane index use set A and fetch into set B, odd ones the other way round
        constexpr bool ASYNC = EDGE != kBranches && S::ASYNC;
        constexpr int FETCH = ASYNC ? kSideFetch : kSideNone, USE = ASYNC ? kSideUse : kSideNone;
        pin_t pinA[RH][4], pinB[RH][4];
        mask_t mkA[RH][4], mkB[RH][4];
        // (by its synchronisation point a step with stores has issued LOADS - 1 + 8 >= NV_STEP operations after its
        // side loads, so the wait covers them; the fetch-only step has issued just LOADS - 1 staging loads after
        // them and waits accordingly)
        static_assert(LOADS - 1 + 8 >= NV_STEP, "side loads must be older than what the step's wait lets stay in flight");
        // the first three steps have no finished plane to store (nplanes >= 3 always); the third one fetches
        // what the first store needs
        plane_step<0, false, MODE, RELU, EDGE, KD, kSideNone, NV_STEP>(c, 0, lcol, wf, acc, pinA, mkA, pinB, mkB, b0);
        plane_step<1, false, MODE, RELU, EDGE, KD, kSideNone, NV_STEP>(c, 1, lcol, wf, acc, pinA, mkA, pinB, mkB, b0);
        plane_step<2, false, MODE, RELU, EDGE, KD, FETCH, (ASYNC ? LOADS - 1 : NV_STEP)>(c, 2, lcol, wf, acc, pinA,
                                                                                        mkA, pinB, mkB, b0);
        // steps 3, 4, 5, 6, 7, ...: planes mod 4 = 3, 0, 1, 2, 3, ...
#define SP3D_MAIN_STEP(OFF, PHASE, CP, CM, NP, NM)                                                            \
    if (D + (OFF) < nplanes)                                                                                  \
        plane_step<PHASE, true, MODE, RELU, EDGE, KD, USE, NV_STEP>(c, D + (OFF), lcol, wf, acc, CP, CM, NP, NM, b0);
        for (int D = 3; D < nplanes; D += 4) {
            SP3D_MAIN_STEP(0, 3, pinB, mkB, pinA, mkA)
            SP3D_MAIN_STEP(1, 0, pinA, mkA, pinB, mkB)
            SP3D_MAIN_STEP(2, 1, pinB, mkB, pinA, mkA)
            SP3D_MAIN_STEP(3, 2, pinA, mkA, pinB, mkB)
        }
#undef SP3D_MAIN_STEP
        // the last output plane (dn-1) finished in the last step; it sits in slot (dn-1) mod 4, and with side
        // loads the last step (plane index dn + 1, of the parity of dn - 1) fetched its values: into set B if
        // that index is even
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (!ASYNC && S::PINS) {
#pragma unroll
            for (int h = 0; h < RH; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q) pinA[h][q] = pinB[h][q] = load_partial<EDGE>(c, dn - 1, h, q);
        }
        if (!ASYNC && S::MASK) {
#pragma unroll
            for (int h = 0; h < RH; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q) mkA[h][q] = mkB[h][q] = load_mask<EDGE, S::BITS>(c, dn - 1, h, q);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (s == ((dn - 1) & 3)) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    store_unit<MODE, RELU, EDGE>(c, dn - 1, acc[s], (s & 1) ? pinA : pinB, (s & 1) ? mkA : mkB, 0, q);
                    store_unit<MODE, RELU, EDGE>(c, dn - 1, acc[s], (s & 1) ? pinA : pinB, (s & 1) ? mkA : mkB, 1, q);
                }
            }
    };
    if constexpr (PATCHES == kWhole3) march(std::integral_constant<Edge, kInside>{});
    else if constexpr (PATCHES == kRagged3) march(std::integral_constant<Edge, kDrops>{});
    else if constexpr (MODE == kSingle) march(std::integral_constant<Edge, kBranches>{});       // slices side by side: 15 columns at most
    else if (h0 + PH <= bx.bh && w0 + PW <= bx.bw) march(std::integral_constant<Edge, kInside>{});
    else march(std::integral_constant<Edge, kBranches>{});
}

}  // namespace


bool conv_mfma_supported(const Geo &g, int ki, int ko, sp_dtype_t dt) {
    // per-lane staging offsets inside a padded plane are 32-bit: element offsets in the one-chunk kernel, byte
    // offsets in the two-chunk kernel (input channels in multiples of 64)
    const long long lim = ki % (2 * C) == 0 ? 0x3fffffffLL : 0x7fffffffLL;
    return dt == SP_BF16 && ki % C == 0 && ko % C == 0 && ki <= 1024 && ko <= 1024 &&
           1LL * g.ph * g.pw * (ki > ko ? ki : ko) < lim;
}

static size_t pack_bytes(int ki, int ko) {
    return static_cast<size_t>(ki / C) * (ko / C) * NFRAG * 64 * 16;
}

// How a layer is cut into workgroups (the same for every launch of the layer).
struct PatchPlan { int nh, nw, dchunk, nd; long long nblocks; bool pairs; int fold, fold_w; };      // dchunk: a multiple of fold
static PatchPlan plan_patches(const Geo &g, int ki, int ko) {
    PatchPlan p;
    const int nco = ko / C;
    // input channels in multiples of 64: two chunks per launch, summed on chip (4-row patches)
    p.pairs = ki % (2 * C) == 0;
    const int ph = p.pairs ? wide::PH : PH;
    // patches cover the largest output box of the grid (the interior grown on both sides)
    const int ed = g.td + 2 * grow_d(g), eh = g.th + 2 * g.grow, ew = g.tw + 2 * g.grow;
    p.nh = (eh + ph - 1) / ph;
    p.nw = (ew + PW - 1) / PW;
    const long long base = 1LL * g.ntiles * p.nh * p.nw * nco;
    // 2-D variant, tiles narrower than half a patch: up to 4 slices side by side (see fold_col); the tile's
    // slice count and the D chunk must be multiples of it
    p.fold = 1;
    p.fold_w = ew + 2;
    if (g.flat && 2 * (ew + 2) <= LCOLS) {
        int f = LCOLS / (ew + 2);
        if (f > 4) f = 4;
        while (f > 1 && g.td % f) --f;
        p.fold = f;
    }
    // D chunk: the whole depth, halved until there are 1024 workgroups but never below 16 planes; or, where that is estimated to
    // save at least 5 %, what costs least if the 256 compute units (one workgroup each: LDS) take the workgroups in rounds, a
    // round lasting as long as its march - the chunk's planes, the two of the surround (and two that drain the hand-over
    // between the two chunks of a pair), and what a march costs before its first plane, in steps: the weights and three
    // planes on their way, about 6 us = 4 plane steps in 3-D and 16 of the shorter ones in 2-D (2 ... 8 and 4 ... 16
    // measured within 1 %).  (The first rule alone gives 8 workgroups to a layer on 32^3: 256 -> 256 there (128 workgroups of 16
    // planes -> 256 of 8) 48 -> 35 us a launch, 32 -> 32 on 128^3 (512 of 16 -> 256 of 32) 117 -> 104 us.  Taken on any saving, the
    // second cost time where it only merged chunks: 64 -> 256 on 38 x 34 x 47, 2 x 2 x 1 tiles, 99 -> 107 us, 192 -> 64 on 64 x 147
    // x 116 839 -> 896; less than a workgroup per compute unit takes a tenth more than its round: 512 -> 96 on 40 x 76 x 66 as 171
    // workgroups 906 us, as 684 825.)
    const int steps = (ed + p.fold - 1) / p.fold, over = (g.flat ? 16 : 4) + (p.pairs ? 4 : 2);
    const auto cost = [&](int d) {
        const long long n = base * ((steps + d - 1) / d);
        return static_cast<double>((n + 255) / 256 * (d + over)) * (n < 256 ? 1.1 : 1.0);
    };
    int d0 = ed;
    while (base * ((ed + d0 - 1) / d0) < 1024 && d0 > 16) d0 = (d0 + 1) / 2;
    int best = (d0 + p.fold - 1) / p.fold;
    double least = 0.95 * cost(best);
    for (int k = 1; k == 1 || (k <= steps && base * k <= 2048); ++k) {
        const int d = (steps + k - 1) / k;
        if (cost(d) < least) { least = cost(d); best = d; }
    }
    const int dchunk = best * p.fold;
    p.dchunk = dchunk;
    p.nd = (ed + dchunk - 1) / dchunk;
    p.nblocks = base * p.nd;
    return p;
}

// Which family serves a layer: the marching kernels of this file, or the implicit GEMM of conv_gemm.hip.  The marching
// kernels reuse a staged plane for 27 (9) taps and win where the volume fills the chip with long marches; they lose where
// a launch per pair of input chunks carries little work (few voxels, many channels), where stacks of slices are thin and
// where patches are mostly empty.  Both times are estimated from what bounds them, marching: launches x (rounds of the
// 256 compute units x (start + planes) + launch) + the partial sums between launches.  The constants are fitted to 472
// layers measured with both families on their own tile grids (32 ... 1024 channels, 3-D from 64 voxels to 4 million, W split
// in one to four, 2-D to 700 000, on up to 1 x 4 x 4 tiles; 8 % and 11 % rms).  The estimate is that of the whole volume as
// one tile, so that a layer takes the same family, and sums in the same order, on every tile grid and with every output box
// growth; a grid that cuts W into pieces of less than a patch makes the march slower than that.  Over the 472 layers the
// choice costs 3.4 % over the better family of each on its grid (with the estimate of the grid itself it would be 0.4 %; most
// of it on tiles of less than 24 columns), but against marching always none loses more than 4 %.  2-D layers of one launch
// have constants of their own, from 354 such layers (14 % and 6 % rms), and the GEMM has to be ahead by 10 %: 1.2 % over the
// better of each, four more than 4 % behind the march.  Measured, marching -> GEMM: 3-D 256 -> 256 channels on 4^3 53 -> 21 us,
// on 16^3 79 -> 34, on 32^3 146 -> 122, 128 -> 128 on 28 x 44 x 52 96 -> 71; 128 -> 64 on 56 x 88 x 104 279 against 328 (stays),
// 128 -> 128 on 64^3 196 against 279 (stays); 2-D 256 -> 256 on 16 x 64^2 152 -> 107, 128 -> 128 on 2 x 256^2 173 -> 73, 64 -> 64
// there 42 -> 35, 64 -> 256 on 5 x 240 x 177 153 against 170 (stays).
// Figures and constants are of the kernels that they were measured on: since then GEMM workgroups go from one item to the next without
// a gap, and 2-D layers of one launch march by rows (conv_rows2d.hip).  The choice stays where it was, as the family decides in
// which order a layer sums, and with it the last bits of all that follows: 2-D, 128 -> 64 on 16 x 256^2 marches in 280 us where a
// GEMM takes 215, 3-D, 128 -> 128 on 64 x 48 x 24 in 91 against 82, 512 -> 256 on 64^3 in 1570 against 1650; 2-D, 64 -> 64 on 2 x
// 256^2 takes the GEMM in 22.
static bool prefer_gemm(const Geo &g, int ki, int ko) {
    if (!conv_gemm_supported(g, ki, ko)) return false;
    if (conv_gemm_tensor_forms(g, ki, ko)) return true;
    Geo v = g;
    v.ntiles = g.n;
    v.td = g.td * g.gd; v.th = g.th * g.gh; v.tw = g.tw * g.gw;
    v.grow = 0;
    const PatchPlan p = plan_patches(v, ki, ko);
    const int launches = p.pairs ? ki / (2 * C) : ki / C;
    const double rounds = static_cast<double>((p.nblocks + 255) / 256), planes = (p.dchunk + p.fold - 1) / p.fold;
    const double sums = 8.0 * g.ntiles * g.int_vox * ko * (launches - 1);             // bytes written and read
    if (g.flat && launches == 1) return conv_gemm_us(g, ki, ko) < 0.9 * (4 + rounds * (5.6 + (p.pairs ? 1.75 : 1.62) * planes));
    const double us = g.flat ? 2 + launches * (rounds * (6.3 + (p.pairs ? 1.35 : 1.44) * planes) + 0.6) + sums / 7.4e6
                             : 2 + launches * (rounds * (7.2 + (p.pairs ? 2.56 : 2.63) * planes) + 3.6) + sums / 10.3e6;
    return conv_gemm_us(g, ki, ko) < us;
}

int conv_mfma_route(const Geo &g, int ki, int ko, int *detail) {
    if (prefer_gemm(g, ki, ko)) {
        conv_gemm_detail(g, ki, ko, detail);
        return kRouteGemm;
    }
    const PatchPlan p = plan_patches(g, ki, ko);
    detail[0] = p.pairs; detail[1] = p.fold; detail[2] = p.dchunk; detail[3] = p.pairs ? ki / (2 * C) : ki / C;
    return kRouteMarch;
}

// workspace: packed weight fragments, then (layers that need more than one launch: more than one input
// chunk, or more than one pair of chunks when Cin is a multiple of 64) the fp32 partial sums: per workgroup
// and wave that stores results, dchunk planes x RH rows x 4 units x 1 KB (see part_unit)
size_t conv_mfma_ws_bytes(const Geo &g, int ki, int ko) {
    size_t n = pack_bytes(ki, ko);
    if (prefer_gemm(g, ki, ko)) return n + conv_gemm_ws_bytes(g, ki, ko);
    const PatchPlan p = plan_patches(g, ki, ko);
    const int launches = p.pairs ? ki / (2 * C) : ki / C;
    if (launches > 1)
        n += static_cast<size_t>(p.nblocks) * (p.pairs ? wide::NRG : kWaves) * p.dchunk * (RH * 4 * 256 * sizeof(float));
    return n;
}

bool conv_mfma_gather_supported(const Geo &g, int ki, int ko, sp_dtype_t dt) {
    // one-voxel margins, interiors only, 3-D; in the marching kernels per-lane offsets to the H / W neighbours (and
    // their sum at an edge) must fit the 32-bit staging offsets
    if (!conv_mfma_supported(g, ki, ko, dt) || g.halo != 1 || g.grow != 0 || g.flat || conv_gemm_tensor_forms(g, ki, ko))
        return false;
    const long long lim = ki % (2 * C) == 0 ? 0x3fffffffLL : 0x7fffffffLL;       // see conv_mfma_supported
    return static_cast<long long>(g.tile_vox) * (g.gw + 1) * (ki > ko ? ki : ko) < lim;
}

bool conv_mfma_bits_supported(const Geo &g, int ki, int ko, sp_dtype_t dt) {
    // the 3-D kernels (the widest layers on the fewest voxels and the 2-D variant keep the mask tensor)
    return conv_mfma_supported(g, ki, ko, dt) && !g.flat && !conv_gemm_tensor_forms(g, ki, ko);
}

int launch_conv_mfma(const void *Pin, const void *w, const float *bias, void *Pout, const Geo &g,
                     int ki, int ko, bool relu, bool dgrad, void *ws, hipStream_t s, const void *mask,
                     const ConvSplit *split, bool gather, void *bits, const Exchange *ex) {
    if (gather && !conv_mfma_gather_supported(g, ki, ko, SP_BF16)) return SP_EUNSUPPORTED;
    // one-bit mask: read by the data gradient in place of a mask tensor, written by a forward pass with ReLU
    if (bits && (!conv_mfma_bits_supported(g, ki, ko, SP_BF16) || (split && split->out2) || mask || (!dgrad && !relu)))
        return SP_EUNSUPPORTED;
    const int nci = ki / C, nco = ko / C;
    const int ntap = taps_of(g);
    const PackArgs pack{static_cast<const uint16_t *>(w), static_cast<uint4 *>(ws), nci, nco, ntap, dgrad ? 1 : 0};
    int rc;
    // (no neighbours, and margins that stay as they are: nothing to exchange, and the launch that could takes 0.3 us more)
    const bool alone = (g.flat || g.gd == 1) && g.gh == 1 && g.gw == 1 && ex && (ex->border & SP_HALO_KEEP_ZERO);
    if (ex && !alone) {
        rc = launch_exchange_and_pack(*ex, g, pack, s);
    } else {
        hipLaunchKernelGGL(pack_weights_kernel, dim3(pack_blocks(pack)), dim3(64 * kPackWaves), 0, s, pack);
        rc = record_hip(hipGetLastError());
    }
    if (rc != SP_OK) return rc;
    if (prefer_gemm(g, ki, ko))
        return launch_conv_gemm(Pin, ws, static_cast<char *>(ws) + pack_bytes(ki, ko), bias, Pout, g, ki, ko, relu, dgrad, s,
                                mask, split, gather, bits);
    ConvArgs a;
    a.in = static_cast<const uint16_t *>(Pin);
    a.bias = bias;
    a.out = static_cast<uint16_t *>(Pout);
    a.out2 = nullptr;
    a.out_ca = ko;
    a.out2_cs = 0;
    // two-tensor input: kernel channels [0, in_ca) come from Pin (in_ca per voxel), the rest from split->in2
    const uint16_t *in_a = static_cast<const uint16_t *>(Pin), *in_b = nullptr;
    int in_ca = ki;
    if (split && split->in2) {
        in_b = static_cast<const uint16_t *>(split->in2);
        in_ca = split->in_ca;
    }
    if (split && split->out2) {
        a.out2 = static_cast<uint16_t *>(split->out2);
        a.out_ca = split->out_ca;
        a.out2_cs = ko - split->out_ca;
    }
    // channels per voxel of the first output tensor (the whole output if there is no second one)
    const int out_cs_a = a.out2 ? a.out_ca : ko;
    a.mask = static_cast<const uint16_t *>(mask);
    a.bits = static_cast<uint16_t *>(bits);
    a.part = reinterpret_cast<float *>(static_cast<char *>(ws) + pack_bytes(ki, ko));
    a.g = g;
    a.out_cs = out_cs_a;
    a.nco = nco;
    // source of input chunk c (32 channels from channel 32 c of the concatenated input)
    auto chunk_src = [&](int cchunk, const uint16_t **base, int *cs, int *co) {
        const int c0 = C * cchunk;
        if (in_b && c0 >= in_ca) { *base = in_b; *cs = ki - in_ca; *co = c0 - in_ca; }
        else { *base = in_a; *cs = in_b ? in_ca : ki; *co = c0; }
    };
    const PatchPlan pl = plan_patches(g, ki, ko);
    // (slices side by side stay here: strips of 32 columns would be mostly empty; the bits are the same)
    if (g.flat && ki <= 2 * C && pl.fold == 1) return launch_conv_rows2d(Pin, ws, bias, Pout, g, ki, ko, relu, s, mask, split);
    const bool pairs = pl.pairs;
    a.nh = pl.nh;
    a.nw = pl.nw;
    a.dchunk = pl.dchunk;
    a.nd = pl.nd;
    a.fold = pl.fold;
    a.fold_w = pl.fold_w;
    a.gather = gather ? 1 : 0;
    const long long nb = pl.nblocks;
    if (nb > 0x7ffffff0LL) return SP_EGEOM;
    a.nblocks = static_cast<int>(nb);
    const unsigned grid = static_cast<unsigned>((nb + 7) / 8 * 8);
    using Kern = void (*)(ConvArgs);
    // [mode][bias][epilogue]; combinations that cannot occur (bias after the first launch, ReLU or mask before
    // the last, bias together with a mask) reuse the plain variant.  MB, RB: the two bit forms.
    // [patches][mode][bias][epilogue]; the bit forms exist for the 3-D kernels only (the host refuses them
    // for 2-D geometries; their table entries repeat the plain kernel).  The two-chunk kernels have the same table
    // in their own translation unit (conv_mfma_pair.hip).
    static const Kern kern[3][4][2][5] = {SP3D_CONV_TABLE(conv_mfma_kernel, kWhole3, kMaskBits, kReluBits),
                                          SP3D_CONV_TABLE(conv_mfma_kernel, kRagged3, kMaskBits, kReluBits),
                                          SP3D_CONV_TABLE(conv_mfma_kernel, kAny2, kNone, kNone)};
    // (One patch in 32 cut by the box and kRagged3 is the faster one already: 64 -> 64 on 128 x 126 x 128 in 1 x 1 x 4 tiles, forward
    // 422 us with whole patches and others in one launch, 368 with this, masked data gradient 505 and 368.  A grown box differs
    // from tile to tile.)
    // The two-chunk kernel for whole patches takes others too, with branches (see conv_mfma_pair_kernel.h): on marches of one or two
    // planes it is the faster one where sums or masks are read, as those that are fetched a step ahead are waited for twice: data gradient
    // 32 <- 512 on 34 x 20 x 24 in 2 x 1 x 2 tiles 125 us, 133 without branches, masked 96 <- 64 on 22 x 25 x 30 in 2 x 1 x 1 18.6 and 19.5;
    // over three planes and more kRagged3 is (0.98 of the time with three, 0.91 with more than five; forward in one launch: 0.98 with
    // one or two, too).
    const bool whole = g.grow == 0 && g.th % (pairs ? wide::PH : PH) == 0 && g.tw % PW == 0;
    const bool branches = pairs && pl.dchunk <= 2 && (nci > 2 || mask || (bits && dgrad));
    const int patches = g.flat ? kAny2 : (whole || branches ? kWhole3 : kRagged3);
    const int epi = bits ? (dgrad ? kMaskBits : kReluBits) : (mask ? kMask : (relu ? kRelu : kNone));
    // more than 64 KB of dynamic LDS has to be requested explicitly
    static const hipError_t attr = [] {
        for (int i = 0; i < 120; ++i) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern[i / 40][(i / 10) & 3][(i / 5) & 1][i % 5]),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
            if (e != hipSuccess) return e;
        }
        return conv_mfma_pair_prepare();
    }();
    if (attr != hipSuccess) return record_hip(attr);
    const int nsteps = pairs ? nci / 2 : nci;          // launches: input chunks, or pairs of them
    for (int ci = 0; ci < nsteps; ++ci) {
        const int mode = nsteps == 1 ? kSingle : (ci == 0 ? kFirst : (ci == nsteps - 1 ? kLast : kMiddle));
        chunk_src(pairs ? 2 * ci : ci, &a.in, &a.in_cs, &a.in_co);
        if (pairs) chunk_src(2 * ci + 1, &a.in2, &a.in2_cs, &a.in2_co);
        a.wpack = static_cast<const uint4 *>(ws) + static_cast<size_t>(pairs ? 2 * ci : ci) * nco * NFRAG * 64;
        if (pairs)
            conv_mfma_pair_launch(patches, mode, bias ? 1 : 0, epi, grid, s, a);
        else
            hipLaunchKernelGGL(kern[patches][mode][bias ? 1 : 0][epi], dim3(grid), dim3(kThreads), LDS_BYTES, s, a);
        rc = record_hip(hipGetLastError());
        if (rc != SP_OK) return rc;
    }
    return SP_OK;
}

}  // namespace sp3d
