// bf16 weight (and bias) gradient for layers of at least 64 input and output channels where the marching kernels of
// wgrad_mfma.hip leave the matrix cores short: 2-D layers (a staged plane serves 9 taps there) and volumes whose tiles
// fill little of an 8 x 32 patch.
//
//   dw[row, kw][ci][co] = sum over interior voxels v of x[v + (row, kw)][ci] * dz[v][co]
//
// A GEMM with M = input channels, N = output channels and K = voxels, for the three taps kw of one kernel row (kd, kh) at a
// time: a workgroup owns 128 x 128 channels (8 waves, 4 x 2) or 64 x 64 (4 waves, 2 x 2) of one kernel row, three taps
// in registers, and streams voxels,
// numbered across rows, slices and tiles, 64 per stage.  x comes as in conv_gemm.hip, as the records of the padded rows that
// the stage's voxels touch, each once for the three taps; both operands reach LDS by direct loads, NS stages deep, as
// 64-byte records (32 channels) per channel chunk, and are read with the transposing load (4 voxels of one channel per
// lane).  The two 16-channel halves of a record change places with every fourth record, so that eight neighbouring
// records' halves lie in different banks.  Where the loads go is a table that the threads fill one entry each, NS stages
// ahead: the voxel -> address arithmetic is done once per record, not once per lane and load.
//
// Workgroups: kernel rows x channel tiles x splits of the voxels; the splits' sums are added in order by a second launch.
// Voxels past the last one are masked in both operands (a clamped voxel may hold an infinity).
// What bounds it: LDS reads - 20 transposing reads (10 KB) per wave and 24 MFMAs, 104 of the 128 bytes per clock when the
// matrix cores are full - and for few voxels the launches.  (Four waves of 64 x 64 channels read less but need 192
// accumulators: the compiler then moved them between the halves of the register file in every stage, 450 TFLOP/s.)
// Measured: 1024 -> 1024 channels, 2-D, 16 slices of 32 x 32 425 us, 0.73 PFLOP/s (marching 850; with one running sum over all
// products 376 us, see STAGED); 512 -> 512 there 140 us (one running sum; marching 219); 64 -> 64 on 32^3 32 us (marching 48).
#include "common.h"

#include <type_traits>

namespace sp3d {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int C = 32, kThreads = 256, V = 64;        // channels of a chunk; voxels of a stage
constexpr int kRing = 8;                             // stages whose voxel -> record table is kept

// T: channel chunks of a tile (4: 128 x 128 channels, 2: 64 x 64); LX: groups of 16 x records per stage
constexpr int stage_bytes(int t, int lx) { return t * (lx + V / 16) * 1024; }
constexpr int stages(int t, int lx) { return t == 4 && lx > 5 ? 3 : 4; }
constexpr int table_bytes(int lx) { return (2 * (16 * lx + V) + kRing * V + 1) * 4; }
constexpr int lds_bytes(int t, int lx) { return stages(t, lx) * stage_bytes(t, lx) + table_bytes(lx); }
static_assert(lds_bytes(4, 5) <= 160 * 1024 && lds_bytes(4, 6) <= 160 * 1024 && lds_bytes(4, 8) <= 160 * 1024, "LDS of one CU");

// n / d for n < 2^31 without a branch: floor(n m / 2^(31 + L)) with L = ceil(log2 d), m = ceil(2^(31 + L) / d) < 2^32; the
// error of m is below 2^L / 2^(31 + L) per unit of n (Granlund & Montgomery, as FastDiv in common.h).
struct Div31 { uint32_t d, m, shift; };
Div31 make_div31(uint32_t d) {
    uint32_t l = 0;
    while ((1u << l) < d) ++l;
    return Div31{d, static_cast<uint32_t>(((1ull << (31 + l)) + d - 1) / d), 31 + l};
}
__device__ __forceinline__ uint32_t div31(uint32_t n, const Div31 &f) {
    return static_cast<uint32_t>((static_cast<uint64_t>(n) * f.m) >> f.shift);
}

struct WgradGemmArgs {
    const uint16_t *x, *x2, *dz;     // x2: input channels [x_ca, cin), or null
    int x_cs, x2_cs, x_ca, cin, cout;
    float *out, *out_b;              // [split][tap][cin][cout], [split][cout]
    long long out_stride;            // floats between the splits
    Geo g;
    int nrows, nti, ntj, nsplit;     // kernel rows, channel tiles, splits
    int nvox, nstages, nblocks;
    int bias;
    Div31 drow, drec, dth, dtd;    // tw, tw + 2, th, td
};

__device__ __forceinline__ void dma16(const void *src, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(dst) : "memory");
}
__device__ __forceinline__ s16x4 tr_read(const char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(__attribute__((address_space(3))) char *)(p));
}
union Frag { struct { s16x4 lo, hi; } s; u32x4 w; bf16x8 v; };

// STAGED: the products of a stage are summed from zero and then added to the running sums, which are rounded once per stage
// instead of eight times per instruction (an MFMA adds its 32 products four at a time).
template <int T, int LX, bool GATHER, bool STAGED>
__global__ __launch_bounds__(128 * T, T / 2) void wgrad_gemm_kernel(WgradGemmArgs a) {
    constexpr int NI = 2, NJ = T;                    // blocks of 16 input and output channels per wave: 32 x 16 T
    constexpr int NS = stages(T, LX), STAGE = stage_bytes(T, LX), ZOFF = T * LX * 1024;
    constexpr int LZ = V / 16, L = LX;               // loads per wave and stage
    static_assert((NS - 1) * L < 64, "vmcnt");
    extern __shared__ __align__(16) char lds[];
    int *const pos = reinterpret_cast<int *>(lds + NS * STAGE);  // [2][16 LX + V]: padded voxel of every record / dz voxel
    int *const vrec = pos + 2 * (16 * LX + V);                   // [kRing][V]: record of every voxel inside its stage
    const int per_xcd = gridDim.x >> 3;
    const int logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (logical >= a.nblocks) return;
    const Geo &g = a.g;
    // neighbours (the same XCD, hence the same L2) stream the same voxels: the split is the slowest index
    int u = logical;
    const int r = u % a.nrows; u /= a.nrows;
    const int ti = u % a.nti; u /= a.nti;
    const int tj = u % a.ntj, split = u / a.ntj;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wi = wave & (T - 1), wj = wave / T;
    const int kd = a.nrows == 3 ? 1 : r / 3, kh = a.nrows == 3 ? r : r - 3 * (r / 3);
    const int prow = g.pw, pplane = g.ph * g.pw, tvox = static_cast<int>(g.tile_vox);
    const int s0 = static_cast<int>(1LL * split * a.nstages / a.nsplit), s1 = static_cast<int>(1LL * (split + 1) * a.nstages / a.nsplit);
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char *)lds));

    // Table of stage s, one entry per thread: threads [0, 16 LX) the x records, [128, 192) the dz voxels.  The two are one
    // computation on different numbers (record numbers in rows of tw + 2, tap (kd, kh), column w; voxel numbers in rows of
    // tw, centre, column w + 1), and threads without an entry write a spare word: no branch in the loop.
    const bool zthread = wave >= 2;
    const Div31 &dw0 = a.drec, &dw1 = a.drow;
    const uint32_t fm = zthread ? dw1.m : dw0.m, fs = zthread ? dw1.shift : dw0.shift;
    const int fw = zthread ? g.tw : g.tw + 2, centre = zthread ? pplane + prow + 1 : kd * pplane + kh * prow;
    const int pslot = tid < 16 * LX ? tid : (zthread && tid < 128 + V ? 16 * LX + tid - 128 : -1);
    const int spare = 2 * (16 * LX + V) + kRing * V;
    auto fill = [&](int s) {
        const int q0 = s * V, last = min(q0 + V, a.nvox) - 1;
        const int rec0 = q0 + 2 * static_cast<int>(div31(q0, a.drow)), rec1 = last + 2 * static_cast<int>(div31(last, a.drow)) + 2;
        const int n = zthread ? min(q0 + tid - 128, a.nvox - 1) : min(rec0 + tid, rec1);      // past the last one: that one
        const int row = static_cast<int>((static_cast<uint64_t>(n) * fm) >> fs), w = n - row * fw;
        const int t = static_cast<int>(div31(row, a.dth)), tile = static_cast<int>(div31(t, a.dtd));
        const int h = row - t * g.th, d = t - tile * g.td;
        int at = tile * tvox + d * pplane + h * prow + w + centre;
        if (GATHER && !zthread) {    // (host: one-voxel margins, 3-D) margins that have a neighbour: one tile extent further on
            const int tc = tile % g.gw, t1 = tile / g.gw, tb = t1 % g.gh, ta = (t1 / g.gh) % g.gd;
            const int sw = tvox - g.tw, sh = tvox * g.gw - g.th * prow, sd = tvox * g.gw * g.gh - g.td * pplane;
            at += (w == 0 && tc > 0 ? -sw : 0) + (w == g.tw + 1 && tc < g.gw - 1 ? sw : 0);
            at += (h + kh == 0 && tb > 0 ? -sh : 0) + (h + kh == g.th + 1 && tb < g.gh - 1 ? sh : 0);
            at += (d + kd == 0 && ta > 0 ? -sd : 0) + (d + kd == g.td + 1 && ta < g.gd - 1 ? sd : 0);
        }
        pos[pslot >= 0 ? (s & 1) * (16 * LX + V) + pslot : spare] = at;
        pos[zthread && pslot >= 0 ? 2 * (16 * LX + V) + (s & (kRing - 1)) * V + tid - 128 : spare] = n + 2 * row - rec0;
    };
    // This wave's loads of a stage: group j = records 16 j + lane / 4, 16-byte piece lane % 4 of each in stored order.  The
    // first T waves load a channel chunk of x each, the others one of dz (repeating its last group to the same count).
    const int piece = 8 * ((lane & 3) ^ (((lane >> 4) & 1) << 1));
    const int c0 = C * (ti * T + wi);
    const uint16_t *const xsrc = (a.x2 && c0 >= a.x_ca ? a.x2 + c0 - a.x_ca : a.x + c0) + piece;
    const uint16_t *const src = wj == 0 ? xsrc : a.dz + C * (tj * T + wi) + piece;
    const long long cs = wj == 0 ? (a.x2 && c0 >= a.x_ca ? a.x2_cs : a.x_cs) : a.cout;
    const uint32_t dst0 = lds0 + (wj == 0 ? wi * LX * 1024 : ZOFF + wi * LZ * 1024);
    auto fetch = [&](int s, int slot) {
        const int *const p = pos + (s & 1) * (16 * LX + V) + (wj == 0 ? 0 : 16 * LX) + (lane >> 2);
#pragma unroll
        for (int j = 0; j < LX; ++j) {
            const int jj = wj == 0 ? j : min(j, LZ - 1);
            dma16(src + p[16 * jj] * cs, dst0 + slot * STAGE + jj * 1024);
        }
    };

    // Transposing reads: lane 16 G + q + 4 j reads voxel 4 G + j of a block of 16, channels 4 q .. 4 q + 3 of a half chunk.
    const int G = lane >> 4, quad = lane & 3, vj = 4 * G + ((lane >> 2) & 3);
    int zoff[2];                                      // voxels vj and vj + 16 (+ 32 for the second half of the stage)
#pragma unroll
    for (int b = 0; b < 2; ++b) zoff[b] = ZOFF + (16 * b + vj) * 64 + (((vj >> 2) & 1) << 5) + quad * 8;
    // block n of a wave: half chunk 2 wi + n (x) / wj NJ + n (dz) of the tile
    auto xread = [&](const char *st, int base, int n) {
        return tr_read(st + wi * (LX * 1024) + (base ^ (n << 5)));
    };
    auto zread = [&](const char *st, int base, int n) {
        return tr_read(st + (wj * (NJ / 2) + (n >> 1)) * (LZ * 1024) + (base ^ ((n & 1) << 5)));
    };

    f32x4 acc[3][NI][NJ];
    double accb[NJ];
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[t][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NJ; ++j) accb[j] = 0.0;
    const f32x4 zero{0.f, 0.f, 0.f, 0.f};
    Frag ones;
    ones.w = u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    const bool bias_wave = a.bias && r == 0 && ti == 0 && wi == 0;

#pragma unroll 1
    for (int i = 0; i < NS; ++i) {                    // past the last stage the loads repeat it
        fill(min(s0 + i, s1 - 1));
        __syncthreads();
        fetch(min(s0 + i, s1 - 1), i);
        __syncthreads();
    }

    Frag xf[2][NI], zf[2][NJ];
    int xoff[4][3];                                   // record bases of this lane's voxel in block b, taps kw
    auto offsets = [&](int s) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int rec = vrec[(s & (kRing - 1)) * V + 16 * b + vj];
#pragma unroll
            for (int kw = 0; kw < 3; ++kw) xoff[b][kw] = (rec + kw) * 64 + ((((rec + kw) >> 2) & 1) << 5) + quad * 8;
        }
    };
    auto read_x = [&](const char *st, int gi) {       // group gi = (kw, half of the stage) -> fragment set gi % 2
        const int kb = gi & 1, kw = gi >> 1;
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            xf[gi & 1][n].s.lo = xread(st, xoff[2 * kb][kw], n);
            xf[gi & 1][n].s.hi = xread(st, xoff[2 * kb + 1][kw], n);
        }
    };
    auto read_z = [&](const char *st, int kb) {
#pragma unroll
        for (int n = 0; n < NJ; ++n) {
            zf[kb][n].s.lo = zread(st, zoff[0] + 2048 * kb, n);
            zf[kb][n].s.hi = zread(st, zoff[1] + 2048 * kb, n);
        }
    };
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * L) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    offsets(s0);
    read_z(lds, 0);
    read_x(lds, 0);
    int cur = 0;
    auto step = [&](int s, auto ragged_tag, auto bias_tag) {
        constexpr bool ragged = decltype(ragged_tag)::value, bias = decltype(bias_tag)::value;
        const int nxt = cur + 1 == NS ? 0 : cur + 1;
        const char *const st = lds + cur * STAGE;
        const int ahead = min(s + NS, s1 - 1);
        f32x4 sum[NI][NJ];                            // STAGED: of the stage's 64 voxels
#pragma unroll
        for (int gi = 0; gi < 6; ++gi) {
            const int kb = gi & 1, kw = gi >> 1;
            if (gi == 0) read_z(st, 1);
            if (gi == 1) fill(ahead);
            if (gi < 5) {
                read_x(st, gi + 1);
            } else {
                // every wave has read this stage's last fragments and filled its table entries (lgkmcnt), and the next
                // stage's loads have landed: those of the NS - 2 stages after it may stay in flight
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * L) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                offsets(min(s + 1, s1 - 1));
                read_z(lds + nxt * STAGE, 0);
                read_x(lds + nxt * STAGE, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (gi == 5) fetch(ahead, cur);
            if (ragged) {                             // this lane's values are voxels 4 G .. + 3 of blocks 2 kb, 2 kb + 1
                uint32_t m[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int q = s * V + 32 * kb + 16 * (e >> 1) + 4 * G + 2 * (e & 1);
                    m[e] = (q < a.nvox ? 0xffffu : 0u) | (q + 1 < a.nvox ? 0xffff0000u : 0u);
                }
                const u32x4 mask{m[0], m[1], m[2], m[3]};
#pragma unroll
                for (int n = 0; n < NI; ++n) xf[gi & 1][n].w &= mask;
#pragma unroll
                for (int n = 0; n < NJ; ++n)
                    if (kw == 0) zf[kb][n].w &= mask;
            }
            if (kw == 0 && bias) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) accb[j] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones.v, zf[kb][j].v, zero, 0, 0, 0)[0];
            }
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    if (STAGED)
                        sum[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[gi & 1][i].v, zf[kb][j].v, kb ? sum[i][j] : zero, 0, 0, 0);
                    else
                        acc[kw][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[gi & 1][i].v, zf[kb][j].v, acc[kw][i][j], 0, 0, 0);
                }
            if (STAGED && kb) {
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[kw][i][j] += sum[i][j];
            }
        }
        cur = nxt;
    };
    const int whole = s1 * V > a.nvox ? s1 - 1 : s1;             // the very last stage may hold fewer than V voxels
    auto run = [&](auto bias_tag) {
        for (int s = s0; s < whole; ++s) step(s, std::false_type{}, bias_tag);
        if (whole < s1) step(s1 - 1, std::true_type{}, bias_tag);
    };
    if (bias_wave) run(std::true_type{});
    else run(std::false_type{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the repeated loads

    float *const out = a.out + split * a.out_stride;
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int ci = C * T * ti + 32 * wi + 16 * i + 4 * G + e;
                float *o = out + (static_cast<long long>(3 * r + t) * a.cin + ci) * a.cout + C * T * tj + 16 * wj * NJ + (lane & 15);
#pragma unroll
                for (int j = 0; j < NJ; ++j) o[16 * j] = acc[t][i][j][e];
            }
    if (bias_wave && lane < 16) {                     // row 0 of the ones-product: the column sums
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            a.out_b[split * a.out_stride + C * T * tj + 16 * (wj * NJ + j) + lane] = static_cast<float>(accb[j]);
    }
}

// dw and db as the splits' sums in fp64, four values per thread and run (ndw and cout are multiples of four; db may lie
// anywhere): run r adds the splits r, r + 4, ... in order, then the runs are added.  A block serves 64 neighbouring fours.
// What bounds it: HBM for wide layers, the chain of loads for narrow ones, which the runs cut to a quarter.
__global__ __launch_bounds__(kThreads) void wgrad_gemm_join_kernel(const float4 *__restrict__ part, float4 *__restrict__ dw,
                                                                   float *__restrict__ db, long long ndw4, long long n4, int nsplit) {
    __shared__ double red[3][4][64];
    const int l = threadIdx.x & 63, run = threadIdx.x >> 6;
    const long long e = 64LL * blockIdx.x + l;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (e < n4) {
#pragma unroll 8
        for (int p = run; p < nsplit; p += 4) {
            const float4 v = part[p * n4 + e];
            s[0] += v.x; s[1] += v.y; s[2] += v.z; s[3] += v.w;
        }
    }
    if (run) {
#pragma unroll
        for (int i = 0; i < 4; ++i) red[run - 1][i][l] = s[i];
    }
    __syncthreads();
    if (run || e >= n4) return;
    float f[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = static_cast<float>((s[i] + red[0][i][l]) + (red[1][i][l] + red[2][i][l]));
    if (e < ndw4) {
        dw[e] = make_float4(f[0], f[1], f[2], f[3]);
    } else if (db) {
#pragma unroll
        for (int i = 0; i < 4; ++i) db[4 * (e - ndw4) + i] = f[i];
    }
}

// Splits of the voxels: what costs least in microseconds if 256 compute units take the workgroups in rounds, those of 64 x 64
// channels two at a time (LDS).  Fitted to 382 measured layers (6 % rms): a stage lasts 1.37 us (128 x 128 channels; 1.59 summed
// by stage), 0.96 us (64 x 64; 1.2 for both of a pair of workgroups), a workgroup 8.8 and 7 us besides, launch included; the
// splits' sums are written and read at 5.4 TB/s.  They stay within SP_STATIC_SCRATCH_BYTES, so that conv3d_wgrad_static takes
// every layer it takes with the marching kernels.
struct Plan { int t, lx, nsplit, nblocks, staged; double us; };
Plan plan(const Geo &g, int cin, int cout) {
    Plan p;
    p.t = cin % (4 * C) == 0 && cout % (4 * C) == 0 ? 4 : 2;
    const int rows = V % g.tw == 0 ? V / g.tw - 1 : (V + g.tw - 2) / g.tw;      // row ends that 64 voxels cross at most
    const int lx = (V + 2 + 2 * rows + 15) / 16;
    p.lx = lx <= 5 ? 5 : (lx <= 6 ? 6 : 8);
    const long long nvox = 1LL * g.ntiles * g.int_vox, stages = (nvox + V - 1) / V;
    const long long tiles = (g.flat ? 3LL : 9LL) * (cin / (C * p.t)) * (cout / (C * p.t));
    const double bytes = 4.0 * (1.0 * taps_of(g) * cin * cout + cout);
    const int groups = wgrad_march_groups(g, cin, cout);
    p.us = 0;
    p.nsplit = 1;
    for (int s = 1; s <= 256 && s <= stages && (s == 1 || (s * bytes <= SP_STATIC_SCRATCH_BYTES && tiles * s <= 1024)); ++s) {
        const long long wgs = tiles * s, left = wgs % 512;
        const bool staged = s < 2 * groups;
        const double n = static_cast<double>((stages + s - 1) / s);
        double us = s > 1 ? 2.4 + 2 * s * bytes / 5.4e6 : 0;
        if (p.t == 4) us += (wgs + 255) / 256 * (n * (staged ? 1.59 : 1.37) + 8.8);
        else us += (wgs / 512 + (left > 256)) * (n * 1.2 + 7) + (left > 0 && left <= 256 ? n * 0.97 + 7 : 0);
        if (s == 1 || us < p.us) { p.us = us; p.nsplit = s; }
    }
    p.nblocks = static_cast<int>(tiles * p.nsplit);
    // The running sums may be no longer than those of the marching kernels, which add up two halves of every workgroup's
    // voxels.  Where the splits are as many, one sum over all products is exact enough; where they are fewer, a sum per stage
    // keeps the error below theirs (against 64 bits, marching, one sum, per stage: 512 -> 64 on 18 x 16 x 16 1.1e-7, 2.2e-7,
    // 1.1e-7; 128 -> 512 on 17 x 24 x 22 2.7e-7, 2.8e-7, 1.2e-7; 2-D 128 -> 64 on 2 x 288 x 256 2.9e-7, 3.8e-7, 1.6e-7).  It costs
    // 32 (T = 4) additions per wave for 16 products: 1024 -> 1024, 2-D, 16 x 32 x 32 376 -> 426 us.
    p.staged = p.nsplit < 2 * groups;
    return p;
}

}  // namespace

bool wgrad_gemm_supported(const Geo &g, int cin, int cout) {
    // voxels are numbered in 32 bits, with two records per row end; a stage's records fit 8 groups of 16
    return cin % (2 * C) == 0 && cout % (2 * C) == 0 && g.tw >= 2 && 1LL * g.ntiles * g.tile_vox < (1LL << 30);
}

double wgrad_gemm_us(const Geo &g, int cin, int cout) { return plan(g, cin, cout).us; }

void wgrad_gemm_detail(const Geo &g, int cin, int cout, int *detail) {
    const Plan p = plan(g, cin, cout);
    detail[0] = p.t; detail[1] = p.lx; detail[2] = p.nsplit; detail[3] = p.staged;
}

size_t wgrad_gemm_ws_bytes(const Geo &g, int cin, int cout) {
    const Plan p = plan(g, cin, cout);
    return p.nsplit == 1 ? 0 : p.nsplit * (static_cast<size_t>(taps_of(g)) * cin * cout + cout) * sizeof(float);
}

int launch_wgrad_gemm(const void *Px, const void *Pdz, float *dw, float *db, const Geo &g, int cin, int cout, void *ws,
                      hipStream_t s, const void *Px2, int ca, bool gather) {
    const Plan p = plan(g, cin, cout);
    WgradGemmArgs a;
    a.x = static_cast<const uint16_t *>(Px);
    a.x2 = static_cast<const uint16_t *>(Px2);
    a.dz = static_cast<const uint16_t *>(Pdz);
    a.x_ca = a.x_cs = Px2 ? ca : cin;
    a.x2_cs = cin - a.x_ca;
    a.cin = cin; a.cout = cout;
    const long long ndw = static_cast<long long>(taps_of(g)) * cin * cout;
    a.out = p.nsplit == 1 ? dw : static_cast<float *>(ws);
    a.out_b = p.nsplit == 1 ? db : a.out + ndw;
    a.out_stride = ndw + cout;
    a.g = g;
    a.nrows = g.flat ? 3 : 9;
    a.nti = cin / (C * p.t); a.ntj = cout / (C * p.t);
    a.nsplit = p.nsplit;
    a.nvox = static_cast<int>(g.ntiles * g.int_vox);
    a.nstages = (a.nvox + V - 1) / V;
    a.nblocks = p.nblocks;
    a.bias = db != nullptr || p.nsplit > 1;
    a.drow = make_div31(g.tw);
    a.drec = make_div31(g.tw + 2);
    a.dth = make_div31(g.th);
    a.dtd = make_div31(g.td);
    using Kern = void (*)(WgradGemmArgs);
    // [staged][tile][record groups; gathered halos: whole 8 x 32 patches, rows of at least 32]
#define SP3D_TILES(T, S) {wgrad_gemm_kernel<T, 5, false, S>, wgrad_gemm_kernel<T, 6, false, S>, wgrad_gemm_kernel<T, 8, false, S>, \
                          wgrad_gemm_kernel<T, 5, true, S>}
    static const Kern kern[2][2][4] = {{SP3D_TILES(2, false), SP3D_TILES(4, false)}, {SP3D_TILES(2, true), SP3D_TILES(4, true)}};
#undef SP3D_TILES
    static const int lxs[4] = {5, 6, 8, 5};
    // more than 64 KB of dynamic LDS has to be requested explicitly
    static const hipError_t attr = [] {
        for (int i = 0; i < 16; ++i) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern[i / 8][i / 4 % 2][i % 4]),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes(i / 4 % 2 ? 4 : 2, lxs[i % 4]));
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (attr != hipSuccess) return record_hip(attr);
    if (gather && p.lx != 5) return SP_EUNSUPPORTED;
    const int k = gather ? 3 : (p.lx == 5 ? 0 : (p.lx == 6 ? 1 : 2));
    hipLaunchKernelGGL(kern[p.staged][p.t / 2 - 1][k], dim3(static_cast<unsigned>((p.nblocks + 7) / 8 * 8)), dim3(128 * p.t), lds_bytes(p.t, p.lx), s, a);
    int rc = record_hip(hipGetLastError());
    if (rc != SP_OK || p.nsplit == 1) return rc;
    const long long n4 = (ndw + cout) / 4;
    hipLaunchKernelGGL(wgrad_gemm_join_kernel, dim3(static_cast<unsigned>((n4 + 63) / 64)), dim3(kThreads), 0, s,
                       static_cast<const float4 *>(ws), reinterpret_cast<float4 *>(dw), db, ndw / 4, n4, p.nsplit);
    return record_hip(hipGetLastError());
}

}  // namespace sp3d
