// Convolution in fp32 arithmetic on the matrix cores, any channel count, f32 or bf16 tensors: the fp32 layers, bf16
// layers whose output channels are no multiple of 32, 1x1x1 convolutions that glue_kernels.hip does not serve, and the
// gradient with respect to an image.  Kernel extent 3 or 1 per axis (1 along D in the 2-D variant).
//
// Forward and data gradient: an implicit GEMM on v_mfma_f32_16x16x4_f32 (fp32 products and sums), M = 16 output
// channels, N = 16 voxels, K = (tap, input channel).  A workgroup stages the input of a brick of output voxels, with its
// surround, once in LDS and takes all taps from there.  The four K values of an instruction are free to name, as long
// as both operands agree: lane group q = lane / 16 supplies the channel quad 4 s + q of step s, and the four
// instructions of a step walk through the quad, so that ONE 16-byte LDS read per lane feeds four of them (and one
// weight read serves all of a wave's voxels).  A quad is four channels of one tap; records of fewer channels than 16
// simply put several taps side by side, so 8 channels fill the instructions as well as 16 do.  The offset of a quad
// inside the staged brick comes from a small table in LDS, which keeps channel count, kernel extent and brick shape
// run-time values.  LDS records are an odd number of 16-byte units apart (no bank conflicts between the 16 voxels).
// What bounds it: at 16 channels the instructions' 32 cycles each (a brick of 256 voxels: 432 per wave against 600
// staged records of 64 bytes); at 1 - 4 channels and in small volumes the staging and the launch.
// Measured, fp32, 8 -> 16 -> 16 channels on 51 x 62 x 70 (one thread per output with scalar FMAs before): forward 255 and
// 486 us, data gradient 759 and 2732 us -> 31 ... 54 us each (16 -> 16: 3.06 GFLOP, 60 TFLOP/s); 8 -> 16 on 32^3 44 -> 10 us.
// Of the 50 us of a 16 -> 16 forward pass the products take 29 (20 at the instructions' rate), weights and launch 8, two
// bricks of staging 10.  (Operands read at the top of the step that multiplies them: 54 us, 32 -> 32 on 64^3 190 -> 180.
// Tried without gain: the next brick's records on their way in registers, neighbouring bricks on one XCD.)
//
// Weight gradient: M = rows (tap, input channel) of dw, flattened, so that 16 rows may span taps; N = 16 output
// channels; K = 4 voxels.  A wave keeps ALL rows of a 16 x 16 channel block (27 blocks of 16 rows = 108 registers) over
// every brick it sees: per 4 voxels one read of dz and one of x per instruction.  Partial sums per workgroup, added in
// workgroup order by a second kernel, so results are reproducible.
#include "common.h"

namespace sp3d {

namespace {

constexpr int kThreads = 256, kWaves = 4;
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename E> __device__ __forceinline__ float ldf(const E *p, long long i);
template <> __device__ __forceinline__ float ldf<float>(const float *p, long long i) { return p[i]; }
template <> __device__ __forceinline__ float ldf<uint16_t>(const uint16_t *p, long long i) {
    return bf16_to_f32(p[i]);
}
template <typename E> __device__ __forceinline__ f32x4 ldf4(const E *p);
template <> __device__ __forceinline__ f32x4 ldf4<float>(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
template <> __device__ __forceinline__ f32x4 ldf4<uint16_t>(const uint16_t *p) {
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    return f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                 __uint_as_float(v.y & 0xffff0000u)};
}
template <typename E> __device__ __forceinline__ void stf(E *p, float v);
template <> __device__ __forceinline__ void stf<float>(float *p, float v) { *p = v; }
template <> __device__ __forceinline__ void stf<uint16_t>(uint16_t *p, float v) { *p = f32_to_bf16(v); }
template <typename E> __device__ __forceinline__ void stf4(E *p, f32x4 v);
template <> __device__ __forceinline__ void stf4<float>(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }
template <> __device__ __forceinline__ void stf4<uint16_t>(uint16_t *p, f32x4 v) {
    *reinterpret_cast<uint2 *>(p) = make_uint2(f32_to_bf16(v[0]) | (static_cast<uint32_t>(f32_to_bf16(v[1])) << 16),
                                               f32_to_bf16(v[2]) | (static_cast<uint32_t>(f32_to_bf16(v[3])) << 16));
}

// A brick of output voxels and the box of input voxels ("records") that its taps read.
struct BrickGeo {
    int s, r, c;                 // output voxels along D, H, W
    int kd, ks;                  // kernel extent along D, and along H and W
    int ns, nr, nc;              // bricks that cover the largest output box
    int nbricks;                 // over all tiles
    int nrec;                    // records: (s + kd - 1) * (r + ks - 1) * (c + ks - 1)
    FastDiv dvc, dvrc;           // voxel index of the brick -> coordinates: c, r * c
    FastDiv drc, drrc;           // record index -> coordinates: c + ks - 1, (r + ks - 1) * (c + ks - 1)
    FastDiv dnc, dnr, dns;       // brick index -> position
};

struct BrickPos {
    bool any;                    // false: the brick lies outside its tile's output box
    TileBox bx;
    long long base;              // padded voxel index of the corner one voxel before the output box
    int d0, h0, w0;              // first output voxel, in coordinates of the box
};

__device__ __forceinline__ BrickPos brick_pos(const Geo &g, const BrickGeo &b, uint32_t brick) {
    uint32_t t = brick, q;
    BrickPos p;
    q = fdiv(t, b.dnc); p.w0 = static_cast<int>(fmod_(t, q, b.dnc)) * b.c; t = q;
    q = fdiv(t, b.dnr); p.h0 = static_cast<int>(fmod_(t, q, b.dnr)) * b.r; t = q;
    q = fdiv(t, b.dns); p.d0 = static_cast<int>(fmod_(t, q, b.dns)) * b.s; t = q;
    p.bx = tile_box(g, static_cast<int>(t));
    p.base = static_cast<long long>(t) * g.tile_vox + p.bx.org;
    p.any = p.d0 < p.bx.bd && p.h0 < p.bx.bh && p.w0 < p.bx.bw;
    return p;
}

// Padded voxel index of record `rec`.  Records beyond what the box's own voxels read (bricks that stick out of it) are
// moved to the nearest one inside: their values reach no result, and nothing outside the tile is touched.
__device__ __forceinline__ long long record_voxel(const Geo &g, const BrickGeo &b, const BrickPos &p, uint32_t rec) {
    const uint32_t i = fdiv(rec, b.drrc), r1 = fmod_(rec, i, b.drrc), j = fdiv(r1, b.drc), k = fmod_(r1, j, b.drc);
    const int od = b.kd / 2, o = b.ks / 2;
    const int d = min(p.d0 + static_cast<int>(i) - od, p.bx.bd - 1 + od), h = min(p.h0 + static_cast<int>(j) - o, p.bx.bh - 1 + o),
              w = min(p.w0 + static_cast<int>(k) - o, p.bx.bw - 1 + o);
    return p.base + (1LL * (d + 1) * g.ph + h + 1) * g.pw + w + 1;
}

// Record offset of tap t: the record of output voxel (0, 0, 0) of the brick at that tap.
__device__ __forceinline__ int tap_record(const BrickGeo &b, int t) {
    const int kk = b.ks * b.ks, kd = t / kk, r = t - kd * kk, kh = r / b.ks, kw = r - kh * b.ks;
    return (kd * (b.r + b.ks - 1) + kh) * (b.c + b.ks - 1) + kw;
}
__device__ __forceinline__ int voxel_record(const BrickGeo &b, uint32_t v, int *d, int *h, int *w) {
    const uint32_t i = fdiv(v, b.dvrc), r1 = fmod_(v, i, b.dvrc), j = fdiv(r1, b.dvc), k = fmod_(r1, j, b.dvc);
    *d = static_cast<int>(i); *h = static_cast<int>(j); *w = static_cast<int>(k);
    return static_cast<int>((i * (b.r + b.ks - 1) + j) * (b.c + b.ks - 1) + k);
}

// Stage channels [c0, c0 + kc) of the brick's records as floats, `stride` floats apart (channels beyond `ki`: zeros).
// Four loads per thread are in flight at a time, two times four where the channels do not come in whole quads (dq divides by
// the number of quads, the last one partial); a loop over the channels of a record where that is
// a single quad or the quads are less than three quarters full (weight gradient of 1 -> 24 on 63 x 96 x 113: 77 us, in quads
// 85; 3 -> 3 on 98 x 122 x 180 216, in quads 235).
template <typename E>
__device__ __forceinline__ void stage_records(const E *__restrict__ in, float *xs, const Geo &g, const BrickGeo &b,
                                              const BrickPos &p, int ki, int c0, int kc, int stride, const FastDiv &dq) {
    if ((ki & 3) == 0 && (kc & 3) == 0) {
        const uint32_t nq = static_cast<uint32_t>(kc) >> 2, n = b.nrec * nq;
        for (uint32_t e0 = threadIdx.x; e0 < n; e0 += 4 * kThreads) {
            f32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t e = min(e0 + u * kThreads, n - 1), rec = fdiv(e, dq);
                const int c = c0 + 4 * static_cast<int>(fmod_(e, rec, dq));
                v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (c < ki) v[u] = ldf4<E>(in + record_voxel(g, b, p, rec) * ki + c);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t e = e0 + u * kThreads;
                if (e < n) {
                    const uint32_t rec = fdiv(e, dq);
                    *reinterpret_cast<f32x4 *>(xs + rec * stride + 4 * fmod_(e, rec, dq)) = v[u];
                }
            }
        }
    } else if (kc < 4 || kc < 3 * ((kc + 3) >> 2)) {
        for (uint32_t rec = threadIdx.x; rec < static_cast<uint32_t>(b.nrec); rec += kThreads) {
            const E *src = in + record_voxel(g, b, p, rec) * ki + c0;
            for (int c = 0; c < kc; ++c) xs[rec * stride + c] = c0 + c < ki ? ldf<E>(src, c) : 0.f;
        }
    } else {
        const uint32_t nq = static_cast<uint32_t>(kc + 3) >> 2, n = b.nrec * nq;
        for (uint32_t e0 = threadIdx.x; e0 < n; e0 += 2 * kThreads) {
            float v[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t e = min(e0 + u * kThreads, n - 1), rec = fdiv(e, dq);
                const int c = c0 + 4 * static_cast<int>(fmod_(e, rec, dq));
                const E *src = in + record_voxel(g, b, p, rec) * ki + c;
#pragma unroll
                for (int j = 0; j < 4; ++j) v[u][j] = c + j < ki ? ldf<E>(src, j) : 0.f;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t e = e0 + u * kThreads;
                if (e >= n) continue;
                const uint32_t rec = fdiv(e, dq);
                const int c = 4 * static_cast<int>(fmod_(e, rec, dq));
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (c + j < kc) xs[rec * stride + c + j] = v[u][j];
            }
        }
    }
}

struct ConvDirectArgs {
    const void *in, *w, *mask;
    const float *bias;
    void *out;
    Geo g;
    BrickGeo b;
    int ki, ko, ntap;
    int kc, nck, stride;         // channels per staged chunk (a multiple of 4), chunks, floats per LDS record
    int steps;                   // K steps of 4 quads per chunk
    int dgrad, relu;
    FastDiv dq;                  // kc / 4
};

// NV: voxel segments of 16 per wave (the brick has 64 NV voxels).  blockIdx.y: block of 16 output channels.
template <typename E, int NV>
__global__ __launch_bounds__(kThreads) void conv_direct_kernel(ConvDirectArgs a) {
    extern __shared__ __align__(16) float lds[];
    float *const xs = lds, *const wts = lds + static_cast<size_t>(a.b.nrec) * a.stride;
    int *const tab = reinterpret_cast<int *>(wts + a.steps * 256);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, q = lane >> 4;
    const int nq = a.kc >> 2, nquads = a.ntap * nq;
    const E *const in = static_cast<const E *>(a.in), *const w = static_cast<const E *>(a.w);
    const int co0 = blockIdx.y * 16 + 4 * q;       // this lane's four output channels

    for (int k = tid; k < 4 * a.steps; k += kThreads) {
        const int kg = min(k, nquads - 1), t = kg / nq;
        tab[k] = tap_record(a.b, t) * a.stride + 4 * (kg - t * nq);
    }
    // (four quads of weights per thread on their way at a time)
    auto stage_weights = [&](int chunk) {
        for (int e0 = tid; e0 < a.steps * 64; e0 += 4 * kThreads) {
            f32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = min(e0 + u * kThreads, a.steps * 64 - 1);
                const int l = e & 63, kg = 4 * (e >> 6) + (l >> 4), co = blockIdx.y * 16 + (l & 15);
                const int t = static_cast<int>(fdiv(kg, a.dq)), c = chunk * a.kc + 4 * (kg - t * nq);
                v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (kg < nquads && co < a.ko) {
                    const E *const src = a.dgrad ? w + (1LL * (a.ntap - 1 - t) * a.ko + co) * a.ki + c : w + (1LL * t * a.ki + c) * a.ko + co;
                    const int step = a.dgrad ? 1 : a.ko;
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (c + j < a.ki) v[u][j] = ldf<E>(src, 1LL * j * step);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (e0 + u * kThreads < a.steps * 64) *reinterpret_cast<f32x4 *>(wts + 4 * (e0 + u * kThreads)) = v[u];
        }
    };
    f32x4 init;
#pragma unroll
    for (int i = 0; i < 4; ++i) init[i] = a.bias && co0 + i < a.ko ? a.bias[co0 + i] : 0.f;

    int rec[NV], vd[NV], vh[NV], vw[NV];            // this lane's voxels: LDS float offset, brick coordinates
    bool real[NV];
#pragma unroll
    for (int n = 0; n < NV; ++n) {
        const uint32_t v = (wave * NV + n) * 16 + col;
        real[n] = v < static_cast<uint32_t>(a.b.s * a.b.r * a.b.c);
        rec[n] = voxel_record(a.b, real[n] ? v : 0u, &vd[n], &vh[n], &vw[n]) * a.stride;
    }

    bool have_weights = false;
    for (uint32_t brick = blockIdx.x; brick < static_cast<uint32_t>(a.b.nbricks); brick += gridDim.x) {
        const BrickPos p = brick_pos(a.g, a.b, brick);
        if (!p.any) continue;
        f32x4 acc[NV];
#pragma unroll
        for (int n = 0; n < NV; ++n) acc[n] = init;
        for (int chunk = 0; chunk < a.nck; ++chunk) {
            __syncthreads();                        // everybody is done with the previous brick / chunk
            if (a.nck > 1 || !have_weights) stage_weights(chunk);
            have_weights = true;
            stage_records<E>(in, xs, a.g, a.b, p, a.ki, chunk * a.kc, a.kc, a.stride, a.dq);
            __syncthreads();
            // the operands of step s + 1 are read before the products of step s, their offset a step earlier still
            f32x4 x[2][NV], wt[2];
            int off = tab[q];
            auto read = [&](int s, int b) {
                wt[b] = *reinterpret_cast<const f32x4 *>(wts + (s * 64 + lane) * 4);
#pragma unroll
                for (int n = 0; n < NV; ++n) x[b][n] = *reinterpret_cast<const f32x4 *>(xs + rec[n] + off);
                off = tab[4 * min(s + 1, a.steps - 1) + q];
            };
            auto products = [&](int s, int b) {
                // quads past the last one repeat the last quad's voxels; both operands are zero there (zero weights
                // alone would turn an infinite voxel into NaN)
                if (4 * s + 3 >= nquads) {
#pragma unroll
                    for (int n = 0; n < NV; ++n)
#pragma unroll
                        for (int j = 0; j < 4; ++j) x[b][n][j] = 4 * s + q < nquads ? x[b][n][j] : 0.f;
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int n = 0; n < NV; ++n) acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(wt[b][j], x[b][n][j], acc[n], 0, 0, 0);
            };
            read(0, 0);
            for (int s = 0; s < a.steps; s += 2) {
                if (s + 1 < a.steps) read(s + 1, 1);
                __builtin_amdgcn_sched_barrier(0);
                products(s, 0);
                if (s + 2 < a.steps) read(s + 2, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (s + 1 < a.steps) products(s + 1, 1);
            }
        }
#pragma unroll
        for (int n = 0; n < NV; ++n) {
            const int d = p.d0 + vd[n], h = p.h0 + vh[n], wv = p.w0 + vw[n];
            if (!real[n] || d >= p.bx.bd || h >= p.bx.bh || wv >= p.bx.bw) continue;
            const long long o = (p.base + (1LL * (d + 1) * a.g.ph + h + 1) * a.g.pw + wv + 1) * a.ko + co0;
            f32x4 v = acc[n];
            if (a.relu) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = v[i] < 0.f ? 0.f : v[i];
            }
            E *dst = static_cast<E *>(a.out) + o;
            const E *m = static_cast<const E *>(a.mask) + o;       // backward of the ReLU that produced the input
            if ((a.ko & 3) == 0) {
                if (co0 >= a.ko) continue;
                if (a.mask) {
                    const f32x4 mv = ldf4<E>(m);
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = mv[i] > 0.f ? v[i] : 0.f;
                }
                stf4<E>(dst, v);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (co0 + i < a.ko) stf<E>(dst + i, a.mask && !(ldf<E>(m, i) > 0.f) ? 0.f : v[i]);
            }
        }
    }
}

// One thread per (voxel of the output box, output channel), scalar FMAs: where a call has so few products that staging bricks
// costs more than they do (see prefer_threads).  KS = kernel extent per axis; with `dgrad` the taps are mirrored and w is read
// as w[tap][ko][ki].  A thread whose voxel lies beyond a side on which its tile has no neighbour has nothing to do.
// What bounds it: the loads, one line per lane at worst, and the chain of ntap * ki products per thread.
template <typename E, bool DGRAD, int KS>
__global__ __launch_bounds__(kThreads) void conv_threads_kernel(const E *__restrict__ in, const E *__restrict__ w,
                                                                const float *__restrict__ bias, E *__restrict__ out, Geo g, int ki,
                                                                int ko, int relu, long long total, const E *__restrict__ mask) {
    const int gd_ = grow_d(g), ed = g.td + 2 * gd_, eh = g.th + 2 * g.grow, ew = g.tw + 2 * g.grow;
    const long long box_vox = 1LL * ed * eh * ew;
    const unsigned ehw = static_cast<unsigned>(eh) * ew;
    constexpr int O = KS / 2;
    const int KD = g.flat ? 1 : KS, OD = KD / 2;
    const long long idx = 1LL * blockIdx.x * kThreads + threadIdx.x;
    if (idx >= total) return;
    const int co = static_cast<int>(idx % ko);
    const long long v = idx / ko, tile = v / box_vox;
    const unsigned r = static_cast<unsigned>(v % box_vox);
    // padded coordinates of the output voxel
    const int pd = static_cast<int>(r / ehw) + g.halo - gd_, ph = static_cast<int>((r % ehw) / ew) + g.halo - g.grow,
              pw = static_cast<int>(r % ew) + g.halo - g.grow;
    if (g.grow > 0) {
        const int tc = static_cast<int>(tile % g.gw), tb = static_cast<int>((tile / g.gw) % g.gh),
                  ta = static_cast<int>((tile / (1LL * g.gw * g.gh)) % g.gd);
        if ((pd < g.halo && ta == 0) || (pd >= g.halo + g.td && ta == g.gd - 1) || (ph < g.halo && tb == 0) ||
            (ph >= g.halo + g.th && tb == g.gh - 1) || (pw < g.halo && tc == 0) || (pw >= g.halo + g.tw && tc == g.gw - 1))
            return;
    }
    const long long base = tile * g.tile_vox;
    float acc = bias ? bias[co] : 0.f;
    for (int kd = 0; kd < KD; ++kd)
        for (int kh = 0; kh < KS; ++kh)
            for (int kw = 0; kw < KS; ++kw) {
                const E *x = in + (base + (1LL * (pd + kd - OD) * g.ph + ph + kh - O) * g.pw + pw + kw - O) * ki;
                const int tap = DGRAD ? ((KD - 1 - kd) * KS + KS - 1 - kh) * KS + KS - 1 - kw : (kd * KS + kh) * KS + kw;
                const E *wt = DGRAD ? w + (1LL * tap * ko + co) * ki : w + 1LL * tap * ki * ko + co;
                for (int c = 0; c < ki; ++c) acc = fmaf(ldf<E>(x, c), ldf<E>(wt, DGRAD ? c : 1LL * c * ko), acc);
            }
    if (relu && acc < 0.f) acc = 0.f;
    const long long o = (base + (1LL * pd * g.ph + ph) * g.pw + pw) * ko + co;
    if (mask && !(ldf<E>(mask, o) > 0.f)) acc = 0.f;      // backward of the ReLU that produced the input
    stf<E>(out + o, acc);
}

struct WgradDirectArgs {
    const void *x, *dz;
    float *part;                 // [workgroup along x][ntap * cin * cout, then cout]
    Geo g;                       // (grow = 0)
    BrickGeo b;
    int cin, cout, ntap;
    int kc, bias;                // channels per chunk; bias: sum dz as well
    int share;                   // voxels of a brick per wave
    FastDiv dq, dkc;             // ceil(kc / 4), kc
};

constexpr int kWgradVox = 256;   // voxels of a brick at most

// blockIdx.x: share of the bricks, blockIdx.y: block of 16 output channels, blockIdx.z: chunk of input channels.  MB: blocks of 16
// rows, at least ceil(ntap * kc / 16).
template <typename E, int MB>
__global__ __launch_bounds__(kThreads, 2) void wgrad_direct_kernel(WgradDirectArgs a) {
    extern __shared__ __align__(16) float lds[];
    float *const dzs = lds, *const xs = lds + kWgradVox * 16;
    int *const vrec = reinterpret_cast<int *>(xs + ((a.b.nrec * a.kc + 3) & ~3));
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, q = lane >> 4;
    const int chunk = blockIdx.z, cob = blockIdx.y;
    const int c0 = chunk * a.kc, rows = a.ntap * a.kc, co = cob * 16 + col;
    const int nvox = a.b.s * a.b.r * a.b.c;
    const E *const x = static_cast<const E *>(a.x), *const dz = static_cast<const E *>(a.dz);

    // LDS float offset of this lane's row of every row block (the taps' records come from a table: they take three
    // divisions by run-time values, 27 times in every lane)
    int *const taps = reinterpret_cast<int *>(lds);
    if (tid < a.ntap) taps[tid] = tap_record(a.b, tid) * a.kc;
    __syncthreads();
    int off[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        const int row = 16 * m + col, t = static_cast<int>(fdiv(row, a.dkc));
        off[m] = row < rows ? taps[min(t, a.ntap - 1)] + row - t * a.kc : 0;
    }
    f32x4 acc[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
    double bsum = 0.0;

    for (uint32_t brick = blockIdx.x; brick < static_cast<uint32_t>(a.b.nbricks); brick += gridDim.x) {
        const BrickPos p = brick_pos(a.g, a.b, brick);
        __syncthreads();
        stage_records<E>(x, xs, a.g, a.b, p, a.cin, c0, a.kc, a.kc, a.dq);
        // dz, zero for voxels outside the tile and channels beyond the last; x counts as zero at those voxels as well
        // (vrec < 0), so that the products vanish also where a neighbour's record holds an infinity
        for (int e = tid; e < kWaves * a.share * 4; e += kThreads) {
            const int v = e >> 2, c4 = cob * 16 + 4 * (e & 3);
            int d, h, w;
            const int vr = voxel_record(a.b, v < nvox ? v : 0, &d, &h, &w) * a.kc;
            d += p.d0; h += p.h0; w += p.w0;
            const bool live = v < nvox && d < p.bx.bd && h < p.bx.bh && w < p.bx.bw;
            if ((e & 3) == 0) vrec[v] = live ? vr : -1;
            f32x4 z{0.f, 0.f, 0.f, 0.f};
            if (live) {
                const E *src = dz + (p.base + (1LL * (d + 1) * a.g.ph + h + 1) * a.g.pw + w + 1) * a.cout + c4;
                if ((a.cout & 3) == 0) {
                    if (c4 < a.cout) z = ldf4<E>(src);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (c4 + i < a.cout) z[i] = ldf<E>(src, i);
                }
            }
            *reinterpret_cast<f32x4 *>(dzs + 4 * e) = z;
        }
        __syncthreads();
        // 16 voxels at a time, summed from zero and then added: the chain that rounds against the whole sum is 16 times
        // shorter (1 -> 8 channels on 132 x 112 x 115, error against 64 bits 8.8e-7 -> 2.1e-7).  Voxels of a brick inside its
        // box first; where x has to be masked, a loop of its own (with the mask in the main loop the 8 -> 16 -> 16 pair's
        // weight gradients took 110 -> 165 us)
        constexpr int MG = MB % 9 == 0 ? 9 : (MB % 7 == 0 ? 7 : MB);
        const bool inside = p.d0 + a.b.s <= p.bx.bd && p.h0 + a.b.r <= p.bx.bh && p.w0 + a.b.c <= p.bx.bw;
        const int mine = min(max(nvox - wave * a.share, 0), a.share), whole = inside ? mine & ~15 : 0;
        const int v0 = wave * a.share + q;
        auto sixteen = [&](int k, auto masked_tag) {
            constexpr bool masked = decltype(masked_tag)::value;
            float b[4];
            int vr[4];
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                b[n] = dzs[(v0 + k + 4 * n) * 16 + col];
                vr[n] = vrec[v0 + k + 4 * n];
            }
            bsum += (b[0] + b[1]) + (b[2] + b[3]);
            // steps (group of row blocks, quad of voxels); the x values of a step are read before the products of the last
            constexpr int NG = MB / MG;
            float xv[2][MG];
            f32x4 t[MG];
            auto read = [&](int i) {
                const float *xr = xs + (masked ? max(vr[i & 3], 0) : vr[i & 3]);
                const uint32_t keep = masked && vr[i & 3] < 0 ? 0u : 0xffffffffu;     // (no branch around the load)
#pragma unroll
                for (int m = 0; m < MG; ++m) {
                    const float x = xr[off[(i >> 2) * MG + m]];
                    xv[i & 1][m] = masked ? __uint_as_float(__float_as_uint(x) & keep) : x;
                }
            };
            read(0);
#pragma unroll
            for (int i = 0; i < 4 * NG; ++i) {
                if (i + 1 < 4 * NG) read(i + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < MG; ++m)
                    t[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[i & 1][m], b[i & 3], i & 3 ? t[m] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                if ((i & 3) == 3) {
#pragma unroll
                    for (int m = 0; m < MG; ++m) acc[(i >> 2) * MG + m] += t[m];
                }
            }
        };
        for (int k = 0; k < whole; k += 16) sixteen(k, std::false_type{});
        for (int k = whole; k < mine; k += 16) sixteen(k, std::true_type{});
    }
    // the four waves' sums, added in wave order
    __syncthreads();
    float *const red = lds;
    double *const redb = reinterpret_cast<double *>(lds + MB * 256);
    for (int wv = 0; wv < kWaves; ++wv) {
        if (wave == wv) {
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float *r = red + (m * 4 + i) * 64 + lane;
                    *r = wv ? *r + acc[m][i] : acc[m][i];
                }
            redb[lane] = wv ? redb[lane] + bsum : bsum;
        }
        __syncthreads();
    }
    const size_t ndw = static_cast<size_t>(a.ntap) * a.cin * a.cout;
    float *const part = a.part + blockIdx.x * (ndw + a.cout);
    for (int e = tid; e < 16 * MB * 16; e += kThreads) {          // row-major: 16 output channels side by side
        const int row = e >> 4, cc = e & 15, t = static_cast<int>(fdiv(row, a.dkc)), c = c0 + row - t * a.kc;
        if (row < rows && c < a.cin && cob * 16 + cc < a.cout)
            part[(static_cast<size_t>(t) * a.cin + c) * a.cout + cob * 16 + cc] =
                red[((row >> 4) * 4 + (row & 3)) * 64 + ((row & 15) >> 2) * 16 + cc];
    }
    if (a.bias && chunk == 0 && tid < 16 && co < a.cout)
        part[ndw + co] = static_cast<float>((redb[tid] + redb[16 + tid]) + (redb[32 + tid] + redb[48 + tid]));
}

// Second stage: out[e] = sum over the partials in a fixed order (16 runs, then the runs in order), in fp64; a block serves 64
// neighbouring outputs, so every load of a wave is a whole 256-byte piece, and goes on to others where a launch of all of
// them would exceed the 2^32 threads of a grid (more than 9.9 million pairs of channels).
__global__ __launch_bounds__(1024) void reduce_runs_kernel(const float *__restrict__ part, float *__restrict__ dw,
                                                           float *__restrict__ db, int nparts, long long ndw, long long n) {
    __shared__ double red[16][64];
    const int l = threadIdx.x & 63, run = threadIdx.x >> 6;
    const int per = (nparts + 15) / 16, p1 = min(nparts, (run + 1) * per);
    for (long long e0 = 64LL * blockIdx.x; e0 < n; e0 += 64LL * gridDim.x) {
        const long long e = e0 + l;
        double s = 0.0;
        if (e < n) {
#pragma unroll 8
            for (int p = run * per; p < p1; ++p) s += part[p * n + e];
        }
        red[run][l] = s;
        __syncthreads();
        if (run == 0 && e < n) {
            double t = 0.0;
#pragma unroll
            for (int r = 0; r < 16; ++r) t += red[r][l];
            if (e < ndw) dw[e] = static_cast<float>(t);
            else if (db) db[e - ndw] = static_cast<float>(t);
        }
        __syncthreads();
    }
}

}  // namespace

// Stage 2 (shared with the MFMA weight-gradient kernel): out[e] = sum_s part[s][e] in order of s.
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float *__restrict__ part,
                                                              float *__restrict__ out, int nparts,
                                                              long long n) {
    const long long e = 1LL * blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    float s = 0.f;
    for (int p = 0; p < nparts; ++p) s += part[1LL * p * n + e];
    out[e] = s;
}

// Same sum for few outputs and many partials (one serial chain per output would be latency-bound): a block
// per output; thread t adds the partials t, t + 256, ... in order, then the 256 thread sums are combined
// by a fixed binary tree.  The grouping depends only on nparts, so the result is still reproducible.
__global__ __launch_bounds__(256) void reduce_partials_wide_kernel(const float *__restrict__ part,
                                                                   float *__restrict__ out, int nparts,
                                                                   long long n) {
    __shared__ float red[256];
    const long long e = blockIdx.x;
    float s = 0.f;
    for (int p = threadIdx.x; p < nparts; p += 256) s += part[1LL * p * n + e];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[e] = red[0];
}

int launch_reduce_partials(const float *part, float *out, int nparts, long long n, hipStream_t s) {
    if (nparts >= 32 && n <= 16384) {          // (a serial chain of 128 loads: about 60 us; a block per output: 4)
        hipLaunchKernelGGL(reduce_partials_wide_kernel, dim3(static_cast<unsigned>(n)), dim3(256), 0, s, part, out,
                           nparts, n);
        return record_hip(hipGetLastError());
    }
    dim3 grid(static_cast<unsigned>((n + 255) / 256)), block(256);
    hipLaunchKernelGGL(reduce_partials_kernel, grid, block, 0, s, part, out, nparts, n);
    return record_hip(hipGetLastError());
}


// Brick shape for an output box (ed, eh, ew): at most nvox voxels and max_rec staged records, such that covering the box
// costs least: an instruction slot per voxel of every brick, used or not, plus a share for every staged record.
static BrickGeo plan_brick(const Geo &g, int ed, int eh, int ew, int kd, int ks, int nvox, int max_rec) {
    BrickGeo best{};
    double cost = 0;
    // extents that cut n into equal parts: the largest such extent below e + 1
    auto even = [](int n, int e) { return e < 1 ? 0 : (n + (n + e - 1) / e - 1) / ((n + e - 1) / e); };
    for (int c = even(ew, ew < nvox ? ew : nvox); c > 0; c = even(ew, c - 1))
        for (int r = even(eh, eh < nvox / c ? eh : nvox / c); r > 0; r = even(eh, r - 1)) {
            int s = even(ed, ed < nvox / (c * r) ? ed : nvox / (c * r));
            while (s > 1 && (s + kd - 1) * (r + ks - 1) * (c + ks - 1) > max_rec) s = even(ed, s - 1);
            const int nrec = (s + kd - 1) * (r + ks - 1) * (c + ks - 1);
            if (nrec > max_rec) continue;
            const int nd = (ed + s - 1) / s, nh = (eh + r - 1) / r, nw = (ew + c - 1) / c;
            const double k = 1.0 * nd * nh * nw * (nvox + 0.15 * nrec);
            if (best.s == 0 || k < cost) {
                cost = k;
                best.s = s; best.r = r; best.c = c;
                best.ns = nd; best.nr = nh; best.nc = nw;
                best.nrec = nrec;
            }
        }
    best.kd = kd;
    best.ks = ks;
    best.nbricks = best.ns * best.nr * best.nc * g.ntiles;
    best.dvc = make_fastdiv(best.c);
    best.dvrc = make_fastdiv(best.r * best.c);
    best.drc = make_fastdiv(best.c + ks - 1);
    best.drrc = make_fastdiv((best.r + ks - 1) * (best.c + ks - 1));
    best.dnc = make_fastdiv(best.nc);
    best.dnr = make_fastdiv(best.nr);
    best.dns = make_fastdiv(best.ns);
    return best;
}

// Workgroups for n bricks when `most` fit the chip at a time: every one gets the same number of bricks.
static int even_share(int n, int most) {
    const int rounds = static_cast<int>((n + most - 1LL) / most);
    return static_cast<int>((n + rounds - 1LL) / rounds);
}

constexpr int kHalfLds = 80 * 1024;      // two workgroups per compute unit

// How a call is cut up, apart from the shape of its bricks: channels per chunk, chunks, K steps, blocks of 16 output channels,
// voxel segments per wave.  `vox`: voxels to compute.
struct ConvDirectPlan { int ntap, kc, nck, steps, ncg, nv; };
static ConvDirectPlan conv_direct_plan(double vox, int ntap, int ki, int ko) {
    ConvDirectPlan p;
    p.ntap = ntap;
    p.nck = (ki + 15) / 16;
    p.kc = ((ki + p.nck - 1) / p.nck + 3) / 4 * 4;
    p.nck = (ki + p.kc - 1) / p.kc;
    p.steps = (ntap * (p.kc / 4) + 3) / 4;
    p.ncg = (ko + 15) / 16;
    // 256 voxels per workgroup; fewer where that would leave the chip's 512 places (two per compute unit) empty
    p.nv = vox / 256 * p.ncg >= 512 ? 4 : (vox / 128 * p.ncg >= 512 ? 2 : 1);
    return p;
}

// Whether a thread per output is taken instead of bricks: unless bricks are estimated at less than 0.60 (extent 1) or 0.85
// (extent 3) of its time.  Estimates in microseconds, threads: launch + waves x (outputs, taps, products: the lines of x and w
// that a wave touches per channel) + the chain of a thread; bricks: launch + rounds of 512 workgroups x chunks x (staged quads,
// K steps).  Fitted to 1356 calls measured both ways (1 ... 128 channels, 9 voxels ... 5 million, 2-D and 3-D; 24 % and 11 %
// rms: hence the margins, with which four of them take more than 5 % longer than with a thread per output; without one 60 do).
// Measured, threads against bricks: 1x1x1 40 -> 3 on 44 x 32 x 44, bf16, 8 against 17 us, 4 -> 2 on 102 x 110 x 134 16 against 67,
// data gradient of 16 -> 128 on 90 x 96 x 68, fp32, 2122 against 149; 3x3x3 1 -> 3 on 84 x 131 x 138, bf16, 68 against 124, 8 ->
// 16 on 32^3, fp32, 44 against 11.  Only what does not depend on the tile grid and on the growth of the output box counts, so
// that a voxel is computed in one order of sums on all of them.
static bool prefer_threads(const Geo &g, int ki, int ko, sp_dtype_t dt, bool dgrad, int ks) {
    const double vox = 1.0 * g.ntiles * g.int_vox, es = static_cast<double>(elem_size(dt));
    const ConvDirectPlan p = conv_direct_plan(vox, (g.flat ? 1 : ks) * ks * ks, ki, ko);
    static const double c[2][13] = {{6.83, 0.110, 0.0375, 0.0073, 0.0027, 0.0016, 0.0268, 5.16, 1.35, 0.271, 0.592, 0.476, 2.64},
                                    {5.35, 0.000, 0.0144, 0.0105, 0.0019, 0.0015, 0.0536, 3.97, 1.13, 1.276, 3.205, 0.258, 0.574}};
    const double *k = c[ks == 3];
    const auto most = [](double a, double b) { return a > b ? a : b; };
    const double row = ki * es < 64 ? ki * es / 64 : 1, lanes = ko < 64 ? ko : 64;      // lines of a record; output channels of a wave
    const double xl = most(1, 64 / lanes * row), wl = most(1, lanes * (dgrad ? row : es / 64));
    const double threads = k[0] + vox * ko / 64e3 * (k[1] + k[2] * p.ntap + p.ntap * ki * (k[3] + k[4] * xl + k[5] * wl)) + k[6] * p.ntap * ki;
    const double surround = ks == 1 ? 1.0 : (g.flat ? 1.9 : 3.0);                       // staged records per voxel
    const double quads = 64e-3 * p.nv * surround * (ki % 4 ? p.kc * k[11] : p.kc / 4);
    const double places = p.ncg < 512 ? 512 / p.ncg : 1, wgs = vox / (64 * p.nv);
    const double rounds = wgs <= places ? 1 : static_cast<double>(static_cast<long long>((wgs + places - 1) / places));
    const double bricks = k[7] + rounds * (k[8] + p.nck * (k[9] + k[10] * quads + k[12] * p.steps * p.nv / 4));
    return !(bricks < (ks == 1 ? 0.60 : 0.85) * threads);
}

int conv_direct_route(const Geo &g, int ki, int ko, sp_dtype_t dt, bool dgrad, int ks) {
    return prefer_threads(g, ki, ko, dt, dgrad, ks) ? kRouteThreads : kRouteBricks;
}

static int launch_conv_threads(const void *Pin, const void *w, const float *bias, void *Pout, const Geo &g, int ki, int ko,
                               sp_dtype_t dt, bool relu, bool dgrad, hipStream_t s, int ks, const void *mask, long long total) {
    const dim3 grid(static_cast<unsigned>((total + kThreads - 1) / kThreads)), block(kThreads);
    const auto launch = [&](auto kern, auto e) {
        typedef decltype(e) E;
        hipLaunchKernelGGL(kern, grid, block, 0, s, static_cast<const E *>(Pin), static_cast<const E *>(w), bias,
                           static_cast<E *>(Pout), g, ki, ko, relu ? 1 : 0, total, static_cast<const E *>(mask));
        return record_hip(hipGetLastError());
    };
    const uint16_t h = 0;
    if (dt == SP_BF16)
        return ks == 1 ? (dgrad ? launch(conv_threads_kernel<uint16_t, true, 1>, h) : launch(conv_threads_kernel<uint16_t, false, 1>, h))
                       : (dgrad ? launch(conv_threads_kernel<uint16_t, true, 3>, h) : launch(conv_threads_kernel<uint16_t, false, 3>, h));
    return ks == 1 ? (dgrad ? launch(conv_threads_kernel<float, true, 1>, 0.f) : launch(conv_threads_kernel<float, false, 1>, 0.f))
                   : (dgrad ? launch(conv_threads_kernel<float, true, 3>, 0.f) : launch(conv_threads_kernel<float, false, 3>, 0.f));
}

int launch_conv_direct(const void *Pin, const void *w, const float *bias, void *Pout, const Geo &g,
                       int ki, int ko, sp_dtype_t dt, bool relu, bool dgrad, hipStream_t s, int ks,
                       const void *mask) {
    const int kd = g.flat ? 1 : ks;
    const int ed = g.td + 2 * grow_d(g), eh = g.th + 2 * g.grow, ew = g.tw + 2 * g.grow;
    const double vox = 1.0 * g.ntiles * ed * eh * ew;
    if (vox / 16 > 0x7fffffff) return SP_EGEOM;
    if (prefer_threads(g, ki, ko, dt, dgrad, ks) && vox * ko < 0xffffff00u)              // (a launch has less than 2^32 threads)
        return launch_conv_threads(Pin, w, bias, Pout, g, ki, ko, dt, relu, dgrad, s, ks, mask, 1LL * g.ntiles * ed * eh * ew * ko);
    const ConvDirectPlan p = conv_direct_plan(vox, kd * ks * ks, ki, ko);
    ConvDirectArgs a;
    a.in = Pin; a.w = w; a.bias = bias; a.out = Pout; a.mask = mask;
    a.g = g;
    a.ki = ki; a.ko = ko;
    a.ntap = p.ntap;
    a.kc = p.kc; a.nck = p.nck;
    a.stride = (a.kc / 4) % 2 ? a.kc : a.kc + 4;
    a.steps = p.steps;
    a.dgrad = dgrad; a.relu = relu;
    a.dq = make_fastdiv(a.kc / 4);
    const int ncg = p.ncg, nv = p.nv;
    const int fixed = a.steps * (1024 + 16);
    a.b = plan_brick(g, ed, eh, ew, kd, ks, 64 * nv, (kHalfLds - fixed) / (4 * a.stride));
    const size_t lds = fixed + 4u * a.b.nrec * a.stride;
    int most = 512 / ncg;
    if (most < 1) most = 1;
    const dim3 grid(even_share(a.b.nbricks, most), ncg), block(kThreads);
    using Kern = void (*)(ConvDirectArgs);
    static const Kern kern[2][3] = {{conv_direct_kernel<float, 1>, conv_direct_kernel<float, 2>, conv_direct_kernel<float, 4>},
                                    {conv_direct_kernel<uint16_t, 1>, conv_direct_kernel<uint16_t, 2>, conv_direct_kernel<uint16_t, 4>}};
    static const hipError_t attr = [] {
        for (int i = 0; i < 6; ++i) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern[i / 3][i % 3]),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kHalfLds);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (attr != hipSuccess) return record_hip(attr);
    hipLaunchKernelGGL(kern[dt == SP_BF16][nv == 4 ? 2 : nv - 1], grid, block, lds, s, a);
    return record_hip(hipGetLastError());
}

int launch_reduce_runs(const float *part, float *dw, float *db, int nparts, long long ndw, long long n, hipStream_t s) {
    const long long blocks = (n + 63) / 64;
    hipLaunchKernelGGL(reduce_runs_kernel, dim3(static_cast<unsigned>(blocks < (1 << 20) ? blocks : 1 << 20)), dim3(1024), 0, s,
                       part, dw, db, nparts, ndw, n);
    return record_hip(hipGetLastError());
}

// How the weight gradient is cut up: channels per chunk, row blocks, bricks, workgroups per channel-block pair.
struct WgradDirectPlan { int kc, nck, nco, ntap, kd, nparts, share; BrickGeo b; };
static WgradDirectPlan wgrad_direct_plan(const Geo &g, int cin, int cout, int ks) {
    WgradDirectPlan p;
    p.kd = g.flat ? 1 : ks;
    p.ntap = p.kd * ks * ks;
    p.nck = (cin + 15) / 16;
    p.kc = (cin + p.nck - 1) / p.nck;
    if (cin % 4 == 0) p.kc = (p.kc + 3) / 4 * 4;                  // keep the 16-byte staging loads
    p.nck = (cin + p.kc - 1) / p.kc;
    p.nco = (cout + 15) / 16;
    const int fixed = kWgradVox * (16 + 1) * 4 + 16, pairs = p.nck * p.nco;
    // fewer voxels per brick where full ones would leave compute units without a workgroup: a wave of a full brick has 432
    // instructions of 32 cycles one after the other (16 -> 3 on 7 x 6 x 5 28.9 -> 19.7 us, one thread per product before 16.3;
    // 17 -> 4 on 7 x 9 x 14 40 -> 20, before 21)
    int vox = kWgradVox;
    while (vox > 64 && 1.0 * g.ntiles * g.int_vox / vox * pairs < 256) vox /= 2;
    p.share = vox / kWaves;
    p.b = plan_brick(g, g.td, g.th, g.tw, p.kd, ks, vox, (kHalfLds - fixed) / (4 * p.kc));
    // two workgroups per compute unit, shared out over the channel-block pairs
    int most = 512 / pairs;
    if (most < 1) most = 1;
    p.nparts = even_share(p.b.nbricks, most);
    return p;
}

size_t wgrad_direct_ws_bytes(const Geo &g, int cin, int cout, int ks) {
    const WgradDirectPlan p = wgrad_direct_plan(g, cin, cout, ks);
    return p.nparts * (static_cast<size_t>(p.ntap) * cin * cout + cout) * sizeof(float);
}

int launch_wgrad_direct(const void *Px, const void *Pdz, float *dw, float *db, const Geo &g, int cin,
                        int cout, sp_dtype_t dt, void *ws, hipStream_t s, int ks) {
    const WgradDirectPlan p = wgrad_direct_plan(g, cin, cout, ks);
    WgradDirectArgs a;
    a.x = Px; a.dz = Pdz;
    a.part = static_cast<float *>(ws);
    a.g = g;
    a.g.grow = 0;
    a.b = p.b;
    a.cin = cin; a.cout = cout; a.ntap = p.ntap;
    a.kc = p.kc; a.bias = db != nullptr;
    a.share = p.share;
    a.dq = make_fastdiv((p.kc + 3) / 4);
    a.dkc = make_fastdiv(p.kc);
    using Kern = void (*)(WgradDirectArgs);
    constexpr int kSizes = 6;
    static const int mbs[kSizes] = {1, 2, 7, 9, 14, 27};          // row blocks of the kernels that exist
    static const Kern kern[2][kSizes] = {
        {wgrad_direct_kernel<float, 1>, wgrad_direct_kernel<float, 2>, wgrad_direct_kernel<float, 7>,
         wgrad_direct_kernel<float, 9>, wgrad_direct_kernel<float, 14>, wgrad_direct_kernel<float, 27>},
        {wgrad_direct_kernel<uint16_t, 1>, wgrad_direct_kernel<uint16_t, 2>, wgrad_direct_kernel<uint16_t, 7>,
         wgrad_direct_kernel<uint16_t, 9>, wgrad_direct_kernel<uint16_t, 14>, wgrad_direct_kernel<uint16_t, 27>}};
    static const hipError_t attr = [] {
        for (int i = 0; i < 2 * kSizes; ++i) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern[i / kSizes][i % kSizes]),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, kHalfLds);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }();
    if (attr != hipSuccess) return record_hip(attr);
    int k = 0;
    while (16 * mbs[k] < p.ntap * p.kc) ++k;                       // (ntap * kc <= 27 * 16)
    size_t lds = kWgradVox * 16 * 4 + (static_cast<size_t>(p.b.nrec) * p.kc + 3) / 4 * 16 + kWgradVox * 4;
    const size_t red = mbs[k] * 256 * sizeof(float) + 64 * sizeof(double);        // the sums of the waves reuse the staging area
    if (lds < red) lds = red;
    hipLaunchKernelGGL(kern[dt == SP_BF16][k], dim3(p.nparts, p.nco, p.nck), dim3(kThreads), lds, s, a);
    int rc = record_hip(hipGetLastError());
    if (rc != SP_OK) return rc;
    const long long ndw = 1LL * p.ntap * cin * cout, n = ndw + cout;
    return launch_reduce_runs(a.part, dw, db, p.nparts, ndw, n, s);
}

}  // namespace sp3d
