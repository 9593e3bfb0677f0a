// Register-resident shared MLP for narrow fp32 layers on many rows, gfx950.
//
// The per-point MLP F (Sec. 4: with delayed aggregation it runs once per
// input point) on layers of at most 128 channels, e.g. the last feature
// propagation level and the per-point head of the segmentation network
// (65536 rows), where a layer-by-layer GEMM writes and re-reads every
// intermediate activation and stages it through LDS.
//
// Each wave pushes 32-row tiles through every layer on its own.  The
// product is taken transposed, Y^T = W X^T, on MFMAs of 32 x 32 outputs: the
// weights are the A operand (32 output channels) and the activations the B
// operand (32 rows), so a lane's 16 accumulators of a 32-channel block hold
// 16 output channels of ONE row, its lane % 32 (channel 8(r/4) + 4(lane/32)
// + r%4 of register r).  An MFMA sums over whatever k order its two operands
// share, so the next layer takes its k steps in exactly that register order:
// step (j, r) is the k pair {32j + 8(r/4) + r%4, +4}, lane half h supplying
// its own accumulator r of block j.  The activations never leave registers
// between layers: no LDS round trip, no barrier, no transpose.  The weights,
// permuted once per workgroup into each layer's k order, are the only LDS
// data: a workgroup is persistent, its eight waves stream tiles.
//
// The fp32 matrix instruction bounded this kernel (65536 x 131 -> 128 -> 128
// -> 128: 41 of 77 us; it runs at a sixteenth of the bf16 rate).  So every
// fp32 value is taken as the exact sum of three bf16 values (24 = 3 x 8 bits
// of mantissa, each part rounded to nearest) and a product as the six largest
// of its nine partial products, on v_mfma_f32_32x32x16_bf16 with fp32 sums:
// eight k steps of a lane half make one of these instructions.
// The three products left out are below 2^-24 of the product together (0.99
// of that at w = x = 1 + 2^-8 - 2^-17): as much as the rounding of an fp32
// product, which this form has besides.  It makes up for that with fewer
// roundings of large sums (one per 16 k instead of eight).  2-norm error
// against 64 bits, here and with the fp32 instruction: 16, 64 and 128 normal
// values a row 3.4e-8, 4.6e-8, 6.2e-8 and 7.3e-8, 1.4e-7, 2.0e-7; half of them
// 0: 3.3e-8, 4.1e-8, 5.1e-8 and 5.5e-8, 1.1e-7, 1.5e-7; but rows with a single
// value that is not 0: 3.5e-8 and 2.5e-8 (at most 2.7 and 1.0 times 2^-24 of
// it).  With two more of the partial products these last figures are 3.4e-8
// and 2.0, and the kernel takes 6 to 15 % longer.
// The parts of huge values would overflow, those of infinities would be NaN
// and those of very small ones denormal, and products that overflow would
// meet others of the opposite sign.  So the weights and each row's largest
// value are tested against a range in which none of this occurs (kRrSmall).
// Weights with one outside it are staged again as fp32 and multiplied by
// v_mfma_f32_32x32x2_f32; so are the rows of a tile with one outside it, by
// the weights' parts put together again (rr_products_plain).
// Measured: 524288 gathered rows 3 -> 64 -> 64 -> 128, pooled: 128 -> 103 us;
// 65536 x 131 -> 128 -> 128 -> 128: 77 -> 57 us with its launch.  What bounds
// it now is the split (44 vector instructions per 16 k of a row) and the LDS
// reads of the weights, not yet the matrix cores (33 and 16 us).
// The first layer reads its rows straight from memory, the two lanes of a
// row taking alternate 4-channel chunks.  Its input may have two parts: a
// wide source of whole aligned 4-channel chunks, and a narrow one of at most
// 8 channels (the xyz of a module's first layer, the skip features of the
// finest propagation level), which makes one more group of four k steps.
//
// Neighbor rows [xyz_j - cxyz_c | feat_j] of the conventional module are
// gathered by the same loader, and the max over a centroid's K rows is taken
// in registers: with K = 32 a tile is one centroid, with K = 16 two, and a
// lane's accumulators are reduced over the lanes of its half wave (16), so
// the rows' outputs are neither stored nor cleared beforehand.
#include <algorithm>
#include <array>

#include "common.h"
#include "mlp_internal.h"

namespace meso {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kRrWaves = 8;          // waves per workgroup (two per SIMD)
constexpr int kRrMaxWidth = 128;     // widest layer input or output
constexpr int kRrMaxSteps = 64;      // k steps of a layer (128 inputs / 2)
constexpr int kRrMaxLds = 160 * 1024;
// The split takes weights that are 0 or in [2^-50, 2^20) and a row whose
// largest value is 0 or in [2^-50, 2^96), so that every product, part and sum
// of 136 is finite.  (A value below 2^-103 beside larger ones of its row has
// parts that are not normal: an output is off by less than 2^-97 by it.)
constexpr float kRrSmall = 0x1p-50f, kRrMaxW = 0x1p20f, kRrMaxX = 0x1p96f;

struct RrArgs {
    const float* x0;
    int64_t ld0;
    const float* x1;
    int64_t ld1;
    int c0, c1;
    int64_t rows;
    int64_t tiles;
    int n_layers;
    int dims[MESORASI_MAX_LAYERS + 1];
    const float* W[MESORASI_MAX_LAYERS];
    const float* bias[MESORASI_MAX_LAYERS];
    int woff[MESORASI_MAX_LAYERS];   // float offset of layer l's permuted weights in LDS
    int boff[MESORASI_MAX_LAYERS];   // float offset of its padded bias
    int foff;                        // int offset of the waves' flags (a weight outside the split's range)
    // weights staged in phases when all layers do not fit at once: phase p
    // holds layers phase_first[p] .. phase_first[p + 1] - 1 (offsets above
    // relative to the phase)
    int nphase;
    int phase_first[MESORASI_MAX_LAYERS + 1];
    uint32_t relu_mask;
    float* y;
    int64_t ldy;
    int k0h;     // layer-0 k values per lane half of the wide source (a multiple of 16, at most 64)
    int vec0;    // wide layer-0 rows read as aligned float4
    int cs;      // channels of the narrow source (0: none), at weight column sw; the wide source's are at ww
    int sw, ww;
    const float* xs;
    int64_t lds;
    int cs0;     // of them the first cs0 from xs, the others from xs1
    const float* xs1;
    int64_t lds1;
    int vecy;    // output rows stored as aligned float4
    MlpGather g; // neighbor rows (xs, x0 = xyz, feat), pooled over g.k
    // interpolated first-layer rows (instead of [x0 | x1]): row r = b Nd + i
    // is phi(sum_k u_k g[b, nn[r, k]] + add[r]) over the first dims[0]
    // channels, u_k the normalised inverse squared distances
    int interp;
    RrInterp ip;
};

__host__ __device__ inline int rr_blocks(int n) { return (n + 31) / 32; }
// bf16 steps (of 16 k) of layer l: 2 per 32-channel input block; the first
// layer's wide source is padded to whole blocks too (k0h = 16 nj k per lane
// half).
__host__ __device__ inline int rr_steps(const int* dims, int l, int k0h) {
    return l == 0 ? k0h / 8 : 2 * rr_blocks(dims[l]);
}
// LDS floats of layer l: the narrow source's weights as fp32 (64 lanes x 4
// per output block), the others as three bf16 parts, the bias.
__host__ __device__ inline int rr_narrow_floats(int nob, int l, int cs) { return l == 0 && cs > 0 ? nob * 256 : 0; }
inline int rr_floats(const int* dims, int l, int k0h, int cs) {
    const int nob = rr_blocks(dims[l + 1]);
    return rr_narrow_floats(nob, l, cs) + nob * rr_steps(dims, l, k0h) * 3 * 256 + nob * 32;
}

// The input channel that lane half h supplies at k step s of layer l.
__device__ __forceinline__ int rr_k(int l, int s, int h) {
    // first layer: the two lanes of a row take alternate 4-channel chunks,
    // so a row's 128-byte line is read whole by four consecutive loads
    if (l == 0) return 8 * (s >> 2) + 4 * h + (s & 3);
    const int j = s >> 4, r = s & 15;
    return 32 * j + 8 * (r >> 2) + (r & 3) + 4 * h;
}

// Two floats to bf16, round to nearest even, the first in the low half.
__device__ __forceinline__ uint32_t rr_pack(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float rr_low(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float rr_high(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Pins eight values to this point of the program: what is computed from them
// is computed here, not for all steps at once ahead of the products (which
// spilled more registers than the products use).
__device__ __forceinline__ void rr_here(float* v) {
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]));
}

// Eight floats as three vectors of bf16 parts, p[0] + p[1] + p[2] = v.
__device__ __forceinline__ void rr_split(const float* v, uint4 (&p)[3]) {
    uint32_t w[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x = v[2 * i], y = v[2 * i + 1];
        w[0][i] = rr_pack(x, y);
        x -= rr_low(w[0][i]);
        y -= rr_high(w[0][i]);
        w[1][i] = rr_pack(x, y);
        x -= rr_low(w[1][i]);
        y -= rr_high(w[1][i]);
        w[2][i] = rr_pack(x, y);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) p[q] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
}

__device__ __forceinline__ bf16x8 rr_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// A step's weights of two output blocks (the second clamped to the first where
// there is none).
__device__ __forceinline__ void rr_weights(const uint4* __restrict__ wl, int stride, uint4 (&w)[2][3]) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int q = 0; q < 3; ++q) w[b][q] = wl[b * stride + q * 64];
}

// A step's five small partial products on NB output blocks, whose
// accumulation chains interleave.
template <int NB>
__device__ __forceinline__ void rr_small(const uint4 (&w)[2][3], const uint4 (&x)[3], f32x16* __restrict__ acc) {
    constexpr int pw[5] = {2, 0, 1, 1, 0}, px[5] = {0, 2, 1, 0, 1};
#pragma unroll
    for (int m = 0; m < 5; ++m)
#pragma unroll
        for (int b = 0; b < NB; ++b)
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rr_bf16x8(w[b][pw[m]]), rr_bf16x8(x[px[m]]), acc[b], 0, 0,
                                                             0);
    __builtin_amdgcn_sched_barrier(0);
}

// One layer's products: nt steps, nob output blocks, taken in pairs.  All the
// small partial products are summed first and the large ones after them, so
// that only one rounding per 16 k is a rounding of a large sum.  A pair's
// weights are requested ahead of the split of its activations or of the other
// pair's products.  (The steps and blocks are guarded, not switched over: one
// instance is in the kernel, and the activations keep their registers around
// it; sixteen instances spilled 200 to 800 of them, this one 4 and 16 in the
// unphased forms and 23 and 30 in the phased ones.)
__device__ __forceinline__ void rr_products(int nt, int nob, const uint4* __restrict__ wl, float (&act)[kRrMaxSteps],
                                            f32x16 (&acc)[kRrMaxWidth / 32]) {
    static_assert(kRrMaxWidth == 128, "two pairs of output blocks");
    const int stride = nt * 3 * 64;
#pragma unroll
    for (int t = 0; t < kRrMaxSteps / 8; ++t) {
        if (t < nt) {
            const uint4* wt = wl + t * 3 * 64;
            uint4 w0[2][3], x[3];
            rr_weights(wt, nob > 1 ? stride : 0, w0);
            __builtin_amdgcn_sched_barrier(0);
            rr_here(&act[8 * t]);
            rr_split(&act[8 * t], x);
            if (nob > 2) {
                uint4 w1[2][3];
                rr_weights(wt + 2 * stride, nob > 3 ? stride : 0, w1);
                __builtin_amdgcn_sched_barrier(0);
                rr_small<2>(w0, x, &acc[0]);
                if (nob > 3) rr_small<2>(w1, x, &acc[2]);
                else rr_small<1>(w1, x, &acc[2]);
            } else {
                __builtin_amdgcn_sched_barrier(0);
                if (nob > 1) rr_small<2>(w0, x, &acc[0]);
                else rr_small<1>(w0, x, &acc[0]);
            }
        }
    }
    uint4 v[kRrMaxWidth / 32];
#pragma unroll
    for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) v[ob] = wl[(ob < nob ? ob : 0) * stride];
#pragma unroll
    for (int t = 0; t < kRrMaxSteps / 8; ++t) {
        if (t < nt) {
            uint4 vn[kRrMaxWidth / 32];
            const uint4* wt = wl + (t + 1 < nt ? t + 1 : t) * 3 * 64;
#pragma unroll
            for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) vn[ob] = wt[(ob < nob ? ob : 0) * stride];
            rr_here(&act[8 * t]);   // (rounded again, not held in registers since the first loop)
            const float* z = &act[8 * t];
            const uint4 x0 = make_uint4(rr_pack(z[0], z[1]), rr_pack(z[2], z[3]), rr_pack(z[4], z[5]),
                                        rr_pack(z[6], z[7]));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ob = 0; ob < kRrMaxWidth / 32; ++ob)
                if (ob < nob)
                    acc[ob] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rr_bf16x8(v[ob]), rr_bf16x8(x0), acc[ob], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) v[ob] = vn[ob];
        }
    }
}

// The same products on the fp32 instruction, the weights staged as fp32: two
// float4 (8 k) per lane and step.
__device__ __forceinline__ void rr_products_f32_any(int nt, int nob, const float4* __restrict__ wl,
                                                    const float (&act)[kRrMaxSteps], f32x16 (&acc)[kRrMaxWidth / 32]) {
#pragma unroll
    for (int t = 0; t < kRrMaxSteps / 8; ++t) {
        if (t < nt) {
#pragma unroll
            for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) {
                if (ob < nob) {
                    const float4 u = wl[(ob * nt + t) * 128], v = wl[(ob * nt + t) * 128 + 64];
                    const float w[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[e], act[8 * t + e], acc[ob], 0, 0, 0);
                }
            }
        }
    }
}

// The same on the weights' parts, for rows outside the range of rr_split.
__device__ __forceinline__ void rr_products_plain(int nt, int nob, const uint4* __restrict__ wl,
                                                  const float (&act)[kRrMaxSteps], f32x16 (&acc)[kRrMaxWidth / 32]) {
#pragma unroll
    for (int t = 0; t < kRrMaxSteps / 8; ++t) {
        if (t < nt) {
#pragma unroll
            for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) {
                if (ob < nob) {
                    const uint32_t* p = reinterpret_cast<const uint32_t*>(wl + (ob * nt + t) * 3 * 64);
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const uint32_t a0 = p[e >> 1], a1 = p[256 + (e >> 1)], a2 = p[512 + (e >> 1)];
                        const float w = e & 1 ? rr_high(a0) + (rr_high(a1) + rr_high(a2))
                                              : rr_low(a0) + (rr_low(a1) + rr_low(a2));
                        acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, act[8 * t + e], acc[ob], 0, 0, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
}

// The narrow source's four steps.
__device__ __forceinline__ void rr_narrow(int nob, const float4* __restrict__ wl, const float (&sm)[4],
                                          f32x16 (&acc)[kRrMaxWidth / 32]) {
#pragma unroll
    for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) {
        if (ob < nob) {
            const float4 w = wl[ob * 64];
            acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.x, sm[0], acc[ob], 0, 0, 0);
            acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.y, sm[1], acc[ob], 0, 0, 0);
            acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.z, sm[2], acc[ob], 0, 0, 0);
            acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w.w, sm[3], acc[ob], 0, 0, 0);
        }
    }
}

// ReLU in one instruction (a NaN gives 0, as a comparison with 0 does).
__device__ __forceinline__ float rr_relu(float v) {
    float r;
    asm("v_max_f32 %0, 0, %1" : "=v"(r) : "v"(v));
    return r;
}

// One tile's layer-0 input but for a narrow source: the lane's row, step s
// taking channel kb + 8 (s / 4) + s % 4.
__device__ __forceinline__ void rr_load_rows(const RrArgs& a, int64_t row, bool rok, int kb,
                                             float (&dst)[kRrMaxSteps]) {
            if (a.interp) {
                // the interpolation of mesorasi_interpolate3_add, in its fp32
                // operations, then the addition and phi
                const RrInterp& q = a.ip;
                const int64_t r0 = rok ? row : 0;
                const int64_t b = r0 / q.nd;
                const float w0 = 1.0f / fmaxf(q.dist[r0 * 3 + 0], 1e-10f);
                const float w1 = 1.0f / fmaxf(q.dist[r0 * 3 + 1], 1e-10f);
                const float w2 = 1.0f / fmaxf(q.dist[r0 * 3 + 2], 1e-10f);
                const float ws = w0 + w1 + w2;
                const float u0 = w0 / ws, u1 = w1 / ws, u2 = w2 / ws;
                const float* gs = q.g + b * q.ns * q.ldg;
                const float* g0 = gs + (int64_t)q.nit[r0 * 3 + 0] * q.ldg;
                const float* g1 = gs + (int64_t)q.nit[r0 * 3 + 1] * q.ldg;
                const float* g2 = gs + (int64_t)q.nit[r0 * 3 + 2] * q.ldg;
                const float* ad = q.add + r0 * q.lda;
    #pragma unroll
                for (int i = 0; i < kRrMaxSteps / 4; ++i) {
                    if (4 * i < a.k0h) {
                        const int k = kb + 8 * i;
                        const bool ok = rok && k < a.c0;
                        const int kk = ok ? k : 0;
                        const float4 x0 = *reinterpret_cast<const float4*>(g0 + kk);
                        const float4 x1 = *reinterpret_cast<const float4*>(g1 + kk);
                        const float4 x2 = *reinterpret_cast<const float4*>(g2 + kk);
                        const float4 p = *reinterpret_cast<const float4*>(ad + kk);
                        float v[4] = {u0 * x0.x + u1 * x1.x + u2 * x2.x, u0 * x0.y + u1 * x1.y + u2 * x2.y,
                                      u0 * x0.z + u1 * x1.z + u2 * x2.z, u0 * x0.w + u1 * x1.w + u2 * x2.w};
                        v[0] += p.x;
                        v[1] += p.y;
                        v[2] += p.z;
                        v[3] += p.w;
    #pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (q.relu) v[e] = v[e] > 0.0f ? v[e] : 0.0f;
                            dst[4 * i + e] = ok ? v[e] : 0.0f;
                        }
                    }
                }
            } else if (a.vec0) {
                const float* src = a.x0 + (rok ? row : 0) * a.ld0;
    #pragma unroll
                for (int i = 0; i < kRrMaxSteps / 4; ++i) {
                    if (4 * i < a.k0h) {
                        const int k = kb + 8 * i;
                        const bool ok = rok && k < a.c0;
                        const float4 v = *reinterpret_cast<const float4*>(src + (ok ? k : 0));
                        dst[4 * i + 0] = ok ? v.x : 0.0f;
                        dst[4 * i + 1] = ok ? v.y : 0.0f;
                        dst[4 * i + 2] = ok ? v.z : 0.0f;
                        dst[4 * i + 3] = ok ? v.w : 0.0f;
                    }
                }
            } else {
                // [x0 | x1] element by element from clamped, in-bounds addresses
                const int64_t r0 = rok ? row : 0;
                const float* src0 = a.x0 + r0 * a.ld0;
                const float* src1 = a.c1 > 0 ? a.x1 + r0 * a.ld1 : src0;
    #pragma unroll
                for (int i = 0; i < kRrMaxSteps; ++i) {
                    if (i < a.k0h) {
                        const int k = kb + 8 * (i >> 2) + (i & 3);
                        const bool in0 = k < a.c0, in1 = !in0 && k < a.c0 + a.c1;
                        const float v = in0 ? src0[k] : (in1 ? src1[k - a.c0] : src0[0]);
                        dst[i] = (rok && (in0 || in1)) ? v : 0.0f;
                    }
                }
            }
}

// Eight waves, two per SIMD: while one wave waits on its rows or runs its
// epilogue, the other keeps the SIMD's MFMA pipe busy.  (A four-wave form
// with 512 registers per wave that requested its next tile's rows before
// computing the current one measured 9-18 % slower.)
// PHASED: the weights staged in phases.  POOLED: gathered neighbor rows, the
// output their max per centroid.
template <bool PHASED, bool POOLED>
__global__ __launch_bounds__(64 * kRrWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void mlp_rr_kernel(RrArgs a) {
    extern __shared__ float4 smem4[];
    float* smem = reinterpret_cast<float*>(smem4);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hk = lane >> 5;

    float act[kRrMaxSteps], sm[4];
    // layer-0 input of tile t: this lane's row; step s takes channel
    // 8 (s / 4) + 4 hk + s % 4
    auto load_tile = [&](int64_t t, float (&dst)[kRrMaxSteps]) {
        const int64_t row = t * 32 + (lane & 31);
        const bool rok = row < a.rows;
        // (opaque per tile: the per-element bounds below are cheap to
        // recompute, while hoisting them out of the tile loop would hold
        // some hundred registers for its whole length)
        int kb = 4 * hk;
        asm volatile("" : "+v"(kb));
        if constexpr (POOLED) {
            const int64_t r0 = rok ? row : 0;
            const int64_t cloud = (int64_t)((uint64_t)r0 / (uint64_t)a.g.mk);
            const int64_t j = cloud * a.g.n + a.g.nit[r0];
            const float* pj = a.xs + j * 3;
            const float* pc = a.g.cxyz + (int64_t)((uint64_t)r0 / (uint32_t)a.g.k) * 3;
            const bool ok = rok && hk == 0;
            sm[0] = ok ? pj[0] - pc[0] : 0.0f;
            sm[1] = ok ? pj[1] - pc[1] : 0.0f;
            sm[2] = ok ? pj[2] - pc[2] : 0.0f;
            sm[3] = 0.0f;
            const float* src = a.x0 + j * a.ld0;
#pragma unroll
            for (int i = 0; i < kRrMaxSteps / 4; ++i) {
                if (4 * i < a.k0h) {
                    const int k = kb + 8 * i;
                    const bool in = rok && k < a.c0;
                    const float4 v = *reinterpret_cast<const float4*>(src + (in ? k : 0));
                    dst[4 * i + 0] = in ? v.x : 0.0f;
                    dst[4 * i + 1] = in ? v.y : 0.0f;
                    dst[4 * i + 2] = in ? v.z : 0.0f;
                    dst[4 * i + 3] = in ? v.w : 0.0f;
                }
            }
            return;
        }
        if (a.cs > 0) {
            const float* xr = a.xs + (rok ? row : 0) * a.lds;
            const float* xq = a.cs0 < a.cs ? a.xs1 + (rok ? row : 0) * a.lds1 - a.cs0 : xr;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = 4 * hk + e;
                const float v = k < a.cs0 || k >= a.cs ? xr[k < a.cs0 ? k : 0] : xq[k];
                sm[e] = rok && k < a.cs ? v : 0.0f;
            }
        }
        rr_load_rows(a, row, rok, kb, dst);
    };

    // the first tile's rows are requested before the weights are staged,
    // so their HBM round trip overlaps the staging
    const int64_t stride = (int64_t)gridDim.x * kRrWaves;
    // interpolated rows gather the coarse level's rows of their cloud:
    // workgroups are dealt to the 8 XCDs round-robin by id, so (the grid
    // being a multiple of 8 then) renumber them to give each XCD one
    // contiguous range of tiles -- whole clouds -- and keep those gathers in
    // its own L2
    int64_t wg = blockIdx.x;
    if ((POOLED || a.interp) && (gridDim.x & 7) == 0)
        wg = (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int64_t t0 = wg * kRrWaves + wave;
    if (t0 < a.tiles) load_tile(t0, act);

    // weights: layer l, output block ob, step t, part, lane: thread tid takes
    // (ob, t, lane) items tid + 512 u (at most 4 blocks x 8 steps x 64
    // lanes), the 8 consecutive k steps of one weight row, two items'
    // loads in flight before their LDS stores.  Each wave leaves a flag: a
    // weight is outside the range of the split.
    constexpr int kPer = 2;   // items per thread in flight
    auto stage = [&](int l0, int l1, bool plain) {
        bool outside = false;
        for (int l = l0; l < l1; ++l) {
            const int K = a.dims[l], N = a.dims[l + 1], nob = rr_blocks(N);
            const int nt = rr_steps(a.dims, l, a.k0h);
            const int total = nob * nt * 64;
            const unsigned inv = nt > 0 ? (65536u + nt - 1) / nt : 0u;   // gg / nt exactly for gg < 128
            const float* __restrict__ W = a.W[l];
            // columns [base, end): a layer's inputs, or the first layer's
            // wide source
            const int base = l == 0 && a.cs > 0 ? a.ww : 0, end = l == 0 && a.cs > 0 ? base + K - a.cs : K;
            float4* dn = smem4 + (a.woff[l] >> 2);
            if (l == 0 && a.cs > 0 && tid < nob * 64) {
                const int n = (tid >> 6) * 32 + (lane & 31), k = 4 * hk;
                const float* wr = W + (int64_t)(n < N ? n : 0) * K + a.sw;
                float q[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) q[e] = n < N && k + e < a.cs ? wr[k + e] : 0.0f;
                dn[tid] = make_float4(q[0], q[1], q[2], q[3]);
            }
            dn += rr_narrow_floats(nob, l, a.cs) / 4;
            uint4* dst = reinterpret_cast<uint4*>(dn);
            for (int i0 = tid; i0 < total + tid; i0 += 64 * kRrWaves * kPer) {
                float v[kPer][8];
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const int i = i0 + 64 * kRrWaves * u;
                    const int ln = i & 63, gg = i >> 6;
                    const int ob = (int)(((unsigned)gg * inv) >> 16), t = gg - ob * nt;
                    const int n = ob * 32 + (ln & 31);
                    const float* wr = W + (int64_t)n * K;
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int k = base + rr_k(l, 8 * t + 4 * c, ln >> 5);
                        float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (i < total && n < N) {
                            if (k + 4 <= end) {
                                // (global loads of 16 bytes take any 4-byte alignment)
                                struct __attribute__((packed, aligned(4))) F4 { float x, y, z, w; };
                                const F4 p = *reinterpret_cast<const F4*>(wr + k);
                                q = make_float4(p.x, p.y, p.z, p.w);
                            } else {
                                q.x = k + 0 < end ? wr[k + 0] : 0.0f;
                                q.y = k + 1 < end ? wr[k + 1] : 0.0f;
                                q.z = k + 2 < end ? wr[k + 2] : 0.0f;
                            }
                        }
                        v[u][4 * c + 0] = q.x;
                        v[u][4 * c + 1] = q.y;
                        v[u][4 * c + 2] = q.z;
                        v[u][4 * c + 3] = q.w;
                    }
                }
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const int i = i0 + 64 * kRrWaves * u;
                    if (i < total) {
                        if (plain) {
                            float4* d = dn + (i >> 6) * 128 + (i & 63);
                            d[0] = make_float4(v[u][0], v[u][1], v[u][2], v[u][3]);
                            d[64] = make_float4(v[u][4], v[u][5], v[u][6], v[u][7]);
                            continue;
                        }
                        // (the smallest by its bits doubled, less one, which
                        // puts 0 last; a NaN is above the range)
                        unsigned most = 0, least = ~0u;
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const unsigned d = __float_as_uint(v[u][e]) << 1;
                            most = max(most, d);
                            least = min(least, d - 1);
                        }
                        outside |= most >= __float_as_uint(kRrMaxW) << 1 || least < (__float_as_uint(kRrSmall) << 1) - 1;
                        uint4 p[3];
                        rr_split(v[u], p);
#pragma unroll
                        for (int q = 0; q < 3; ++q) dst[((i >> 6) * 3 + q) * 64 + (i & 63)] = p[q];
                    }
                }
            }
            const float* __restrict__ bs = a.bias[l];
            for (int e = tid; e < nob * 32; e += 64 * kRrWaves)
                smem[a.boff[l] + e] = (bs && e < N) ? bs[e] : 0.0f;
        }
        if (plain) return;
        const bool any = __any(outside);
        if (lane == 0) reinterpret_cast<int*>(smem)[a.foff + wave] = any;
    };
    bool plain_w = false;   // the staged weights are fp32
    auto stage_phase = [&](int l0, int l1) {
        stage(l0, l1, false);
        __syncthreads();
        int f = 0;
#pragma unroll
        for (int i = 0; i < kRrWaves; ++i) f |= reinterpret_cast<const int*>(smem)[a.foff + i];
        plain_w = __builtin_amdgcn_readfirstlane(f) != 0;
        if (plain_w) {
            stage(l0, l1, true);
            __syncthreads();
        }
    };

    // layer l on this wave's tile (rows row - lane % 32 ..): act in, act
    // out, or the output rows after the last layer
    auto layer = [&](int l, int64_t row, bool rok) {
        const int N = a.dims[l + 1];
        const int nob = rr_blocks(N);
        const int nt = rr_steps(a.dims, l, a.k0h);
        const float4* __restrict__ wn = smem4 + (a.woff[l] >> 2) + lane;
        const uint4* __restrict__ wl = reinterpret_cast<const uint4*>(wn) + rr_narrow_floats(nob, l, a.cs) / 4;
        f32x16 acc[kRrMaxWidth / 32];
        const bool relu = (a.relu_mask >> l) & 1u;
#pragma unroll
        for (int ob = 0; ob < kRrMaxWidth / 32; ++ob)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ob][r] = 0.0f;
        if (plain_w) {
            rr_products_f32_any(nt, nob, reinterpret_cast<const float4*>(wl), act, acc);
        } else {
            // the row's largest value (NaN apart, whose parts are NaN)
            float top = 0.0f;
#pragma unroll
            for (int i = 0; i < kRrMaxSteps; i += 8)
                if (i < 8 * nt)
#pragma unroll
                    for (int e = 0; e < 8; e += 2)
                        asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(top) : "v"(act[i + e]), "v"(act[i + e + 1]));
            if (__any(!(top < kRrMaxX) || (top < kRrSmall && top > 0.0f))) rr_products_plain(nt, nob, wl, act, acc);
            else if (nt > 0) rr_products(nt, nob, wl, act, acc);
        }
        if (l == 0 && a.cs > 0) rr_narrow(nob, wn, sm, acc);
        const float* __restrict__ bl = smem + a.boff[l] + 4 * hk;
#pragma unroll
        for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) {
            if (ob < nob) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 b4 = *reinterpret_cast<const float4*>(bl + 32 * ob + 8 * q);
                    acc[ob][4 * q + 0] += b4.x;
                    acc[ob][4 * q + 1] += b4.y;
                    acc[ob][4 * q + 2] += b4.z;
                    acc[ob][4 * q + 3] += b4.w;
                }
            }
        }
        if (l + 1 < a.n_layers) {
            // the accumulators, activated, become the next layer's B operand
            // in its k order (steps past the layer's blocks are never read)
#pragma unroll
            for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) {
                if (ob < nob) {
                    if (relu) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) act[16 * ob + r] = rr_relu(acc[ob][r]);
                    } else {
#pragma unroll
                        for (int r = 0; r < 16; ++r) act[16 * ob + r] = acc[ob][r];
                    }
                }
            }
        } else if constexpr (POOLED) {
            // the max over the 16 or 32 lanes that hold a centroid's rows
            // (the values are not negative: they order as their bits); the
            // last quad of the group stores it
            const bool whole = a.g.k == 32;
            const bool last = rok && (lane & (whole ? 28 : 12)) == (whole ? 28 : 12);
            float* yr = a.y + (int64_t)((uint64_t)row / (uint32_t)a.g.k) * a.ldy;
            const bool odd = lane & 1, high = lane & 2;
#pragma unroll
            for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) {
                if (ob < nob) {
                    // quads first, halving the registers: lane i of a quad
                    // ends with the quad's max of channel i of each four
                    int m[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        int v[4], h[2];
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = __float_as_int(rr_relu(acc[ob][4 * q + i]));
#pragma unroll
                        for (int i = 0; i < 2; ++i) {   // channels 2 i, 2 i + 1: even lanes keep the first
                            const int give = odd ? v[2 * i] : v[2 * i + 1], keep = odd ? v[2 * i + 1] : v[2 * i];
                            h[i] = max(keep, __builtin_amdgcn_mov_dpp(give, 0xB1, 0xf, 0xf, true));   // lane ^ 1
                        }
                        const int give = high ? h[0] : h[1], keep = high ? h[1] : h[0];
                        m[q] = max(keep, __builtin_amdgcn_mov_dpp(give, 0x4E, 0xf, 0xf, true));       // lane ^ 2
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) m[q] = dpp_max_i32<0x124>(m[q]);   // row_ror:4
#pragma unroll
                    for (int q = 0; q < 4; ++q) m[q] = dpp_max_i32<0x128>(m[q]);   // row_ror:8
                    if (whole) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {   // the row above and the row below
                            auto w = __builtin_amdgcn_permlane16_swap((unsigned)m[q], (unsigned)m[q], false, false);
                            m[q] = max((int)w[0], (int)w[1]);
                        }
                    }
                    if (last) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int c = 32 * ob + 8 * q + 4 * hk + (lane & 3);
                            if (c < N) yr[c] = __int_as_float(m[q]);
                        }
                    }
                }
            }
        } else if (rok) {
            float* yr = a.y + row * a.ldy;
#pragma unroll
            for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) {
                if (ob < nob) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int c = 32 * ob + 8 * q + 4 * hk;
                        float v[4] = {acc[ob][4 * q + 0], acc[ob][4 * q + 1], acc[ob][4 * q + 2], acc[ob][4 * q + 3]};
                        if (relu) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) v[i] = rr_relu(v[i]);
                        }
                        if (a.vecy && c + 4 <= N) {
                            *reinterpret_cast<float4*>(yr + c) = make_float4(v[0], v[1], v[2], v[3]);
                        } else {
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (c + i < N) yr[c + i] = v[i];
                        }
                    }
                }
            }
        }
    };

    if constexpr (!PHASED) {
        stage_phase(0, a.n_layers);
        for (int64_t t = t0; t < a.tiles; t += stride) {
            const int64_t row = t * 32 + (lane & 31);
            const bool rok = row < a.rows;
            if (t != t0) load_tile(t, act);
            for (int l = 0; l < a.n_layers; ++l) layer(l, row, rok);
        }
    } else {
        // the weights do not fit at once: the layers run in phases, the
        // workgroup staging the LDS anew between them while the tiles'
        // activations stay in registers; every wave takes every barrier,
        // with or without a tile
        for (int64_t w0 = t0 - wave; w0 < a.tiles; w0 += stride) {
            const int64_t t = w0 + wave;
            const int64_t row = t * 32 + (lane & 31);
            const bool rok = row < a.rows;
            if (t != t0 && t < a.tiles) load_tile(t, act);
            for (int p = 0; p < a.nphase; ++p) {
                __syncthreads();   // every wave is done with the previous phase's weights
                stage_phase(a.phase_first[p], a.phase_first[p + 1]);
                if (t < a.tiles)
                    for (int l = a.phase_first[p]; l < a.phase_first[p + 1]; ++l) layer(l, row, rok);
            }
        }
    }
}

// Layers of at most 64 outputs, most of them of one block of 32, take the fp32
// instruction throughout: the split of a row and the ten LDS reads of a step
// would serve one or two blocks' products (rr_fp32_form).  All weights are in
// LDS as fp32, in groups of four k steps.  Bound by the latency of a wave's one
// or few tiles: rows from memory, a chain of products, rows to memory.
template <int NJ, int NOB>
__device__ __forceinline__ void rr_products_f32(const float4* __restrict__ wl, const float (&act)[kRrMaxSteps],
                                                f32x16 (&acc)[2]) {
#pragma unroll
    for (int ob = 0; ob < NOB; ++ob)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ob][r] = 0.0f;
    float4 w[NOB];
#pragma unroll
    for (int ob = 0; ob < NOB; ++ob) w[ob] = wl[ob * 4 * NJ * 64];
#pragma unroll
    for (int g = 0; g < 4 * NJ; ++g) {
        // the next group's weights are requested before this group's MFMAs
        float4 wn[NOB];
        if (g + 1 < 4 * NJ) {
#pragma unroll
            for (int ob = 0; ob < NOB; ++ob) wn[ob] = wl[(ob * 4 * NJ + g + 1) * 64];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int ob = 0; ob < NOB; ++ob)
                acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32((&w[ob].x)[e], act[4 * g + e], acc[ob], 0, 0, 0);
        // keeps the compiler from hoisting every group's weights at once
        __builtin_amdgcn_sched_barrier(0);
        if (g + 1 < 4 * NJ) {
#pragma unroll
            for (int ob = 0; ob < NOB; ++ob) w[ob] = wn[ob];
        }
    }
}

__global__ __launch_bounds__(64 * kRrWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void mlp_rr_f32_kernel(RrArgs a) {
    extern __shared__ float4 smem4[];
    float* smem = reinterpret_cast<float*>(smem4);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hk = lane >> 5;

    float act[kRrMaxSteps];
    auto load_tile = [&](int64_t t) {
        const int64_t row = t * 32 + (lane & 31);
        int kb = 4 * hk;
        asm volatile("" : "+v"(kb));
        rr_load_rows(a, row, row < a.rows, kb, act);
    };
    const int64_t stride = (int64_t)gridDim.x * kRrWaves;
    int64_t wg = blockIdx.x;
    if (a.interp && (gridDim.x & 7) == 0) wg = (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int64_t t0 = wg * kRrWaves + wave;
    if (t0 < a.tiles) load_tile(t0);

    // a layer's float4s, four consecutive k of one weight row each: at most 2
    // blocks x 16 groups x 64 lanes, all of its loads in flight before the
    // first LDS store
    constexpr int kPer = 2 * 16 * 64 / (64 * kRrWaves);
    for (int l = 0; l < a.n_layers; ++l) {
        const int K = a.dims[l], N = a.dims[l + 1];
        const int ng = 2 * rr_steps(a.dims, l, a.k0h);
        const int total = rr_blocks(N) * ng * 64;
        const unsigned inv = (65536u + ng - 1) / ng;   // gg / ng exactly for gg < 32
        const float* __restrict__ W = a.W[l];
        float4 v[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = tid + 64 * kRrWaves * u;
            const int ln = i & 63, gg = i >> 6;
            const int ob = (int)(((unsigned)gg * inv) >> 16), g = gg - ob * ng;
            const int n = ob * 32 + (ln & 31);
            const int k = rr_k(l, 4 * g, ln >> 5);   // k .. k + 3 are consecutive
            v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (i < total && n < N) {
                const float* wr = W + (int64_t)n * K;
                if (k + 4 <= K) {
                    struct __attribute__((packed, aligned(4))) F4 { float x, y, z, w; };
                    const F4 p = *reinterpret_cast<const F4*>(wr + k);
                    v[u] = make_float4(p.x, p.y, p.z, p.w);
                } else {
                    v[u].x = k + 0 < K ? wr[k + 0] : 0.0f;
                    v[u].y = k + 1 < K ? wr[k + 1] : 0.0f;
                    v[u].z = k + 2 < K ? wr[k + 2] : 0.0f;
                }
            }
        }
        float4* dst = smem4 + (a.woff[l] >> 2);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = tid + 64 * kRrWaves * u;
            if (i < total) dst[i] = v[u];
        }
        const float* __restrict__ bs = a.bias[l];
        for (int e = tid; e < rr_blocks(N) * 32; e += 64 * kRrWaves)
            smem[a.boff[l] + e] = (bs && e < N) ? bs[e] : 0.0f;
    }
    __syncthreads();

    for (int64_t t = t0; t < a.tiles; t += stride) {
        const int64_t row = t * 32 + (lane & 31);
        const bool rok = row < a.rows;
        if (t != t0) load_tile(t);
        for (int l = 0; l < a.n_layers; ++l) {
            const int N = a.dims[l + 1];
            const int nob = rr_blocks(N), nj = rr_steps(a.dims, l, a.k0h) / 2;
            const float4* __restrict__ wl = smem4 + (a.woff[l] >> 2) + lane;
            f32x16 acc[2];
            switch (2 * nj + nob) {
                case 3: rr_products_f32<1, 1>(wl, act, acc); break;
                case 4: rr_products_f32<1, 2>(wl, act, acc); break;
                case 5: rr_products_f32<2, 1>(wl, act, acc); break;
                case 6: rr_products_f32<2, 2>(wl, act, acc); break;
                case 7: rr_products_f32<3, 1>(wl, act, acc); break;
                case 8: rr_products_f32<3, 2>(wl, act, acc); break;
                case 9: rr_products_f32<4, 1>(wl, act, acc); break;
                default: rr_products_f32<4, 2>(wl, act, acc); break;
            }
            const bool relu = (a.relu_mask >> l) & 1u, last = l + 1 == a.n_layers;
            const float* __restrict__ bl = smem + a.boff[l] + 4 * hk;
            float* yr = a.y + row * a.ldy;
#pragma unroll
            for (int ob = 0; ob < 2; ++ob) {
                if (ob < nob) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 b4 = *reinterpret_cast<const float4*>(bl + 32 * ob + 8 * q);
                        float v[4] = {acc[ob][4 * q + 0] + b4.x, acc[ob][4 * q + 1] + b4.y,
                                      acc[ob][4 * q + 2] + b4.z, acc[ob][4 * q + 3] + b4.w};
                        if (relu) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) v[i] = rr_relu(v[i]);
                        }
                        const int c = 32 * ob + 8 * q + 4 * hk;
                        if (!last) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) act[16 * ob + 4 * q + i] = v[i];
                        } else if (rok) {
                            if (a.vecy && c + 4 <= N) {
                                *reinterpret_cast<float4*>(yr + c) = make_float4(v[0], v[1], v[2], v[3]);
                            } else {
#pragma unroll
                                for (int i = 0; i < 4; ++i)
                                    if (c + i < N) yr[c + i] = v[i];
                            }
                        }
                    }
                }
            }
        }
    }
}

struct RrPlan {
    bool ok;
    int k0h;
    int lds_floats, foff;
    int woff[MESORASI_MAX_LAYERS], boff[MESORASI_MAX_LAYERS];
    int nphase;
    int phase_first[MESORASI_MAX_LAYERS + 1];
};

// Layers packed greedily into phases whose permuted weights and biases fit
// the LDS (one phase when they all fit).
// cs: the channels of dims[0] that come from a narrow source.
RrPlan rr_plan(int n_layers, const int32_t* dims, int cs) {
    RrPlan p{};
    if (n_layers < 1 || cs > 8 || cs > dims[0]) return p;
    p.k0h = (int)(ceil_div(ceil_div(dims[0] - cs, 2), 16) * 16);
    if (p.k0h > kRrMaxSteps) return p;
    const int cap = kRrMaxLds / (int)sizeof(float) - kRrWaves;   // (the waves' flags behind the weights)
    int off = 0, most = 0;
    p.nphase = 1;
    p.phase_first[0] = 0;
    for (int l = 0; l < n_layers; ++l) {
        if (dims[l + 1] > kRrMaxWidth || (l > 0 && dims[l] > kRrMaxWidth)) return p;
        const int nob = rr_blocks(dims[l + 1]);
        const int size = rr_floats(dims, l, p.k0h, cs);
        if (size > cap) return p;
        if (off + size > cap) {
            p.phase_first[p.nphase++] = l;
            off = 0;
        }
        p.woff[l] = off;
        p.boff[l] = off + size - nob * 32;
        off += size;
        most = std::max(most, off);
    }
    p.phase_first[p.nphase] = n_layers;
    p.foff = most;
    p.lds_floats = most + kRrWaves;
    p.ok = true;
    return p;
}

// All layers at most 64 wide and 3 F <= 5 S, F the output blocks' steps and S
// the steps: the fp32 instruction (mlp_rr_f32_kernel), for sources without a
// narrow one.  Measured, fp32 instruction against split, 65536 and 262144 rows:
// F = S: 128 -> 32 16.2 / 18.8 and 50 / 53 us, 16 -> 8 x 32 23.3 / 31.7 and 66 /
// 83; 128 -> 32 -> 32 -> 64 (14 : 12) 22.9 / 25.5 and 73 / 77; on the line, 128 ->
// 64 -> 32, 23.5 / 25.1 and 76 / 72; beyond it 64 -> 64 -> 64 (2 : 1) 22.0 / 19.9
// and 69 / 57, 128 -> 64 -> 64 27.8 / 25.3 and 92 / 77.
bool rr_fp32_form(int n_layers, const int32_t* dims, int k0h) {
    int f = 0, st = 0;
    for (int l = 0; l < n_layers; ++l) {
        const int nob = rr_blocks(dims[l + 1]), nt = rr_steps(dims, l, k0h);
        if (nob > 2) return false;
        f += nob * nt;
        st += nt;
    }
    return 3 * f <= 5 * st;
}

hipError_t rr_lds_attr(void (*kernel)(RrArgs)) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               kRrMaxLds);
}

int rr_cus() {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) cus = v;
    }
    return cus;
}

}  // namespace

// How a first layer's sources [x0 | x1] are read: which one is narrow (0 or
// 1; 2: both, -1: neither, the element loader of at most 128 channels).
static int rr_narrow_source(const float* x0, int c0, int64_t ld0, const float* x1, int c1, int64_t ld1) {
    const auto wide = [](const float* x, int c, int64_t ld) { return c % 4 == 0 && ld % 4 == 0 && aligned(x, 16); };
    if (!x1 || c1 == 0) return c0 <= 8 ? 2 : -1;
    if (c0 + c1 <= 8) return 2;
    if (c0 <= 8 && wide(x1, c1, ld1)) return 0;
    if (c1 <= 8 && wide(x0, c0, ld0)) return 1;
    return -1;
}

// Any row count for layers of at most 160 KB of fp32 weights; with more, which
// take three or more phases of staging, only while every wave holds at most
// one 32-row tile (one persistent workgroup of kRrWaves waves per CU).
static bool rr_rows_ok(int n_layers, const int32_t* dims, int cs, int64_t tiles_per_wave) {
    const RrPlan pl = rr_plan(n_layers, dims, cs);
    if (!pl.ok) return false;
    int64_t bytes = 0;
    for (int l = 0; l < n_layers; ++l)
        bytes += rr_blocks(dims[l + 1]) * (rr_steps(dims, l, pl.k0h) * 2048 + (l == 0 && cs > 0 ? 1024 : 0) + 128);
    return bytes <= kRrMaxLds || tiles_per_wave <= 1;
}
static int64_t rr_tiles_per_wave(int64_t rows) { return ceil_div(ceil_div(rows, 32), (int64_t)rr_cus() * kRrWaves); }

bool rr_mlp_supported(int n_layers, const int32_t* dims, int64_t rows) {
    return dims[0] <= kRrMaxWidth && rr_rows_ok(n_layers, dims, 0, rr_tiles_per_wave(rows));
}

bool rr_mlp_supported(const float* x0, int c0, int64_t ld0, const float* x1, int c1, int64_t ld1, int n_layers,
                      const int32_t* dims, int64_t rows) {
    const int narrow = rr_narrow_source(x0, c0, ld0, x1, c1, ld1);
    if (narrow < 0) return rr_mlp_supported(n_layers, dims, rows);
    // a single layer of more than 128 inputs, whose GEMM has no intermediate
    // to keep from memory, is that GEMM (65536 x 131 -> 13, 32, 64: 15.6, 16.3,
    // 18.5 us, here 18.5, 19.0, 21.1; 262144 x 131 -> 64: 56 against 69)
    if (n_layers == 1 && dims[0] > kRrMaxWidth) return false;
    return rr_rows_ok(n_layers, dims, narrow == 2 ? dims[0] : narrow == 0 ? c0 : c1, rr_tiles_per_wave(rows));
}

bool rr_pool_supported(int cf, const float* feat, int64_t ld_f, int n_layers, const int32_t* dims, int K) {
    if (K != 16 && K != 32) return false;
    if (cf > 0 && (cf % 4 != 0 || ld_f % 4 != 0 || !aligned(feat, 16))) return false;
    return rr_rows_ok(n_layers, dims, 3, 2);
}

int run_rr_mlp(const float* x0, int c0, int64_t ld0, const float* x1, int c1, int64_t ld1, int64_t rows,
               int n_layers, const int32_t* dims, const void* const* W, const float* const* bias,
               uint32_t relu_mask, float* y, int64_t ld_y, hipStream_t s, const RrInterp* ip, const MlpGather* g) {
    const int narrow = ip ? -1 : g ? 0 : rr_narrow_source(x0, c0, ld0, x1, c1, ld1);
    const int cs = narrow < 0 ? 0 : narrow == 2 ? dims[0] : narrow == 0 ? c0 : c1;
    const RrPlan pl = rr_plan(n_layers, dims, cs);
    MESO_REQUIRE(pl.ok, MESORASI_EUNSUPPORTED, "mesorasi_pointwise_mlp: layers too wide for the register MLP");
    if (rows == 0) return MESORASI_OK;
    const int cus = rr_cus();
    static const auto kernels = std::array<void (*)(RrArgs), 4>{
        &mlp_rr_kernel<false, false>, &mlp_rr_kernel<false, true>, &mlp_rr_kernel<true, false>,
        &mlp_rr_kernel<true, true>};
    static const hipError_t attr[5] = {rr_lds_attr(kernels[0]), rr_lds_attr(kernels[1]), rr_lds_attr(kernels[2]),
                                       rr_lds_attr(kernels[3]), rr_lds_attr(&mlp_rr_f32_kernel)};
    for (const hipError_t e : attr)
        MESO_REQUIRE(e == hipSuccess, MESORASI_EHIP, "mesorasi_pointwise_mlp: LDS size attribute: %s",
                     hipGetErrorString(e));
    RrArgs a{};
    a.x0 = x0; a.ld0 = ld0; a.x1 = x1; a.ld1 = ld1; a.c0 = c0; a.c1 = x1 ? c1 : 0;
    if (narrow >= 0) {
        // the narrow source apart, the wide one (if any) alone as x0
        a.cs = cs;
        a.xs = narrow == 1 ? x1 : x0;
        a.lds = narrow == 1 ? ld1 : ld0;
        a.cs0 = narrow == 2 ? c0 : cs;
        a.xs1 = narrow == 2 ? a.x1 : nullptr;
        a.lds1 = ld1;
        a.sw = narrow == 1 ? c0 : 0;
        a.ww = narrow == 0 ? c0 : 0;
        if (narrow == 2) {
            a.x0 = nullptr;
            a.c0 = 0;
        }
        if (narrow == 0) {
            a.x0 = a.x1;
            a.ld0 = a.ld1;
            a.c0 = a.c1;
        }
        a.x1 = nullptr;
        a.c1 = 0;
    }
    if (g) a.g = *g;
    a.rows = rows;
    a.tiles = ceil_div(rows, 32);
    a.n_layers = n_layers;
    for (int l = 0; l <= n_layers; ++l) a.dims[l] = dims[l];
    for (int l = 0; l < n_layers; ++l) {
        a.W[l] = static_cast<const float*>(W[l]);
        a.bias[l] = bias ? bias[l] : nullptr;
        a.woff[l] = pl.woff[l];
        a.boff[l] = pl.boff[l];
    }
    a.foff = pl.foff;
    a.nphase = pl.nphase;
    for (int q = 0; q <= pl.nphase; ++q) a.phase_first[q] = pl.phase_first[q];
    a.relu_mask = relu_mask;
    a.y = y;
    a.ldy = ld_y;
    a.k0h = pl.k0h;
    a.vec0 = a.c1 == 0 && a.c0 % 4 == 0 && a.ld0 % 4 == 0 && aligned(a.x0, 16);
    if (ip) {
        a.interp = 1;
        a.ip = *ip;
        a.c0 = dims[0];
        a.c1 = 0;
    }
    a.vecy = ld_y % 4 == 0 && aligned(y, 16);
    // one persistent workgroup per CU (the weights fill most of the LDS);
    // interpolated rows: a multiple of 8 workgroups where that stays within
    // the CUs (the kernel then orders tiles by XCD)
    int64_t grid = std::min<int64_t>(ceil_div(a.tiles, kRrWaves), cus);
    if ((a.interp || g) && 8 * ceil_div(grid, 8) <= cus) grid = 8 * ceil_div(grid, 8);
    if (!g && cs == 0 && rr_fp32_form(n_layers, dims, pl.k0h)) {
        int off = 0;   // at most 32 KB for the first layer and 16 for each other
        for (int l = 0; l < n_layers; ++l) {
            const int nob = rr_blocks(dims[l + 1]);
            a.woff[l] = off;
            a.boff[l] = off + nob * rr_steps(dims, l, pl.k0h) * 512;
            off = a.boff[l] + nob * 32;
        }
        mlp_rr_f32_kernel<<<dim3((unsigned)grid), dim3(64 * kRrWaves), (size_t)off * sizeof(float), s>>>(a);
        return after_launch("mesorasi_pointwise_mlp (register MLP, fp32 products)");
    }
    const size_t lds = (size_t)pl.lds_floats * sizeof(float);
    kernels[(pl.nphase > 1 ? 2 : 0) + (g ? 1 : 0)]<<<dim3((unsigned)grid), dim3(64 * kRrWaves), lds, s>>>(a);
    return after_launch("mesorasi_pointwise_mlp (register MLP)");
}

}  // namespace meso
