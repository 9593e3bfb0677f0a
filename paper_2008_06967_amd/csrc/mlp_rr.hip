// Register-resident shared MLP for narrow fp32 layers on many rows, gfx950.
//
// The per-point MLP F (Sec. 4: with delayed aggregation it runs once per
// input point) on layers of at most 128 channels, e.g. the last feature
// propagation level and the per-point head of the segmentation network
// (65536 rows), where a layer-by-layer GEMM writes and re-reads every
// intermediate activation and stages it through LDS.
//
// Each wave pushes 32-row tiles through every layer on its own.  The
// product is taken transposed, Y^T = W X^T, on v_mfma_f32_32x32x2_f32: the
// weights are the A operand (32 output channels x 2 k) and the activations
// the B operand (2 k x 32 rows), so a lane's 16 accumulators of a 32-channel
// block hold 16 output channels of ONE row, its lane % 32 (channel 8(r/4) +
// 4(lane/32) + r%4 of register r).  An MFMA sums over whatever k order its
// two operands share, so the next layer takes its k steps in exactly that
// register order: step (j, r) is the k pair {32j + 8(r/4) + r%4, +4}, lane
// half h supplying its own accumulator r of block j.  The activations never
// leave registers between layers: no LDS round trip, no barrier, no
// transpose.  The weights, permuted once per workgroup into each layer's k
// order, are the only LDS data: a workgroup is persistent, loads every
// layer's weights and biases once, and its eight waves then stream tiles.
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

#include "common.h"
#include "mlp_internal.h"

namespace meso {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kRrWaves = 8;          // waves per workgroup (two per SIMD)
constexpr int kRrMaxWidth = 128;     // widest layer input or output
constexpr int kRrMaxSteps = 64;      // k steps of a layer (128 inputs / 2)
constexpr int kRrMaxLds = 160 * 1024;

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
    int lds_floats;
    // weights staged in phases when all layers do not fit at once: phase p
    // holds layers phase_first[p] .. phase_first[p + 1] - 1 (offsets above
    // relative to the phase); then every wave holds at most one tile
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
// k steps of layer l: 16 per 32-channel input block; the first layer's
// half-rows are padded to whole blocks of 16 steps too (k0h = 16 nj), and its
// narrow source takes 4 ahead of them
__host__ __device__ inline int rr_steps(const int* dims, int l, int k0h, int cs) {
    return l == 0 ? k0h + (cs > 0 ? 4 : 0) : 16 * rr_blocks(dims[l]);
}

// The input channel that lane half h supplies at k step s of layer l.
__device__ __forceinline__ int rr_k(int l, int s, int h) {
    // first layer: the two lanes of a row take alternate 4-channel chunks,
    // so a row's 128-byte line is read whole by four consecutive loads
    if (l == 0) return 8 * (s >> 2) + 4 * h + (s & 3);
    const int j = s >> 4, r = s & 15;
    return 32 * j + 8 * (r >> 2) + (r & 3) + 4 * h;
}

// One layer's products: NJ input blocks of 16 k steps, NOB output blocks
// whose weights lie `ng` groups of four steps apart, the output blocks'
// accumulation chains interleaved step by step.
template <int NJ, int NOB>
__device__ __forceinline__ void rr_products(const float4* __restrict__ wl, int ng, const float (&act)[kRrMaxSteps],
                                            f32x16 (&acc)[kRrMaxWidth / 32]) {
    float4 w[NOB];
#pragma unroll
    for (int ob = 0; ob < NOB; ++ob) w[ob] = wl[ob * ng * 64];
#pragma unroll
    for (int g = 0; g < 4 * NJ; ++g) {
        // the next group's weights are requested before this group's MFMAs
        float4 wn[NOB];
        if (g + 1 < 4 * NJ) {
#pragma unroll
            for (int ob = 0; ob < NOB; ++ob) wn[ob] = wl[(ob * ng + g + 1) * 64];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ob = 0; ob < NOB; ++ob)
            acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[ob].x, act[4 * g + 0], acc[ob], 0, 0, 0);
#pragma unroll
        for (int ob = 0; ob < NOB; ++ob)
            acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[ob].y, act[4 * g + 1], acc[ob], 0, 0, 0);
#pragma unroll
        for (int ob = 0; ob < NOB; ++ob)
            acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[ob].z, act[4 * g + 2], acc[ob], 0, 0, 0);
#pragma unroll
        for (int ob = 0; ob < NOB; ++ob)
            acc[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[ob].w, act[4 * g + 3], acc[ob], 0, 0, 0);
        // keeps the compiler from hoisting every group's weights at once
        __builtin_amdgcn_sched_barrier(0);
        if (g + 1 < 4 * NJ) {
#pragma unroll
            for (int ob = 0; ob < NOB; ++ob) w[ob] = wn[ob];
        }
    }
}

template <int NJ>
__device__ __forceinline__ void rr_products_nob(int nob, const float4* __restrict__ wl, int ng,
                                                const float (&act)[kRrMaxSteps], f32x16 (&acc)[kRrMaxWidth / 32]) {
    switch (nob) {
        case 1: rr_products<NJ, 1>(wl, ng, act, acc); break;
        case 2: rr_products<NJ, 2>(wl, ng, act, acc); break;
        case 3: rr_products<NJ, 3>(wl, ng, act, acc); break;
        default: rr_products<NJ, 4>(wl, ng, act, acc); break;
    }
}

// The narrow source's four steps.
__device__ __forceinline__ void rr_narrow(int nob, const float4* __restrict__ wl, int ng, const float (&sm)[4],
                                          f32x16 (&acc)[kRrMaxWidth / 32]) {
#pragma unroll
    for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) {
        if (ob < nob) {
            const float4 w = wl[ob * ng * 64];
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

// Eight waves, two per SIMD: while one wave waits on its rows or runs its
// epilogue, the other keeps the SIMD's MFMA pipe busy.  (A four-wave form
// with 512 registers per wave that requested its next tile's rows before
// computing the current one measured 9-18 % slower.)
// PHASED: the weights staged in phases, at most one tile per wave.  POOLED:
// gathered neighbor rows, the output their max per centroid.
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

    // weights: layer l, output block ob, step group g = s / 4, lane, s % 4;
    // thread tid fills float4s tid + 512 u (at most 4 blocks x 17
    // groups x 64 lanes), each 4 consecutive k of one weight row; all of a
    // layer's loads are in flight before the first LDS store
    constexpr int kPer = (4 * 17 * 64 + 64 * kRrWaves - 1) / (64 * kRrWaves);
    auto stage = [&](int l0, int l1) {
        for (int l = l0; l < l1; ++l) {
            const int K = a.dims[l], N = a.dims[l + 1];
            const int ng = rr_steps(a.dims, l, a.k0h, a.cs) / 4;
            const int total = rr_blocks(N) * ng * 64;
            const unsigned inv = (65536u + ng - 1) / ng;   // gg / ng exactly for gg < 128
            const float* __restrict__ W = a.W[l];
            const bool wvec = (K % 4) == 0 && (reinterpret_cast<uintptr_t>(W) & 15) == 0;
            float4 v[kPer];
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const int i = tid + 64 * kRrWaves * u;
                const int ln = i & 63, gg = i >> 6;
                const int ob = (int)(((unsigned)gg * inv) >> 16), g = gg - ob * ng;
                const int n = ob * 32 + (ln & 31);
                // columns k .. k + 3 of [base, end): a layer's inputs, or one
                // of the first layer's two sources
                const bool two = l == 0 && a.cs > 0, narrow = two && g == 0;
                const int base = two ? (narrow ? a.sw : a.ww) : 0;
                const int end = two ? base + (narrow ? a.cs : K - a.cs) : K;
                const int k = base + (narrow ? 4 * (ln >> 5) : rr_k(l, 4 * (two ? g - 1 : g), ln >> 5));
                v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (i < total && n < N) {
                    const float* wr = W + (int64_t)n * K;
                    if (wvec && !two && k + 4 <= K) {
                        v[u] = *reinterpret_cast<const float4*>(wr + k);
                    } else {
                        v[u].x = k + 0 < end ? wr[k + 0] : 0.0f;
                        v[u].y = k + 1 < end ? wr[k + 1] : 0.0f;
                        v[u].z = k + 2 < end ? wr[k + 2] : 0.0f;
                        v[u].w = k + 3 < end ? wr[k + 3] : 0.0f;
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
    };

    // layer l on this wave's tile (rows row - lane % 32 ..): act in, act
    // out, or the output rows after the last layer
    auto layer = [&](int l, int64_t row, bool rok) {
        const int N = a.dims[l + 1];
        const int nob = rr_blocks(N);
        const int ng = rr_steps(a.dims, l, a.k0h, a.cs) / 4;
        const float4* __restrict__ wl = smem4 + (a.woff[l] >> 2) + lane;
        f32x16 acc[kRrMaxWidth / 32];
        const bool relu = (a.relu_mask >> l) & 1u;
        // the sums start from the bias: VALU work that does not overlap the
        // MFMAs is what this kernel loses
        const float* __restrict__ bl = smem + a.boff[l] + 4 * hk;
#pragma unroll
        for (int ob = 0; ob < kRrMaxWidth / 32; ++ob) {
            if (ob < nob) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 b4 = *reinterpret_cast<const float4*>(bl + 32 * ob + 8 * q);
                    acc[ob][4 * q + 0] = b4.x;
                    acc[ob][4 * q + 1] = b4.y;
                    acc[ob][4 * q + 2] = b4.z;
                    acc[ob][4 * q + 3] = b4.w;
                }
            }
        }
        if (l == 0 && a.cs > 0) {
            rr_narrow(nob, wl, ng, sm, acc);
            wl += 64;
        }
        switch (ng >> 2) {   // (the narrow source's group is the odd one)
            case 0: break;
            case 1: rr_products_nob<1>(nob, wl, ng, act, acc); break;
            case 2: rr_products_nob<2>(nob, wl, ng, act, acc); break;
            case 3: rr_products_nob<3>(nob, wl, ng, act, acc); break;
            default: rr_products_nob<4>(nob, wl, ng, act, acc); break;
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
        stage(0, a.n_layers);
        __syncthreads();
        for (int64_t t = t0; t < a.tiles; t += stride) {
            const int64_t row = t * 32 + (lane & 31);
            const bool rok = row < a.rows;
            if (t != t0) load_tile(t, act);
            for (int l = 0; l < a.n_layers; ++l) layer(l, row, rok);
        }
    } else {
        // the weights do not fit at once: the layers run in phases, the
        // workgroup restaging the LDS between them, and each wave holds at
        // most one tile (the host guarantees it), whose activations stay in
        // registers across the phases.  Every wave takes every barrier.
        const int64_t row = t0 * 32 + (lane & 31);
        const bool rok = row < a.rows;
        for (int p = 0; p < a.nphase; ++p) {
            if (p > 0) __syncthreads();   // every wave is done with the previous phase's weights
            stage(a.phase_first[p], a.phase_first[p + 1]);
            __syncthreads();
            if (t0 < a.tiles)
                for (int l = a.phase_first[p]; l < a.phase_first[p + 1]; ++l) layer(l, row, rok);
        }
    }
}

struct RrPlan {
    bool ok;
    int k0h;
    int lds_floats;
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
    const int cap = kRrMaxLds / (int)sizeof(float);
    int off = 0, most = 0;
    p.nphase = 1;
    p.phase_first[0] = 0;
    for (int l = 0; l < n_layers; ++l) {
        if (dims[l + 1] > kRrMaxWidth || (l > 0 && dims[l] > kRrMaxWidth)) return p;
        const int nob = rr_blocks(dims[l + 1]);
        const int size = nob * rr_steps(dims, l, p.k0h, cs) * 64 + nob * 32;
        if (size > cap) return p;
        if (off + size > cap) {
            p.phase_first[p.nphase++] = l;
            off = 0;
        }
        p.woff[l] = off;
        p.boff[l] = off + nob * rr_steps(dims, l, p.k0h, cs) * 64;
        off += size;
        most = std::max(most, off);
    }
    p.phase_first[p.nphase] = n_layers;
    p.lds_floats = most;
    p.ok = true;
    return p;
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

// One phase for any row count; several only while every wave holds at most
// one 32-row tile (one persistent workgroup of kRrWaves waves per CU).
static bool rr_rows_ok(const RrPlan& pl, int64_t rows) {
    return pl.ok && (pl.nphase == 1 || ceil_div(rows, 32) <= (int64_t)rr_cus() * kRrWaves);
}

bool rr_mlp_supported(int n_layers, const int32_t* dims, int64_t rows) {
    return dims[0] <= kRrMaxWidth && rr_rows_ok(rr_plan(n_layers, dims, 0), rows);
}

bool rr_mlp_supported(const float* x0, int c0, int64_t ld0, const float* x1, int c1, int64_t ld1, int n_layers,
                      const int32_t* dims, int64_t rows) {
    const int narrow = rr_narrow_source(x0, c0, ld0, x1, c1, ld1);
    if (narrow < 0) return rr_mlp_supported(n_layers, dims, rows);
    return rr_rows_ok(rr_plan(n_layers, dims, narrow == 2 ? dims[0] : narrow == 0 ? c0 : c1), rows);
}

bool rr_pool_supported(int cf, const float* feat, int64_t ld_f, int n_layers, const int32_t* dims, int K) {
    if (K != 16 && K != 32) return false;
    if (cf > 0 && (cf % 4 != 0 || ld_f % 4 != 0 || !aligned(feat, 16))) return false;
    const RrPlan pl = rr_plan(n_layers, dims, 3);
    return pl.ok && pl.nphase == 1;
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
    MESO_REQUIRE(rr_rows_ok(pl, rows) && (!g || pl.nphase == 1), MESORASI_EUNSUPPORTED,
                 "mesorasi_pointwise_mlp: staged register MLP on more than one tile per wave");
    static const hipError_t attr[3] = {
        hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_rr_kernel<false, false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kRrMaxLds),
        hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_rr_kernel<true, false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kRrMaxLds),
        hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_rr_kernel<false, true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kRrMaxLds)};
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
    a.lds_floats = pl.lds_floats;
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
    const size_t lds = (size_t)pl.lds_floats * sizeof(float);
    if (g) mlp_rr_kernel<false, true><<<dim3((unsigned)grid), dim3(64 * kRrWaves), lds, s>>>(a);
    else if (pl.nphase > 1) mlp_rr_kernel<true, false><<<dim3((unsigned)grid), dim3(64 * kRrWaves), lds, s>>>(a);
    else mlp_rr_kernel<false, false><<<dim3((unsigned)grid), dim3(64 * kRrWaves), lds, s>>>(a);
    return after_launch("mesorasi_pointwise_mlp (register MLP)");
}

}  // namespace meso
