// DiT joint (group size, format) weight search (Sec. 4.6 (i)): for every tuple (g, f) of the
// group sizes {32, 64, 128, 192, 288} and the enabled formats, each output row is quantized
// in groups of g consecutive input channels, each with its own scale (and zero point), and
// the layer's input-aware error sum_n sum_k E[x_k^2] (w - w^)^2 is formed; the tuple with
// the smallest error (ties: the lowest index t = group index * 9 + format) is emitted.  MX
// formats carry their own 32-element blocks and are evaluated at g = 32 only.  Also the
// calibration pre-pass that gives E[x_k^2]: per-input-channel sums of squares.
//
// Three launches: (1) one wavefront per output channel stages its row and the extrema of its
// 32-blocks in LDS, forms every group's parameters (one lane per group of any size) and adds
// the weighted errors of all group sizes in binary64, a format at a time; a workgroup writes
// one partial sum per tuple; (2) one workgroup sums the partials per tuple in a fixed order
// and selects the tuple on the device; (3) one wavefront per channel re-derives the chosen
// tuple's group parameters and writes the codes and group metadata.  The host never reads the
// choice, so the search and a later GEMM need no synchronization.
#include <algorithm>

#include "cham_device.h"

namespace cham {
namespace {

constexpr int kGroupSizes[CHAM_NGROUPS] = {32, 64, 128, 192, 288};
constexpr int kTuples = CHAM_NGROUPS * CHAM_W_NFMT;
constexpr int kGWaves = 4;           // channels (wavefronts) per workgroup at most
// LDS for the rows of a workgroup; the kernels hold up to 2 KB more statically (two workgroups in
// the 160 KB of a CU in any case).  Taking the static part off the 64 KB, one channel fewer per
// workgroup from 13 row lengths on, gave 4608 x 3936 228 us instead of 203, 4608 x 2944 133
// instead of 147.
constexpr int kGLdsMax = 64 * 1024;

CHAM_DEV bool mx_fmt(int f) { return f == CHAM_W_MXINT8 || f == CHAM_W_MXINT4 || f == CHAM_W_MXFP4; }

// Parameters of one group in one format: scale s, its reciprocal r, zero point z; for MX
// formats the block exponent in z.
struct GParam {
    float s, r, z;
};

CHAM_DEV GParam group_param(int f, float lo, float hi) {
    const float amax = fmaxf(fabsf(lo), fabsf(hi));
    GParam p{0.0f, 0.0f, 0.0f};
    switch (f) {
    case CHAM_W_INT8_SYM: p.s = floor_scale(amax / 127.0f); p.r = 1.0f / p.s; break;
    case CHAM_W_INT4_SYM: p.s = floor_scale(amax / 7.0f); p.r = 1.0f / p.s; break;
    case CHAM_W_INT8_ASYM: int_asym_scale_zp(lo, hi, 255.0f, &p.s, &p.z); p.r = 1.0f / p.s; break;
    case CHAM_W_INT4_ASYM: int_asym_scale_zp(lo, hi, 15.0f, &p.s, &p.z); p.r = 1.0f / p.s; break;
    case CHAM_W_FP4: p.s = floor_scale(amax / 6.0f); p.r = 1.0f / p.s; break;
    case CHAM_W_NF4: p.s = floor_scale(amax); p.r = 1.0f / p.s; break;
    case CHAM_W_MXINT8:
    case CHAM_W_MXINT4: p.z = (float)mx_exponent(amax, 0); break;
    default: p.z = (float)mx_exponent(amax, 2); break;  // MXFP4: OCP emax(E2M1) = 2
    }
    return p;
}

// Code and reconstruction of w in format f with its group's parameters (each step one
// binary32 operation, as the format defines it).
CHAM_DEV uint32_t group_quant(int f, float w, const GParam& p, float* wh) {
    switch (f) {
    case CHAM_W_INT8_SYM:
    case CHAM_W_INT4_SYM: {
        const float Q = f == CHAM_W_INT8_SYM ? 127.0f : 7.0f;
        const float q = clampf(rne(w * p.r), -Q, Q);
        *wh = q * p.s;
        return (uint32_t)(int)q & (f == CHAM_W_INT8_SYM ? 0xFFu : 0xFu);
    }
    case CHAM_W_INT8_ASYM:
    case CHAM_W_INT4_ASYM: {
        const float L = f == CHAM_W_INT8_ASYM ? 255.0f : 15.0f;
        const float q = clampf(rne(w * p.r) + p.z, 0.0f, L);
        *wh = (q - p.z) * p.s;
        return (uint32_t)q;
    }
    case CHAM_W_FP4: {
        float e;
        const uint32_t c = e2m1_encode(clampf(w * p.r, -6.0f, 6.0f), &e);
        *wh = e * p.s;
        return c;
    }
    case CHAM_W_NF4: {
        const uint32_t c = nf4_encode(w * p.r);
        *wh = nf4_level(c) * p.s;
        return c;
    }
    case CHAM_W_MXINT8:
    case CHAM_W_MXINT4: {
        const int E = (int)p.z, F = f == CHAM_W_MXINT8 ? 6 : 2;
        const float Q = f == CHAM_W_MXINT8 ? 127.0f : 7.0f;
        const float k = clampf(rne(ldexpf(w, F - E)), -Q, Q);
        *wh = ldexpf(k, E - F);
        return (uint32_t)(int)k & (f == CHAM_W_MXINT8 ? 0xFFu : 0xFu);
    }
    default: {  // MXFP4
        const int E = (int)p.z;
        float e;
        const uint32_t c = e2m1_encode(clampf(ldexpf(w, -E), -6.0f, 6.0f), &e);
        *wh = ldexpf(e, E);
        return c;
    }
    }
}

struct GSArgs {
    int waves;            // channels (wavefronts) per workgroup
    const float* W;
    const float* energy;  // [K]
    int N, K;
    uint32_t mask, gmask;
    int code_bits;
    double* part;          // [kTuples][workgroups] weighted error sums (workspace)
    const int32_t* choice; // emit: {g, f}
    uint8_t* fmt;
    uint8_t* codes;
    float* gscale;
    float* gzero;
    uint8_t* e8;
};

// Groups of all sizes of a row, flattened: those of size kGroupSizes[gi] start at
// group_base(K, gi).  Those of size 32 come first and are the blocks the others are folded from.
__host__ __device__ inline int group_base(int K, int gi) {
    int b = 0;
    for (int i = 0; i < gi; ++i) b += (K + kGroupSizes[i] - 1) / kGroupSizes[i];
    return b;
}

// LDS of one wavefront: its row (K floats), the groups' parameters (4 floats each) and the
// groups' extrema (2 floats each); a multiple of 16 bytes, as is each part.
__host__ __device__ inline int wave_lds_floats(int K) { return (K + 6 * group_base(K, CHAM_NGROUPS) + 3) & ~3; }

CHAM_DEV void wave_lds_fence() {
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

constexpr int kStageLoads = 5;  // 16-byte loads in flight per lane

// Row of channel n (16-byte aligned, K % 32 == 0) into LDS, and the extrema of its 32-blocks:
// 8 consecutive lanes hold one block, all active or none.
CHAM_DEV void stage_row(const GSArgs& a, int n, float* row, float2* ext) {
    const int lane = threadIdx.x & 63;
    const float4* src = reinterpret_cast<const float4*>(a.W + (int64_t)n * a.K);
    for (int q0 = lane; q0 < a.K / 4; q0 += 64 * kStageLoads) {
        float4 v[kStageLoads];
#pragma unroll
        for (int i = 0; i < kStageLoads; ++i)
            if (q0 + 64 * i < a.K / 4) v[i] = src[q0 + 64 * i];
#pragma unroll
        for (int i = 0; i < kStageLoads; ++i) {
            const int q = q0 + 64 * i;
            if (q >= a.K / 4) continue;
            reinterpret_cast<float4*>(row)[q] = v[i];
            float lo = fminf(fminf(v[i].x, v[i].y), fminf(v[i].z, v[i].w));
            float hi = fmaxf(fmaxf(v[i].x, v[i].y), fmaxf(v[i].z, v[i].w));
            lo = fminf(lo, dpp<0xB1>(lo));
            hi = fmaxf(hi, dpp<0xB1>(hi));
            lo = fminf(lo, dpp<0x4E>(lo));
            hi = fmaxf(hi, dpp<0x4E>(hi));
            lo = fminf(lo, dpp<0x141>(lo));
            hi = fmaxf(hi, dpp<0x141>(hi));
            if ((q & 7) == 0) ext[q >> 3] = make_float2(lo, hi);
        }
    }
}

// extrema of the group of g consecutive channels starting at block b0 (the row's last group
// may be short)
CHAM_DEV float2 fold_blocks(const float2* ext, int b0, int g, int nblk) {
    float2 m = ext[b0];
    const int b1 = min(b0 + g / 32, nblk);
    for (int b = b0 + 1; b < b1; ++b) {
        const float2 v = ext[b];
        m.x = fminf(m.x, v.x);
        m.y = fmaxf(m.y, v.y);
    }
    return m;
}

// d = w - w^ of four consecutive weights of one group: group_quant's binary32 steps, the
// E2M1 rounding by the hardware converters and the NF4 level through its cell (exact).
template <int F>
CHAM_DEV void group_diff4(const float (&w)[4], const GParam& p, const NF4Cell* cells, float (&d)[4]) {
    if (F == CHAM_W_FP4) {
        float y[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = __builtin_amdgcn_fmed3f(w[j] * p.r, -6.0f, 6.0f);
        v2f lo, hi;
        fp4_quad(y[0], y[1], y[2], y[3], 1.0f, 0u, lo, hi);
        d[0] = w[0] - lo.x * p.s;
        d[1] = w[1] - lo.y * p.s;
        d[2] = w[2] - hi.x * p.s;
        d[3] = w[3] - hi.y * p.s;
        return;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (F == CHAM_W_INT4_ASYM || F == CHAM_W_INT8_ASYM) {
            const float q = __builtin_amdgcn_fmed3f(rne(w[j] * p.r) + p.z, 0.0f, F == CHAM_W_INT4_ASYM ? 15.0f : 255.0f);
            d[j] = w[j] - (q - p.z) * p.s;
        } else if (F == CHAM_W_NF4) {
            const float y = w[j] * p.r;
            const NF4Cell& c = cells[min((uint32_t)(int)__builtin_fmaf(y, 16.0f, 16.0f), 32u)];
            d[j] = w[j] - (y > c.thr ? c.vhi : c.vlo) * p.s;
        } else {
            float wh;
            (void)group_quant(F, w[j], p, &wh);
            d[j] = w[j] - wh;
        }
    }
}

// Weighted errors of format F at every enabled group size: sums over this channel into the
// wavefront's slots tot[gi * CHAM_W_NFMT + F].
template <int F>
CHAM_DEV void format_errors(const GSArgs& a, const float* row, const float2* ext, float4* gp, const NF4Cell* cells,
                            double* tot) {
    constexpr int NG = F == CHAM_W_MXINT8 || F == CHAM_W_MXINT4 || F == CHAM_W_MXFP4 ? 1 : CHAM_NGROUPS;
    const int lane = threadIdx.x & 63, K = a.K;
    const int G = group_base(K, NG);
    for (int j = lane; j < G; j += 64) {
        const float2 m = ext[j];
        const GParam p = group_param(F, m.x, m.y);
        gp[j] = make_float4(p.s, p.r, p.z, 0.0f);
    }
    wave_lds_fence();
    int base[NG];
    double e[NG];
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
        base[gi] = group_base(K, gi);
        e[gi] = 0.0;
    }
    for (int k0 = 4 * lane; k0 < K; k0 += 256) {
        const float4 w4 = reinterpret_cast<const float4*>(row)[k0 >> 2];
        const float4 e4 = reinterpret_cast<const float4*>(a.energy)[k0 >> 2];
        const float w[4] = {w4.x, w4.y, w4.z, w4.w};
        const double ek[4] = {(double)e4.x, (double)e4.y, (double)e4.z, (double)e4.w};
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) {
            if (!((a.gmask >> gi) & 1u)) continue;
            // 4 consecutive elements share a group (sizes are multiples of 4)
            const float4 q = gp[base[gi] + k0 / kGroupSizes[gi]];
            float d[4];
            group_diff4<F>(w, GParam{q.x, q.y, q.z}, cells, d);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // d d and ek d are exact in binary64, so this is fma(ek, d d, e) to the bit
                const double dj = (double)d[j];
                e[gi] = fma(ek[j] * dj, dj, e[gi]);
            }
        }
    }
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) e[gi] = wave_sum(e[gi]);
    if (lane == 0) {
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) tot[gi * CHAM_W_NFMT + F] = e[gi];
    }
    wave_lds_fence();  // gp is reused by the next format
}

// (1) weighted errors of every enabled tuple, summed over the workgroup's channels.
// Bound by VALU: per weight and tuple about 7 binary32 steps, a conversion and two binary64
// operations.  A format is one pass over the row in LDS that serves all group sizes, so a
// weight, its energy and the address work are read and done once for five tuples, and the
// group parameters come from block extrema reduced in registers.  4608 x 1152, 15 tuples:
// 47.7 us; a pass per tuple with the extrema scanned from LDS, all lanes on one bank, and 15
// comparisons per NF4 code took 339.
__global__ __launch_bounds__(64 * kGWaves) void gsearch_err_kernel(GSArgs a) {
    extern __shared__ __align__(16) float lds[];
    __shared__ NF4Cell cells[33];
    __shared__ double tot[kGWaves][kTuples];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = blockIdx.x * a.waves + wave;
    const int K = a.K;
    // of the 64-thread workgroups of long rows all threads take part
    nf4_cells_init(cells);
    for (int t = lane; t < kTuples; t += 64) tot[wave][t] = 0.0;
    __syncthreads();
    if (n < a.N) {  // wavefront-uniform
        float* row = lds + wave * wave_lds_floats(K);
        const int G = group_base(K, CHAM_NGROUPS);
        float4* gp = reinterpret_cast<float4*>(row + K);
        float2* ext = reinterpret_cast<float2*>(gp + G);
        stage_row(a, n, row, ext);
        wave_lds_fence();
        const int nblk = K / 32;
        for (int j = nblk + lane; j < G; j += 64) {
            int gi = 1;
            int b = nblk;
#pragma unroll
            for (int i = 1; i + 1 < CHAM_NGROUPS; ++i)
                if (j >= group_base(K, i + 1)) { gi = i + 1; b = group_base(K, i + 1); }
            int g = kGroupSizes[1];
#pragma unroll
            for (int i = 2; i < CHAM_NGROUPS; ++i) g = gi == i ? kGroupSizes[i] : g;
            ext[j] = fold_blocks(ext, (j - b) * (g / 32), g, nblk);
        }
        wave_lds_fence();
        double* t = tot[wave];
        if ((a.mask >> CHAM_W_INT8_SYM) & 1u) format_errors<CHAM_W_INT8_SYM>(a, row, ext, gp, cells, t);
        if ((a.mask >> CHAM_W_INT8_ASYM) & 1u) format_errors<CHAM_W_INT8_ASYM>(a, row, ext, gp, cells, t);
        if ((a.mask >> CHAM_W_INT4_SYM) & 1u) format_errors<CHAM_W_INT4_SYM>(a, row, ext, gp, cells, t);
        if ((a.mask >> CHAM_W_INT4_ASYM) & 1u) format_errors<CHAM_W_INT4_ASYM>(a, row, ext, gp, cells, t);
        if ((a.mask >> CHAM_W_NF4) & 1u) format_errors<CHAM_W_NF4>(a, row, ext, gp, cells, t);
        if ((a.mask >> CHAM_W_FP4) & 1u) format_errors<CHAM_W_FP4>(a, row, ext, gp, cells, t);
        if (a.gmask & 1u) {  // MX formats: their own 32-blocks only
            if ((a.mask >> CHAM_W_MXINT8) & 1u) format_errors<CHAM_W_MXINT8>(a, row, ext, gp, cells, t);
            if ((a.mask >> CHAM_W_MXINT4) & 1u) format_errors<CHAM_W_MXINT4>(a, row, ext, gp, cells, t);
            if ((a.mask >> CHAM_W_MXFP4) & 1u) format_errors<CHAM_W_MXFP4>(a, row, ext, gp, cells, t);
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kTuples; t += 64 * a.waves) {
        double s = tot[0][t];
        for (int w = 1; w < a.waves; ++w) s += tot[w][t];
        a.part[(int64_t)t * gridDim.x + blockIdx.x] = s;
    }
}

// (2) layer error of each tuple (partials added in a fixed order) and the choice; one
// wavefront per tuple, the tuple's partials consecutive (1152 of them: 8.3 us; one partial
// per channel, its tuples together, read by four wavefronts: 85)
constexpr int kSelThreads = 1024;

__global__ __launch_bounds__(kSelThreads) void gsearch_select_kernel(const double* part, int P, uint32_t mask,
                                                                     uint32_t gmask, int32_t* choice, double* err_out) {
    __shared__ double tot[kTuples];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int t = wave; t < kTuples; t += kSelThreads / 64) {
        const int gi = t / CHAM_W_NFMT, f = t % CHAM_W_NFMT;
        const bool on = ((gmask >> gi) & 1u) && ((mask >> f) & 1u) && !(mx_fmt(f) && kGroupSizes[gi] != 32);
        double s = 0.0;
        if (on) {
            const double* p = part + (int64_t)t * P;
#pragma unroll 8
            for (int i = lane; i < P; i += 64) s += p[i];
        }
        s = wave_sum(s);
        if (lane == 0) tot[t] = on ? s : -1.0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int best = -1;
        for (int t = 0; t < kTuples; ++t)
            if (tot[t] >= 0.0 && (best < 0 || tot[t] < tot[best])) best = t;
        choice[0] = best >= 0 ? kGroupSizes[best / CHAM_W_NFMT] : 0;
        choice[1] = best >= 0 ? best % CHAM_W_NFMT : CHAM_W_NFMT;
    }
    if (err_out)
        for (int t = threadIdx.x; t < kTuples; t += kSelThreads) err_out[t] = tot[t];
}

// codes of a row in LDS, 4 per lane and store
template <int F>
CHAM_DEV void emit_codes(const GSArgs& a, int n, int g, const float* row, const float4* gp, const NF4Cell* cells) {
    const int lane = threadIdx.x & 63, K = a.K;
    for (int k0 = 4 * lane; k0 < K; k0 += 256) {
        const float4 w4 = reinterpret_cast<const float4*>(row)[k0 >> 2];
        const float4 q = gp[k0 / g];
        const GParam p{q.x, q.y, q.z};
        const float w[4] = {w4.x, w4.y, w4.z, w4.w};
        uint32_t cw = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t c;
            if (F == CHAM_W_NF4) {
                const float y = w[j] * p.r;
                const NF4Cell& cl = cells[min((uint32_t)(int)__builtin_fmaf(y, 16.0f, 16.0f), 32u)];
                c = cl.cnt + (y > cl.thr ? 1u : 0u);
            } else {
                float wh;
                c = group_quant(F, w[j], p, &wh);
            }
            cw |= a.code_bits == 4 ? (c & 15u) << (4 * j) : (c & 255u) << (8 * j);
        }
        if (a.code_bits == 4) reinterpret_cast<uint16_t*>(a.codes + (int64_t)n * (K / 2))[k0 >> 2] = (uint16_t)cw;
        else reinterpret_cast<uint32_t*>(a.codes + (int64_t)n * K)[k0 >> 2] = cw;
    }
}

// (3) codes and group metadata of the chosen tuple (4608 x 1152: 8.3 us; 20.7 with each
// group's extrema scanned by one lane)
__global__ __launch_bounds__(64 * kGWaves) void gsearch_emit_kernel(GSArgs a) {
    extern __shared__ __align__(16) float lds[];
    __shared__ NF4Cell cells[33];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = blockIdx.x * a.waves + wave;
    nf4_cells_init(cells);
    __syncthreads();
    if (n >= a.N) return;
    const int K = a.K;
    const int g = a.choice[0], f = a.choice[1];
    if (f >= CHAM_W_NFMT || g < 32) return;  // nothing was selected (non-finite weights)
    float* row = lds + wave * wave_lds_floats(K);
    float4* gp = reinterpret_cast<float4*>(row + K);
    float2* ext = reinterpret_cast<float2*>(gp + group_base(K, CHAM_NGROUPS));
    stage_row(a, n, row, ext);
    wave_lds_fence();
    const int G = (K + g - 1) / g, nblk = K / 32;
    const bool mx = mx_fmt(f);
    for (int j = lane; j < nblk; j += 64) {
        GParam p{0.0f, 0.0f, 0.0f};
        if (j < G) {
            const float2 m = fold_blocks(ext, j * (g / 32), g, nblk);
            p = group_param(f, m.x, m.y);
            gp[j] = make_float4(p.s, p.r, p.z, 0.0f);
        }
        a.gscale[(int64_t)n * nblk + j] = mx || j >= G ? 0.0f : p.s;
        a.gzero[(int64_t)n * nblk + j] = mx || j >= G ? 0.0f : p.z;
        if (a.e8) a.e8[(int64_t)n * nblk + j] = mx ? (uint8_t)((int)p.z + 127) : (uint8_t)0;
    }
    wave_lds_fence();
    if (lane == 0) a.fmt[n] = (uint8_t)f;
    switch (f) {
    case CHAM_W_INT8_SYM: emit_codes<CHAM_W_INT8_SYM>(a, n, g, row, gp, cells); break;
    case CHAM_W_INT8_ASYM: emit_codes<CHAM_W_INT8_ASYM>(a, n, g, row, gp, cells); break;
    case CHAM_W_INT4_SYM: emit_codes<CHAM_W_INT4_SYM>(a, n, g, row, gp, cells); break;
    case CHAM_W_INT4_ASYM: emit_codes<CHAM_W_INT4_ASYM>(a, n, g, row, gp, cells); break;
    case CHAM_W_NF4: emit_codes<CHAM_W_NF4>(a, n, g, row, gp, cells); break;
    case CHAM_W_FP4: emit_codes<CHAM_W_FP4>(a, n, g, row, gp, cells); break;
    case CHAM_W_MXINT8: emit_codes<CHAM_W_MXINT8>(a, n, g, row, gp, cells); break;
    case CHAM_W_MXINT4: emit_codes<CHAM_W_MXINT4>(a, n, g, row, gp, cells); break;
    default: emit_codes<CHAM_W_MXFP4>(a, n, g, row, gp, cells); break;
    }
}

// ---- per-input-channel sums of squares: partials over row chunks, then a fixed-order sum
constexpr int kColChunks = 64;
constexpr int kColWaves = 4;  // wavefronts per workgroup: 64 channels each, every kColWaves-th row

// Bound by memory: 64 chunks of rows x blocks of 64 channels, so an ordinary layer has over a
// thousand workgroups, each wavefront with 8 rows in flight.  8192 x 1152: 7.6 us (5 TB/s);
// one row in flight per thread and 320 workgroups took 34.6.
__global__ __launch_bounds__(64 * kColWaves) void colsq_partial_kernel(const float* X, int64_t M, int K, double* part) {
    __shared__ double sh[kColWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + lane;
    const int c = blockIdx.y;
    const int64_t m0 = M * c / kColChunks, m1 = M * (c + 1) / kColChunks;
    double s = 0.0;
    if (k < K) {
        int64_t m = m0 + wave;
        for (; m + 7 * kColWaves < m1; m += 8 * kColWaves) {
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = X[(m + i * kColWaves) * K + k];
#pragma unroll
            for (int i = 0; i < 8; ++i) s = fma((double)x[i], (double)x[i], s);
        }
        for (; m < m1; m += kColWaves) {
            const double x = (double)X[m * K + k];
            s = fma(x, x, s);
        }
    }
    sh[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && k < K) {
#pragma unroll
        for (int w = 1; w < kColWaves; ++w) s += sh[w][lane];
        part[(int64_t)c * K + k] = s;
    }
}

// 64 channels per workgroup; each wavefront adds its share of the chunks with every load in
// flight, the wavefronts in order
__global__ __launch_bounds__(64 * kColWaves) void colsq_sum_kernel(const double* part, int K, double* colsq) {
    __shared__ double sh[kColWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + lane;
    constexpr int per = kColChunks / kColWaves;
    const double old = wave == 0 && k < K ? colsq[k] : 0.0;
    double s = 0.0;
    if (k < K) {
        double v[per];
#pragma unroll
        for (int i = 0; i < per; ++i) v[i] = part[(int64_t)(wave * per + i) * K + k];
#pragma unroll
        for (int i = 0; i < per; ++i) s += v[i];
    }
    sh[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && k < K) {
        s = old + s;
#pragma unroll
        for (int w = 1; w < kColWaves; ++w) s += sh[w][lane];
        colsq[k] = s;
    }
}

}  // namespace
}  // namespace cham

using namespace cham;

int cham_pack_grouped(const cham_gwq* gq, hipStream_t s);  // the GEMM's record pre-pass

// wavefronts per workgroup so that their rows and group parameters fit kGLdsMax (one's do up to
// the largest K, 8192)
static int gsearch_waves(int64_t K) {
    const size_t per = (size_t)wave_lds_floats((int)K) * 4;
    return (int)std::max<size_t>(1, std::min<size_t>(kGWaves, kGLdsMax / per));
}

// at most one workgroup, with a partial sum per tuple, per channel
size_t cham_gselect_workspace_bytes(int64_t N) { return N > 0 ? (size_t)N * kTuples * sizeof(double) : 0; }
size_t cham_colsq_workspace_bytes(int64_t K) { return K > 0 ? (size_t)kColChunks * (size_t)K * sizeof(double) : 0; }

extern "C" int cham_select_group_formats(const float* W, const float* energy, cham_gwq* gq, void* ws, size_t ws_bytes,
                                         void* stream) {
    if (!W || !energy || !gq) return CHAM_EINVAL;
    const uint32_t mask = gq->palette_mask, gmask = gq->group_mask;
    if (mask == 0u || (mask >> CHAM_W_NFMT) != 0u || gmask == 0u || (gmask >> CHAM_NGROUPS) != 0u) return CHAM_EFORMAT;
    const uint32_t mxm = (1u << CHAM_W_MXINT8) | (1u << CHAM_W_MXINT4) | (1u << CHAM_W_MXFP4);
    if ((mask & ~mxm) == 0u && !(gmask & 1u)) return CHAM_EFORMAT;  // MX formats only, without g = 32
    if (gq->N < 1 || gq->K < 1 || gq->N > (int64_t)INT32_MAX - kGWaves) return CHAM_EINVAL;
    const int64_t K = gq->K;
    if (K % 32 != 0 || K > 8192) return CHAM_ESHAPE;
    if (!gq->choice || !gq->fmt || !gq->codes || !gq->gscale || !gq->gzero) return CHAM_EINVAL;
    if ((mask & mxm) && !gq->e8m0) return CHAM_EINVAL;
    if (((uintptr_t)W & 15u) || ((uintptr_t)energy & 15u) || ((uintptr_t)gq->codes & 3u)) return CHAM_EINVAL;
    const int code_bits = (mask & 0x7u) ? 8 : 4;
    if (gq->packed) {
        if (code_bits != 4 || K % 64 != 0) return CHAM_ESHAPE;  // the GEMM layout: 4-bit codes, 64-wide k-steps
        if (((uintptr_t)gq->packed & 255u) || gq->N * (K / 64) * 128 > (int64_t)INT32_MAX) return CHAM_EINVAL;
    }
    if (!ws || ws_bytes < cham_gselect_workspace_bytes(gq->N)) return CHAM_EWORKSPACE;
    gq->code_bits = code_bits;
    hipStream_t s = (hipStream_t)stream;
    GSArgs a;
    a.W = W;
    a.energy = energy;
    a.N = (int)gq->N;
    a.K = (int)K;
    a.mask = mask;
    a.gmask = gmask;
    a.code_bits = code_bits;
    a.part = (double*)ws;
    a.choice = gq->choice;
    a.fmt = gq->fmt;
    a.codes = gq->codes;
    a.gscale = gq->gscale;
    a.gzero = gq->gzero;
    a.e8 = (mask & mxm) ? gq->e8m0 : nullptr;
    a.waves = gsearch_waves(K);
    const dim3 grid((unsigned)((gq->N + a.waves - 1) / a.waves)), block((unsigned)(64 * a.waves));
    const size_t lds = (size_t)a.waves * (size_t)wave_lds_floats((int)K) * 4;
    hipLaunchKernelGGL(gsearch_err_kernel, grid, block, lds, s, a);
    CHAM_CHECK_LAUNCH();
    hipLaunchKernelGGL(gsearch_select_kernel, dim3(1), dim3(kSelThreads), 0, s, (const double*)ws, (int)grid.x, mask,
                       gmask, gq->choice, gq->err);
    CHAM_CHECK_LAUNCH();
    hipLaunchKernelGGL(gsearch_emit_kernel, grid, block, lds, s, a);
    CHAM_CHECK_LAUNCH();
    if (gq->packed) return cham_pack_grouped(gq, s);
    return CHAM_OK;
}

extern "C" int cham_act_colsq_accumulate(const float* X, int64_t M, int64_t K, double* colsq, void* ws, size_t ws_bytes,
                                         void* stream) {
    if (!X || !colsq || M < 1 || K < 1 || K > INT32_MAX) return CHAM_EINVAL;
    if (!ws || ws_bytes < cham_colsq_workspace_bytes(K)) return CHAM_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    const unsigned bx = (unsigned)((K + 63) / 64);
    hipLaunchKernelGGL(colsq_partial_kernel, dim3(bx, kColChunks), dim3(64 * kColWaves), 0, s, X, M, (int)K, (double*)ws);
    CHAM_CHECK_LAUNCH();
    hipLaunchKernelGGL(colsq_sum_kernel, dim3(bx), dim3(64 * kColWaves), 0, s, (const double*)ws, (int)K, colsq);
    CHAM_CHECK_LAUNCH();
    return CHAM_OK;
}
