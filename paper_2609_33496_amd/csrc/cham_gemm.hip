// Mixed-format linear layer: Y = DQ(X codes) . DQ(W codes)^T with a per-output-channel
// weight format (Sec. 4.5) and one activation format per call (Sec. 4.3).
//
// Per-channel formats do not map onto one native MFMA operand type (Sec. 6), so the
// weights are brought to a common half-precision operand: base value (NF4 level, E2M1 value,
// integer, q - z) times the block factor (NF4 block absmax, MX 2^E) relative to the channel's
// largest block, rounded to binary32 and then to half precision.  Integers, E2M1 values and MX
// mantissas are exact in half precision; NF4 levels times their block absmax carry the two
// roundings (relative error <= 2^-11 + 2^-24).  The packing pass decodes every weight once --
// 4-bit codes through a 16-entry table per (k-step of 64, channel, half) and v_perm_b32, 8-bit
// integers arithmetically (1024 + c trick, exact) -- into the lane layout of the MFMA operand
// (cham_records.h), 2 bytes per weight.  Decoding in the main loop instead (1.5 bytes per
// weight read, about 200 VALU instructions per k-step and wavefront beside 32 MFMAs) took
// 65.2 us on 2048 x 10240 x 1280 (now 55.8) and, with 8-bit codes, 153 us on
// 8192 x 4608 x 1152 (now 87).
//
// Activations are decoded to half precision while they are staged into LDS: per-tensor formats
// (INT8, E4M3, E5M2) exactly, MX formats relative to the largest block exponent of the row
// (3x3 convolution: of the pixels the tile gathers), which each workgroup finds in the
// exponent bytes first, once per tile column.  That adds 3 us to the MXFP8 product
// 8100 x 640 x 1920 (29.9 -> 32.9) and 5 to the convolution 1920 -> 640 at 2 x 32 x 32
// (49.8 -> 54.9); the pre-passes that wrote a half-precision copy instead took 13.7 and 38.8 us.
// On wide layers too the whole call is faster than with the pre-pass (and the weights' decode in
// the loop): 2048 x 10240 x 1280 70.6 -> 61.7 us with MXFP8, 70.0 -> 69.3 with MXINT8;
// 8192 x 10240 x 1280 244 -> 206 and 243 -> 222.
//
// Main kernel: 128 x 256, 128 x 128 or 64 x 128 output tiles; k-steps of 64; four wavefronts
// side by side that each own all the tile's rows x 32 TN channels (blocks of
// v_mfma_f32_32x32x16_f16, binary32 accumulation).  What bounds it: on long layers the matrix
// cores, at the clock that such a load leaves them (a 4096 x 4096 x 16384 product runs at 1273
// TFLOP/s with them busy 75 % of the cycles at 1.55 GHz; the library's dense f16 product, both
// operands in the memory order of k, at 1481 - 1572, busy 88 % at 1.51 GHz), on short ones the
// rounds of tiles that do not fill the chip and the output write.  Per k-step a 128 x 64
// wavefront block reads 16 KB from LDS and 8 KB from L1 for 1024 MFMA cycles per SIMD, about half
// of either's rate; the 128 x 32 block reads twice as much LDS per MFMA, and three of them per
// SIMD hide latency better.
// Weights go from memory straight to the operand registers (coalesced 16-byte buffer loads, a
// step or two ahead); activation tiles go global -> registers -> one of two LDS buffers, with
// their 16-byte chunks XOR-swizzled per row pair.  Barriers fence LDS only, so the loads in
// flight stay in flight across them.  Layers with too few output tiles to fill the
// CUs split k over several workgroups that write partial outputs, summed in split order
// by a second kernel; every output element is produced by plain stores (no atomics), so
// results do not depend on scheduling.
//
// The MFMA contracts over k in any order as long as both operands agree: lane half h of a
// k-step takes k = 32h .. 32h+31, sub-step s the 8 k at 32h + 8s.
#include <atomic>
#include <cmath>
#include <vector>

#include "cham_device.h"
#include "cham_group.h"
#include "cham_records.h"

namespace cham {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int BK = 64;
// TN = 32-channel MFMA blocks per wavefront, NW wavefronts side by side
constexpr int tile_width(int TN, int NW) { return 32 * TN * NW; }
// 16-byte chunks of a block of 32 channels in one k-step of the packed weights
constexpr int kBlockChunks = 256;
constexpr int kBufferFlags = 0x00020000;  // buffer descriptor word 3: 32-bit data, raw
constexpr int kStoreNonTemporal = 2;      // cache-policy operand of a buffer store: nt

// ------------------------------------------------------------------------------------
// weight decode
// ------------------------------------------------------------------------------------

// Look up 4 codes (one per byte, values 0..15); returns the low and high bytes.
CHAM_DEV void lookup4(const Table& t, uint32_t codes, uint32_t& lo, uint32_t& hi) {
    const uint32_t sel = codes & 0x07070707u;
    const uint32_t sel2 = 0x03020100u | ((codes >> 1) & 0x04040404u);
    const uint32_t l0 = __builtin_amdgcn_perm(t.lo[1], t.lo[0], sel);
    const uint32_t l1 = __builtin_amdgcn_perm(t.lo[3], t.lo[2], sel);
    const uint32_t h0 = __builtin_amdgcn_perm(t.hi[1], t.hi[0], sel);
    const uint32_t h1 = __builtin_amdgcn_perm(t.hi[3], t.hi[2], sel);
    lo = __builtin_amdgcn_perm(l1, l0, sel2);
    hi = __builtin_amdgcn_perm(h1, h0, sel2);
}

union H8 {
    half8 h;
    uint32_t u[4];
};

// 8 codes from a word of 8 nibbles
CHAM_DEV half8 decode_nibbles(const Table& t, uint32_t w) {
    uint32_t lo_e, hi_e, lo_o, hi_o;
    lookup4(t, w & 0x0F0F0F0Fu, lo_e, hi_e);         // k = 0, 2, 4, 6
    lookup4(t, (w >> 4) & 0x0F0F0F0Fu, lo_o, hi_o);  // k = 1, 3, 5, 7
    const uint32_t l01 = __builtin_amdgcn_perm(lo_o, lo_e, 0x05010400u);  // low bytes of k0..k3
    const uint32_t l23 = __builtin_amdgcn_perm(lo_o, lo_e, 0x07030602u);  // k4..k7
    const uint32_t h01 = __builtin_amdgcn_perm(hi_o, hi_e, 0x05010400u);
    const uint32_t h23 = __builtin_amdgcn_perm(hi_o, hi_e, 0x07030602u);
    H8 r;
    r.u[0] = __builtin_amdgcn_perm(h01, l01, 0x05010400u);
    r.u[1] = __builtin_amdgcn_perm(h01, l01, 0x07030602u);
    r.u[2] = __builtin_amdgcn_perm(h23, l23, 0x05010400u);
    r.u[3] = __builtin_amdgcn_perm(h23, l23, 0x07030602u);
    return r.h;
}

// 8 codes from two words of 4 byte-codes (4-bit formats in 8-bit layout)
CHAM_DEV half8 decode_bytes_table(const Table& t, uint32_t w0, uint32_t w1) {
    uint32_t lo0, hi0, lo1, hi1;
    lookup4(t, w0, lo0, hi0);
    lookup4(t, w1, lo1, hi1);
    H8 r;
    r.u[0] = __builtin_amdgcn_perm(hi0, lo0, 0x05010400u);
    r.u[1] = __builtin_amdgcn_perm(hi0, lo0, 0x07030602u);
    r.u[2] = __builtin_amdgcn_perm(hi1, lo1, 0x05010400u);
    r.u[3] = __builtin_amdgcn_perm(hi1, lo1, 0x07030602u);
    return r.h;
}

// 8-bit integer codes: value = fma((1024 + (c ^ x)) + a, f, b) in half precision, 1024 + c
// formed by placing c in the mantissa; x, a, f and b come from the table slot.
CHAM_DEV half8 decode_bytes_int(const Table& t, uint32_t w0, uint32_t w1) {
    w0 ^= t.lo[0];
    w1 ^= t.lo[0];
    H8 r;
    r.u[0] = __builtin_amdgcn_perm(0x64646464u, w0, 0x04010400u);
    r.u[1] = __builtin_amdgcn_perm(0x64646464u, w0, 0x04030402u);
    r.u[2] = __builtin_amdgcn_perm(0x64646464u, w1, 0x04010400u);
    r.u[3] = __builtin_amdgcn_perm(0x64646464u, w1, 0x04030402u);
    const half2v off = __builtin_bit_cast(half2v, t.lo[1]), fac = __builtin_bit_cast(half2v, t.lo[2]),
                 off2 = __builtin_bit_cast(half2v, t.lo[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        half2v v = __builtin_bit_cast(half2v, r.u[i]);
        v = __builtin_elementwise_fma(v + off, fac, off2);
        r.u[i] = __builtin_bit_cast(uint32_t, v);
    }
    return r.h;
}

// ------------------------------------------------------------------------------------
// packing pass: weights in half precision (layout in cham_records.h), a record per (k-step,
// channel, half k-step)
// ------------------------------------------------------------------------------------
struct RecArgs {
    const uint8_t* wfmt;
    const float* wscale;
    const float* wzero;
    const float* wnf4;
    const uint8_t* we8;
    const uint8_t* wc;
    uint32_t mask;
    int N, K, code_bits;
    int kchunk;  // k-steps per workgroup
    ColPrep* cols;
    float* colsum;  // [k-chunks][N] per workgroup chunk of k-steps: the sum of the channel's
                    // decoded weights (the GEMM adds the chunks in order)
    uint4* wh;      // half-precision weights [K/64][channel blocks][4][2][32] x 16 bytes
    // group-scaled weights (the DiT search): the chosen group size on the device (NULL: the
    // per-channel formats above), per-group scale / NF4 absmax and zero point [N][K/32]
    const int32_t* gsel;
    const float* gscale;
    const float* gzero;
};

// Workgroup b handles 32 channels (block b % nblk) and the k-steps of chunk b / nblk.
// 8 threads per channel compute its ColPrep (the reference exponent is the largest NF4
// block absmax or MX block exponent of the whole channel); thread t decodes the records of
// channel t % 32, half t / 32 % 2, at k-steps congruent to t / 64 mod 4, so each wavefront
// stores 1 KB in a row per sub-step.  The codes and block metadata of the thread's first
// kRecPrefetch records are loaded before the ColPrep pass, so both passes' loads are in
// flight together.
constexpr int kRecChannels = 32;
constexpr int kRecPrefetch = 3;

// Several weights' records in one launch: the workgroups of the batch's layers follow
// each other (descriptors in the kernel arguments); before them, one workgroup per entry
// of g groups a searched weight's channels by format (the search's grouping, run here when
// the search also packs the weights, to save a launch; first, so its longer serial work
// overlaps the records instead of trailing them).
constexpr int kRecBatchMax = 16;
struct RecBatch {
    int nl, ng;
    int wg_end[kRecBatchMax];  // record workgroups of layers 0..i
    RecArgs r[kRecBatchMax];
    GroupArgs g[kRecBatchMax];
};

__global__ __launch_bounds__(256) void record_kernel(RecBatch B) {
    __shared__ ColPrep cp[kRecChannels];
    if ((int)blockIdx.x < B.ng) {  // workgroup-uniform
        group_channels<256>(B.g[blockIdx.x], nullptr);
        return;
    }
    const int rb = (int)blockIdx.x - B.ng;  // record workgroup index
    int li = 0;
    while (li + 1 < B.nl && rb >= B.wg_end[li]) ++li;
    const RecArgs& a = B.r[li];
    const int bid = rb - (li ? B.wg_end[li - 1] : 0);
    const int t = threadIdx.x;
    const int K = a.K, nst = K / BK;
    const int nblk = (a.N + kRecChannels - 1) / kRecChannels;
    const int cb = bid % nblk, kc = bid / nblk;
    const int n0 = cb * kRecChannels;
    const int cw = a.code_bits / 4;  // 16-byte code pieces per half k-step
    const int64_t cstride = (int64_t)K * a.code_bits / 8;

    // this thread's records: channel n, half h, k-steps kb, kb + 4, ... below ke
    const int n = n0 + (t & 31), h = (t >> 5) & 1;
    const bool live = n < a.N;
    const int kb = kc * a.kchunk + (t >> 6), ke = min(nst, (kc + 1) * a.kchunk);
    const int gsz = a.gsel ? *a.gsel : 0;  // group size of group-scaled weights, else 0
    // block parameters of a record: NF4 absmax (or the group's scale / absmax) in nfa, the
    // group's zero point in gz, the MX exponent in e8
    auto load_rec = [&](int k, uint4 (&code)[2], float& nfa, float& gz, int& e8) __attribute__((always_inline)) {
        const uint4* src = reinterpret_cast<const uint4*>(a.wc + n * cstride + (int64_t)k * (16 * a.code_bits / 2) +
                                                          (int64_t)h * 16 * cw);
        code[0] = src[0];
        code[1] = cw > 1 ? src[1] : make_uint4(0u, 0u, 0u, 0u);
        if (gsz) {
            const int64_t j = (int64_t)n * (K / 32) + (64 * k + 32 * h) / gsz;
            nfa = a.gscale[j];
            gz = a.gzero[j];
        } else {
            nfa = a.wnf4 ? a.wnf4[(int64_t)n * (K / 64) + k] : 0.0f;
            gz = 0.0f;
        }
        e8 = a.we8 ? (int)a.we8[(int64_t)n * (K / 32) + 2 * k + h] : 0;
    };
    uint4 pc[kRecPrefetch][2];
    float pn[kRecPrefetch], pz[kRecPrefetch];
    int pe[kRecPrefetch];
#pragma unroll
    for (int i = 0; i < kRecPrefetch; ++i)
        if (live && kb + 4 * i < ke) load_rec(kb + 4 * i, pc[i], pn[i], pz[i], pe[i]);

    {
        const int ch = t >> 3, sub = t & 7;
        const int nn = n0 + ch;
        const int f = nn < a.N ? a.wfmt[nn] : CHAM_W_NFMT;
        // a group search of non-finite weights selects nothing (group size 0): no valid format
        const bool ok = f < CHAM_W_NFMT && ((a.mask >> f) & 1u) && !(a.gsel && gsz == 0);
        // the block metadata of every enabled kind is read without waiting for the format
        // (it is zero for channels of other formats), so these loads overlap the format load
        float mxf = 0.0f;
        int mxe = 0;
        if (nn < a.N && a.wnf4) {
            const float* r = a.wnf4 + (int64_t)nn * (K / 64);
#pragma unroll 4
            for (int b = sub; b < K / 64; b += 8) mxf = fmaxf(mxf, r[b]);
        }
        if (nn < a.N && a.we8) {
            const uint8_t* r = a.we8 + (int64_t)nn * (K / 32);
#pragma unroll 4
            for (int b = sub; b < K / 32; b += 8) mxe = max(mxe, (int)r[b]);
        }
        if (gsz && nn < a.N && ok && !is_mx(f)) {
            // group-scaled: the largest decoded magnitude over the channel's groups
            const int G = (K + gsz - 1) / gsz;
            const float* gs = a.gscale + (int64_t)nn * (K / 32);
            const float* gzr = a.gzero + (int64_t)nn * (K / 32);
            for (int j = sub; j < G; j += 8) {
                float m = gs[j];  // NF4: the group absmax
                if (f == CHAM_W_FP4) m = 6.0f * gs[j];
                else if (f == CHAM_W_INT4_SYM) m = 7.0f * gs[j];
                else if (f == CHAM_W_INT8_SYM) m = 127.0f * gs[j];
                else if (f == CHAM_W_INT4_ASYM || f == CHAM_W_INT8_ASYM) {
                    const float L = f == CHAM_W_INT4_ASYM ? 15.0f : 255.0f;
                    m = fmaxf(fabsf(gzr[j]), fabsf(L - gzr[j])) * gs[j];
                }
                mxf = fmaxf(mxf, m);
            }
        } else if (!(ok && f == CHAM_W_NF4)) {
            mxf = 0.0f;
        }
        if (!(ok && is_mx(f))) mxe = 0;
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) {
            mxf = fmaxf(mxf, __shfl_xor(mxf, o, kWave));
            mxe = max(mxe, __shfl_xor(mxe, o, kWave));
        }
        ColPrep c{CHAM_W_NFMT, 0, 0.0f, 0.0f};
        if (ok && gsz && !is_mx(f)) {
            // group-scaled: every table is relative to the channel's largest decoded magnitude
            c.fmt = f;
            c.eref = floor_log2(floor_scale(mxf)) - 14;
            c.colscale = ldexpf(1.0f, c.eref);
        } else if (ok) {
            c.fmt = f;
            c.zero = a.wzero ? a.wzero[nn] : 0.0f;  // group-scaled weights (an MX format here) have none
            if (f == CHAM_W_NF4) {
                // levels (|v| <= 1) times the block absmax over 2^eref stay below 2^15, and a
                // block 2^-28 below the largest is still a normal half-precision number
                c.eref = floor_log2(floor_scale(mxf)) - 14;
                c.colscale = ldexpf(1.0f, c.eref);
            } else if (is_mx(f)) {
                // element magnitudes up to 127 (MXINT8) times 2^8 stay below 2^15
                c.eref = mxe - 127 - mx_F(f) - 8;
                c.colscale = ldexpf(1.0f, c.eref);
            } else if (f == CHAM_W_INT8_ASYM || f == CHAM_W_INT4_ASYM) {
                c.eref = int_asym_eref(c.zero, f == CHAM_W_INT8_ASYM ? 255.0f : 15.0f);
                c.colscale = ldexpf(a.wscale[nn], c.eref);
            } else {
                c.colscale = a.wscale[nn];
            }
        }
        if (sub == 0) {
            cp[ch] = c;
            if (kc == 0 && nn < a.N) a.cols[nn] = c;
        }
    }
    __syncthreads();
    const ColPrep c = cp[t & 31];
    auto table = [&](float nfa, float gz, int e8) __attribute__((always_inline)) {
        return gsz && !is_mx(c.fmt) ? group_table(c, nfa, gz) : record_table(c, nfa, e8);
    };
    // decode the half k-step's 32 weights, store them (sub-step q's 8 at chunk (q, h, channel)
    // of the k-step's block: each wavefront's store is 1 KB in a row) and return their sum, the
    // half-precision values relative to colscale added by binary32 dot products
    const bool int8c = a.code_bits == 8 && is_8bit(c.fmt);
    auto store_rec = [&](int k, const uint4 (&code)[2], const Table& tb) __attribute__((always_inline)) {
        float sum = 0.0f;
        const half2v one = {(_Float16)1.0f, (_Float16)1.0f};
        uint4* dst = a.wh + ((int64_t)k * nblk + cb) * kBlockChunks + 32 * h + (t & 31);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            H8 v;
            if (a.code_bits == 4) {
                const uint32_t w = q == 0 ? code[0].x : q == 1 ? code[0].y : q == 2 ? code[0].z : code[0].w;
                v.h = decode_nibbles(tb, w);
            } else {
                const uint4& cc = code[q >> 1];
                const uint32_t w0 = (q & 1) ? cc.z : cc.x, w1 = (q & 1) ? cc.w : cc.y;
                v.h = int8c ? decode_bytes_int(tb, w0, w1) : decode_bytes_table(tb, w0, w1);
            }
            dst[64 * q] = make_uint4(v.u[0], v.u[1], v.u[2], v.u[3]);
#pragma unroll
            for (int r = 0; r < 4; ++r) sum = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2v, v.u[r]), one, sum, false);
        }
        return sum;
    };
    double psum = 0.0;
    if (live) {
#pragma unroll
        for (int i = 0; i < kRecPrefetch; ++i)
            if (kb + 4 * i < ke) {
                const Table tb = table(pn[i], pz[i], pe[i]);
                psum += (double)store_rec(kb + 4 * i, pc[i], tb);
            }
        for (int k = kb + 4 * kRecPrefetch; k < ke; k += 4) {
            uint4 code[2];
            float nfa, gz;
            int e8;
            load_rec(k, code, nfa, gz, e8);
            const Table tb = table(nfa, gz, e8);
            psum += (double)store_rec(k, code, tb);
        }
    }
    // the channel's sum over this workgroup's k-steps: its 8 threads (2 halves x 4 k-phases)
    // added in a fixed order, times the channel's scale
    __shared__ double part[4][64];
    part[t >> 6][t & 63] = psum;
    __syncthreads();
    if (t < kRecChannels && n0 + t < a.N) {
        double s2 = 0.0;
#pragma unroll
        for (int p = 0; p < 4; ++p) s2 += part[p][t] + part[p][t + 32];
        a.colsum[(int64_t)kc * a.N + n0 + t] = (float)(s2 * (double)cp[t].colscale);
    }
}

// Workgroup barrier that orders LDS accesses only: outstanding global loads (the
// prefetch) stay in flight.
CHAM_DEV void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ------------------------------------------------------------------------------------
// main kernel
// ------------------------------------------------------------------------------------
struct GemmArgs {
    const uint8_t* xc;       // [M][K] activation codes
    const uint8_t* xe8;      // [M][K/32] block exponents, MX activation formats
    const float* xs;         // activation scale per sample [M / rps] (per-tensor formats)
    const float* xz;         // activation zero point per sample
    int rps;                 // rows per sample
    const ColPrep* cols;     // [N]
    const float* colsum;     // [nkc][N] per k-chunk sums of the decoded weights
    int nkc;
    const uint4* wh;         // half-precision weights (layout in cham_records.h)
    float* Y;
    int M, N, K;
    int tn;          // tile columns
    int gm;          // tile rows per group of the XCD-aware tile order, 0: row-major (group_rows)
    int cached;      // 1: ordinary output stores, 0: non-temporal
    int splits;      // k-splits: workgroup b takes tile b % tiles and k-steps of split b / tiles
    int kchunk;      // k-steps per split
    float* part;     // splits > 1: [splits][M][N] partial outputs, summed by reduce_kernel
    // 3x3 convolution (implicit GEMM): xc is [B][H][W][C]; row m = (b, y, x) of the output,
    // k = (ky * 3 + kx) * C + c gathers pixel (y + ky - 1, x + kx - 1), zero past the borders
    int H, W, C;
};

CHAM_DEV constexpr bool mx_act(int af) { return af == CHAM_A_MXFP8_E4M3 || af == CHAM_A_MXINT8; }

// INT8-asym convolution: the power of two 2^-eref that keeps q - z within half precision's range
CHAM_DEV int far_eref(float z) {
    const float zm = fabsf(z) + 255.0f;
    return zm >= 32768.0f ? floor_log2(zm) - 14 : 0;
}

// largest of the bytes p[o0 .. o1), at most 16 (any alignment)
CHAM_DEV int max_bytes(const uint8_t* p, int o0, int o1) {
    int m = 0;
    if (o1 - o0 == 16) {
        uint32_t w[4];
        __builtin_memcpy(w, p + o0, 16);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            m = max(m, max(max((int)(w[i] & 0xFFu), (int)((w[i] >> 8) & 0xFFu)), max((int)((w[i] >> 16) & 0xFFu), (int)(w[i] >> 24))));
    } else {
        for (int o = o0; o < o1; ++o) m = max(m, (int)p[o]);
    }
    return m;
}

// What a staging row's codes are decoded with: INT8-asym -(1024 + zero point), MX the block's
// scale (MXINT8 as two half-precision powers of two).
struct ActDecode {
    half2v negz;
    float scale;
    half2v f1, f2;
};

// E8M0 byte e8 relative to a row whose largest is emax, ebias = 141 - emax: the block scale
// 2^(e8 - emax + 14) puts the largest block in [2^14, 2^15), so blocks down to 2^-28 of it stay
// normal in half precision.  Scales below 2^-126 only decode to zeros and are clamped there.
template <int AF>
CHAM_DEV ActDecode mx_decode(int e8, int ebias) {
    ActDecode d;
    const int b = max(e8 + ebias, 1);  // binary32 exponent field of the scale
    d.scale = __uint_as_float((uint32_t)b << 23);
    if (AF == CHAM_A_MXINT8) {  // 6 fraction bits; q 2^e1 is a normal half, times 2^e2 rounds once
        const int e = b - 127 - 6, e1 = max(e, -14), e2 = max(e - e1, -24);
        const _Float16 a = (_Float16)__uint_as_float((uint32_t)(e1 + 127) << 23);
        const _Float16 c = (_Float16)__uint_as_float((uint32_t)(e2 + 127) << 23);
        d.f1 = half2v{a, a};
        d.f2 = half2v{c, c};
    }
    return d;
}

// 8 activation codes (k0..k3 in w0, k4..k7 in w1) -> 8 halves in that order; exact for the
// per-tensor formats, rounded to half precision once (blocks far below the largest) for MX.
template <int AF>
CHAM_DEV uint4 decode_act8(uint32_t w0, uint32_t w1, const ActDecode& p) {
    // byte selectors of v_perm_b32(w1, w0, sel): 0..3 -> k0..k3, 4..7 -> k4..k7, 12 -> 0
    uint32_t d[4];
    if (AF == CHAM_A_FP8_E5M2) {  // E5M2 is the top byte of binary16
#pragma unroll
        for (int j = 0; j < 4; ++j)
            d[j] = __builtin_amdgcn_perm(w1, w0, 0x0Cu | ((uint32_t)(2 * j) << 8) | (0x0Cu << 16) | ((uint32_t)(2 * j + 1) << 24));
    } else if (AF == CHAM_A_FP8_E4M3 || AF == CHAM_A_MXFP8_E4M3) {  // hardware E4M3 -> binary16 conversion
        const float sc = AF == CHAM_A_FP8_E4M3 ? 1.0f : p.scale;
        d[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w0, sc, false));
        d[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w0, sc, true));
        d[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w1, sc, false));
        d[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w1, sc, true));
    } else {  // INT8-asym: (1024 + c) - (1024 + z); MXINT8: (1024 + (c ^ 128)) - 1152 = c, times the block scale
        const half2v off = AF == CHAM_A_MXINT8 ? half2v{(_Float16)-1152.0f, (_Float16)-1152.0f} : p.negz;
        if (AF == CHAM_A_MXINT8) {
            w0 ^= 0x80808080u;
            w1 ^= 0x80808080u;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t v = __builtin_amdgcn_perm(w1, w0, (uint32_t)(2 * j) | (0x0Cu << 8) | ((uint32_t)(2 * j + 1) << 16) | (0x0Cu << 24)) | 0x64006400u;
            half2v r = __builtin_bit_cast(half2v, v) + off;
            if (AF == CHAM_A_MXINT8) r = (r * p.f1) * p.f2;
            d[j] = __builtin_bit_cast(uint32_t, r);
        }
    }
    return make_uint4(d[0], d[1], d[2], d[3]);
}

// INT8-asym codes of the convolution whose zero point is beyond +-1024 or no integer (1024 + z
// would lose its fraction in half precision): q - z in binary32, times the power of two f that
// keeps it within half precision's range, rounded to half precision.
CHAM_DEV uint4 decode_act8_far(uint32_t w0, uint32_t w1, float z, float f) {
    uint32_t d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t w = (j < 2 ? w0 : w1) >> (16 * (j & 1));
        d[j] = half_pair2(((float)(w & 0xFFu) - z) * f, ((float)((w >> 8) & 0xFFu) - z) * f);
    }
    return make_uint4(d[0], d[1], d[2], d[3]);
}

// NW wavefronts side by side, each TM x TN blocks of 32 x 32 outputs; AF the activation format
// (CHAM_A_*), CONV the 3x3 convolution.
template <int TM, int TN, int NW, int AF, bool CONV>
__global__ __launch_bounds__(64 * NW, TM * TN >= 8 ? 2 : TM * TN >= 4 ? 3 : 4) void gemm_kernel(GemmArgs a) {
    constexpr int NT = 64 * NW;
    constexpr int BM = 32 * TM;
    constexpr int BN = tile_width(TN, NW);
    constexpr bool MX = mx_act(AF);
    constexpr bool INT8 = AF == CHAM_A_INT8_ASYM;
    constexpr bool CORR = INT8 && !CONV;                 // zero-point correction in the epilogue
    constexpr int AL = BM * 4;                           // 16-byte activation loads per k-step
    constexpr int AQ = AL / NT;                          // of them, per thread
    static_assert(AQ * NT == AL && NT % BM == 0, "every load falls inside the tile");
    constexpr int RSTEP = NT / 4;                        // rows between a thread's loads
    __shared__ uint4 lds[2][BM * 8];
    __shared__ __align__(16) float Rs[BM];
    __shared__ __align__(16) float Rc[CORR ? BM : 4];
    __shared__ int Re[MX ? (CONV ? NW : BM) : 1];        // largest block exponents

    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const int l32 = lane & 31, h = lane >> 5;
    const int K = a.K, N = a.N;
    // Workgroup -> (split, tile).  gm = 0: tiles in row-major order.  gm > 0, the XCD-aware
    // order: the dispatcher deals a launch's workgroups to the chip's 8 XCDs in turn (workgroup
    // b runs on XCD b % 8, as its (b / 8)-th), and each XCD has its own L2, so each XCD takes a
    // contiguous run of a logical order that walks groups of gm tile rows column by column.
    // Both maps are bijections of [0, grid), whatever the grid.
    const int mt = (a.M + BM - 1) / BM;
    const int tiles = mt * a.tn;
    const int G = (int)gridDim.x, b = (int)blockIdx.x, xcd = b & 7;
    const int lin = a.gm > 0 ? xcd * (G >> 3) + (xcd < (G & 7) ? xcd : (G & 7)) + (b >> 3) : b;
    const int tile = lin % tiles, split = lin / tiles;
    int m0, n0;
    if (a.gm > 0) {
        const int g0 = (tile / (a.gm * a.tn)) * a.gm;    // first tile row of the group
        const int gm = a.gm < mt - g0 ? a.gm : mt - g0;  // its tile rows (the last may be short)
        const int in = tile - g0 * a.tn;
        m0 = (g0 + in % gm) * BM;
        n0 = (in / gm) * BN;
    } else {
        m0 = (tile / a.tn) * BM;
        n0 = (tile % a.tn) * BN;
    }
    const int rows = a.M - m0 < BM ? a.M - m0 : BM;
    // k-steps [kb, kb + nsteps) of this workgroup; the operand bases below start at kb
    const int kb = split * a.kchunk;
    const int nsteps = K / BK - kb < a.kchunk ? K / BK - kb : a.kchunk;

    // per-row activation scale (the row's sample's s; MX: set below).
    // INT8-asym: codes are decoded as (1024 + c) - (1024 + z1) with z1 the sample's zero point
    // clamped to [-1024, 1024] (exact in half precision); the rest z - z1 (an integer, exact
    // in binary32) is taken out in the epilogue as -(z - z1) s times the channel's weight sum
    // (split 0 only).  The convolution's rows miss taps at the borders, so a zero point beyond
    // +-1024 is taken out while decoding there, rounded to half precision.
    for (int r = t; r < BM; r += NT) {
        const int m = r < rows ? m0 + r : m0;
        if (!MX) {
            Rs[r] = a.xs[m / a.rps];
            if (CORR) {
                const float za = a.xz[m / a.rps], z1 = clampf(za, -1024.0f, 1024.0f);
                Rc[r] = split == 0 ? -((za - z1) * a.xs[m / a.rps]) : 0.0f;
            }
            if (INT8 && CONV) Rs[r] = ldexpf(Rs[r], far_eref(a.xz[m / a.rps]));
        }
    }
    // the staging rows of this thread: their -(1024 + z1), or what far zero points take
    half2v negz[INT8 ? AQ : 1];
    float farz[INT8 && CONV ? AQ : 1], farf[INT8 && CONV ? AQ : 1];
    bool far = false;
#pragma unroll
    for (int i = 0; i < (INT8 ? AQ : 1); ++i) {
        negz[i] = half2v{(_Float16)0.0f, (_Float16)0.0f};
        if (INT8) {
            const int r = t / 4 + RSTEP * i;
            const int m = r < rows ? m0 + r : m0;
            const float za = a.xz[m / a.rps];
            const _Float16 nz = (_Float16)(-(1024.0f + clampf(za, -1024.0f, 1024.0f)));
            negz[i] = half2v{nz, nz};
            if (CONV) {
                farz[i] = za;
                farf[i] = ldexpf(1.0f, -far_eref(za));
                far |= fabsf(za) > 1024.0f || za != rne(za);
            }
        }
    }
    if (INT8 && CONV) far = __any(far);  // wavefront-uniform

    // ---- activation tile: global -> registers two k-steps ahead -> LDS, 16-byte loads
    // through a buffer resource whose range check returns zeros past the last row.  The
    // tile is stored as rows of 8 logical 16-byte chunks (8 k each), chunk c of row r at
    // slot c ^ ((r >> 1) & 7); load q = NT i + t is row q >> 2, codes 16 (q & 3) .. + 15 =
    // chunks 2 (q & 3), + 1.  MX: the exponent byte of the load's block comes with it.
    const int CK = CONV ? a.C : K;  // codes per row in memory
    const __amdgpu_buffer_rsrc_t ra =
        CONV ? __builtin_amdgcn_make_buffer_rsrc((void*)a.xc, (short)0, a.M * CK, kBufferFlags)
             : __builtin_amdgcn_make_buffer_rsrc((void*)(a.xc + (int64_t)m0 * K + kb * BK), (short)0, rows * K - kb * BK, kBufferFlags);
    const __amdgpu_buffer_rsrc_t re = __builtin_amdgcn_make_buffer_rsrc(
        MX ? (void*)(a.xe8 + (CONV ? 0 : (int64_t)m0 * (K / 32) + kb * 2)) : (void*)a.xc, (short)0,
        MX ? (CONV ? a.M * (CK / 32) : rows * (K / 32) - kb * 2) : 0, kBufferFlags);
    const uint32_t aoff0 = (uint32_t)((t / 4) * K + ((t & 3) << 4));
    // convolution: the offset of each staging row's pixel, and the taps that fall inside its image (none for
    // rows past the tile's last)
    int pix[CONV ? AQ : 1];
    uint32_t taps[CONV ? AQ : 1];
#pragma unroll
    for (int i = 0; i < (CONV ? AQ : 1); ++i) {
        pix[i] = 0;
        taps[i] = 0;
        const int r = t / 4 + RSTEP * i;
        if (CONV && r < rows) {
            const int m = m0 + r, x = m % a.W, y = m / a.W % a.H;
            pix[i] = m * a.C + ((t & 3) << 4);
#pragma unroll
            for (int q = 0; q < 9; ++q)
                if ((unsigned)(y + q / 3 - 1) < (unsigned)a.H && (unsigned)(x + q % 3 - 1) < (unsigned)a.W) taps[i] |= 1u << q;
        }
    }
    struct AStage {
        uint4 v[AQ];
        uint32_t e[AQ];  // MX: the block's exponent byte; INT8-asym convolution: the tap is inside
    };
    auto load_a = [&](AStage& S, int k) __attribute__((always_inline)) {
        int tap = 0, tapoff = 0;
        if (CONV) {  // k-step -> tap (ky, kx) and channel offset (C % 64 == 0)
            const int kk = (kb + k) * BK;
            tap = kk / a.C;
            const int ci0 = kk - tap * a.C;
            tapoff = ((tap / 3 - 1) * a.W + tap % 3 - 1) * a.C + ci0;
        }
#pragma unroll
        for (int i = 0; i < AQ; ++i) {
            uint32_t off;
            if (CONV) {  // outside the image: past both buffers, also as a block index
                const bool in = (taps[i] >> tap) & 1u;
                off = in ? (uint32_t)(pix[i] + tapoff) : 0x7FFFFFF0u;
                if (INT8) S.e[i] = in ? 1u : 0u;
            } else {
                off = aoff0 + (uint32_t)(i * RSTEP * K + k * BK);
            }
            S.v[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)off, 0, 0));
            if (MX) S.e[i] = __builtin_amdgcn_raw_buffer_load_b8(re, (int)(off >> 5), 0, 0);
        }
    };
    int ebias[MX ? AQ : 1];  // of the staging rows (mx_decode)
    auto store_a = [&](const AStage& S, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < AQ; ++i) {
            const int q = i * NT + t;
            const int r = q >> 2, c = 2 * (q & 3), sw = (r >> 1) & 7;
            uint4 d0, d1;
            if (INT8 && CONV && far) {
                d0 = decode_act8_far(S.v[i].x, S.v[i].y, farz[i], farf[i]);
                d1 = decode_act8_far(S.v[i].z, S.v[i].w, farz[i], farf[i]);
            } else {
                ActDecode p;
                if (MX) p = mx_decode<AF>((int)S.e[i], ebias[i]);
                p.negz = negz[INT8 ? i : 0];
                d0 = decode_act8<AF>(S.v[i].x, S.v[i].y, p);
                d1 = decode_act8<AF>(S.v[i].z, S.v[i].w, p);
            }
            if (INT8 && CONV && !S.e[i]) d0 = d1 = make_uint4(0u, 0u, 0u, 0u);  // the padding is 0, not the code 0
            lds[buf][r * 8 + (c ^ sw)] = d0;
            lds[buf][r * 8 + ((c + 1) ^ sw)] = d1;
        }
    };

    // ---- weights: the wave's TN blocks of 32 channels, straight from memory into the lane
    // layout of the MFMA operand (1 KB per block and sub-step, consecutive over the lanes).
    // Blocks past the last re-read the last one (their outputs are not stored).
    const int nblk = (N + 31) >> 5;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.wh + (int64_t)kb * nblk * kBlockChunks), (short)0, -1, kBufferFlags);
    const uint32_t wstep = (uint32_t)nblk * kBlockChunks * 16u;  // bytes per k-step
    uint32_t wblk[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int blk = (n0 >> 5) + wave * TN + j;
        wblk[j] = (uint32_t)__builtin_amdgcn_readfirstlane(blk < nblk ? blk : nblk - 1) * (kBlockChunks * 16u);
    }
    const int wlane = lane * 16;
    auto load_w = [&](half8 (&W)[TN], int k, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
            W[j] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(
                                                 rw, wlane, (int)((uint32_t)k * wstep + wblk[j] + 1024u * (uint32_t)s), 0));
    };

    // per-channel epilogue factor (loaded here, off the tail of the kernel)
    const int nl = 32 * TN * wave + l32;
    float cs[TN], csum[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 + nl + 32 * j;
        cs[j] = n < N ? a.cols[n].colscale : 0.0f;
        csum[j] = 0.0f;
        if (CORR && n < N)
            for (int q = 0; q < a.nkc; ++q) csum[j] += a.colsum[(int64_t)q * N + n];
    }

    // LDS chunk offset of the lane's activation operand in sub-step s (row l32 of block i
    // at + 256 i chunks)
    int aoff[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) aoff[s] = l32 * 8 + ((4 * h + s) ^ ((l32 >> 1) & 7));

    float16v acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // ---- main loop.  Step k computes from LDS buffer k & 1 in four sub-steps of 16 k.  Each
    // sub-step first issues its memory work -- the LDS reads of the activations LA sub-steps
    // ahead and the reload of the weight registers that the previous sub-step has just used,
    // with the same sub-step of step k + WD -- and then its MFMAs; scheduling barriers keep the
    // two apart, so a weight register is reloaded WD steps before its next use and needs no
    // second copy.  LA = 1: the activation tile of step k + 1 is decoded and stored to the
    // other buffer behind the MFMAs of sub-step 1, and one barrier before the last sub-step
    // makes it visible and retires every read of this step's buffer.  LA = 3 (tiles whose
    // sub-step is two MFMAs, shorter than an LDS read): the reads of step k + 1 start at
    // sub-step 1, behind the barrier, and the tile of step k + 2 is stored into this step's
    // buffer in sub-step 2.  Step indices past the end are clamped (harmless reloads).
    constexpr int LA = TM * TN <= 2 ? 3 : 1;
    constexpr int WD = TM * TN <= (CONV ? (INT8 ? 0 : 2) : AF == CHAM_A_MXINT8 ? 2 : 4) ? 2 : 1;  // as registers allow
    const int klast = nsteps - 1;
    AStage R[2];
    half8 fr[LA + 1][TM], W[WD][4][TN];
    auto read_a = [&](half8 (&f)[TM], int buf, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i) f[i] = __builtin_bit_cast(half8, lds[buf][i * 256 + aoff[s]]);
    };
    load_a(R[0], 0);
#pragma unroll
    for (int s = 0; s < 4; ++s) load_w(W[0][s], 0, s);
    load_a(R[1], 1 < klast ? 1 : klast);
    if (WD == 2) {
#pragma unroll
        for (int s = 0; s < 4; ++s) load_w(W[WD - 1][s], 1 < klast ? 1 : klast, s);
    }
    if (MX) {
        // the largest block exponent of each row over this split's k (convolution: of the pixels
        // that hold every neighbour of the tile's rows), behind the first loads
        if (CONV) {
            // one run of pixels; for long lines one run per tap line, so that the scan stays in
            // proportion to the tile (64 channels, 1 x 200000 pixels: 87.2 us with one run, 33.3
            // with three; 1 x 1000000: 1179 and 144).  Lines whose pixels take at most three
            // passes of the workgroup stay one run: three cost their latencies one after another
            // (512 x 512: 45.0 with one, 46.9 with three; 64 x 4096: 45.0 with either).
            const bool lines = a.W > rows + 2 && (a.W + 1) * (CK / 32) > 3 * 8 * NT;
            int mx = 0;
            for (int d = lines ? -1 : 0; d <= (lines ? 1 : 0); ++d) {
                const int c0 = m0 + d * a.W, ext = lines ? 1 : a.W + 1;
                const int p0 = max(c0 - ext, 0), p1 = min(c0 + rows + ext, a.M);
                const int e0 = p0 * (CK / 32), e1 = p1 * (CK / 32);
                for (int o = e0 + 16 * t; o < e1; o += 16 * NT) mx = max(mx, max_bytes(a.xe8, o, min(o + 16, e1)));
            }
            for (int o = 32; o > 0; o >>= 1) mx = max(mx, __shfl_xor(mx, o, kWave));
            if (lane == 0) Re[wave] = mx;
        } else {
            constexpr int TPR = NT / BM;  // threads per row, consecutive lanes
            const int r = t / TPR;
            const uint8_t* row = a.xe8 + (int64_t)(m0 + (r < rows ? r : 0)) * (K / 32) + kb * 2;
            int mx = 0;
            for (int o = 16 * (t % TPR); o < 2 * nsteps; o += 16 * TPR) mx = max(mx, max_bytes(row, o, min(o + 16, 2 * nsteps)));
#pragma unroll
            for (int o = 1; o < TPR; o <<= 1) mx = max(mx, __shfl_xor(mx, o, kWave));
            if (t % TPR == 0) Re[r] = mx;
        }
        lds_barrier();
        int tmax = 0;
        if (CONV) {
#pragma unroll
            for (int w = 0; w < NW; ++w) tmax = max(tmax, Re[w]);
        }
#pragma unroll
        for (int i = 0; i < (MX ? AQ : 1); ++i) ebias[i] = 141 - (CONV ? tmax : Re[t / 4 + RSTEP * i]);
        for (int r = t; r < BM; r += NT) Rs[r] = ldexpf(1.0f, (CONV ? tmax : Re[r]) - 141);
    }
    store_a(R[0], 0);
    if (LA == 3) {
        load_a(R[0], 2 < klast ? 2 : klast);
        store_a(R[1], 1);
    }
    lds_barrier();
#pragma unroll
    for (int s = 0; s < LA; ++s) read_a(fr[s], 0, s);

    auto step = [&](int k, int buf, AStage& Rn, AStage& Rl) __attribute__((always_inline)) {
        const int kw = k + WD < klast ? k + WD : klast;
        half8(&Wk)[4][TN] = W[WD == 2 ? buf : 0];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if (s == 4 - LA) lds_barrier();
            read_a(fr[(s + LA) % (LA + 1)], s + LA >= 4 ? buf ^ 1 : buf, (s + LA) & 3);
            if (s > 0) load_w(Wk[s - 1], kw, s - 1);
            if (s == 0) load_a(Rl, k + 1 + (LA + 1) / 2 < klast ? k + 1 + (LA + 1) / 2 : klast);
            __builtin_amdgcn_sched_barrier(0);
            if (LA == 1 && s == 1) store_a(Rn, buf ^ 1);
            if (LA == 3 && s == 2) store_a(Rn, buf);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fr[s % (LA + 1)][i], Wk[s][j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        load_w(Wk[3], kw, 3);
    };
    // LA = 1: step k stores R[(k + 1) & 1] (tile k + 1) and loads tile k + 2 into R[k & 1];
    // LA = 3: step k stores R[k & 1] (tile k + 2) and loads tile k + 3 into R[(k + 1) & 1]
    constexpr int RN = LA == 1 ? 1 : 0;
    int k = 0;
    for (; k + 2 <= nsteps; k += 2) {
        step(k, 0, R[RN], R[RN ^ 1]);
        step(k + 1, 1, R[RN ^ 1], R[RN]);
    }
    if (k < nsteps) step(k, 0, R[RN], R[RN ^ 1]);

    // ---- epilogue: 32x32 block, lane holds column l32, rows 8*(r/4) + 4*h + r%4; the
    // lane's 16 row scales of block i are 4 aligned float4 in LDS.  Stores go through a
    // buffer resource over the tile's rows of the output: the lane's offset is one VGPR per
    // block, each row's offset a wave-uniform SGPR, and the range check drops the rows past
    // the last of a ragged tile (the lane skips columns past the last).  The output is not
    // read again here, so it is stored non-temporally (the L2 stays with the operand tiles
    // other workgroups still read).  Ordinary stores: k-split partials, which the reduction
    // reads back at once, and outputs whose rows are not whole 128-byte lines (N % 32), where
    // each line comes in pieces that only the L2 can put together (2430 x 9119 x 704: 45.8 us
    // against 83.7 non-temporal).
    float* const out = a.splits > 1 ? a.part + (int64_t)split * a.M * N : a.Y;
    const __amdgpu_buffer_rsrc_t ro =
        __builtin_amdgcn_make_buffer_rsrc((void*)(out + (int64_t)m0 * N), (short)0, rows * N * 4, kBufferFlags);
    const bool cached = a.cached != 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        float rs[16], rc[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = *reinterpret_cast<const float4*>(&Rs[32 * i + 8 * q + 4 * h]);
            rs[4 * q] = v.x; rs[4 * q + 1] = v.y; rs[4 * q + 2] = v.z; rs[4 * q + 3] = v.w;
            if (CORR) {
                const float4 c = *reinterpret_cast<const float4*>(&Rc[32 * i + 8 * q + 4 * h]);
                rc[4 * q] = c.x; rc[4 * q + 1] = c.y; rc[4 * q + 2] = c.z; rc[4 * q + 3] = c.w;
            }
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int n = n0 + nl + 32 * j;
            if (n < N) {
                const int voff = ((32 * i + 4 * h) * N + n) * 4;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    // (acc rs) cs, plus the zero-point correction of INT8-asym activations
                    float v = (acc[i][j][r] * rs[r]) * cs[j];
                    if (CORR) v = v + rc[r] * csum[j];
                    const uint32_t bits = __builtin_bit_cast(uint32_t, v);
                    const int soff = (8 * (r >> 2) + (r & 3)) * N * 4;
                    if (cached) __builtin_amdgcn_raw_buffer_store_b32(bits, ro, voff, soff, 0);
                    else __builtin_amdgcn_raw_buffer_store_b32(bits, ro, voff, soff, kStoreNonTemporal);
                }
            }
        }
    }
}

// Sum of the k-split partial outputs in split order (the result does not depend on the
// order in which workgroups ran); 4 outputs per thread when M N is a multiple of 4.
constexpr int kMaxSplits = 8;
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void reduce_kernel(const float* __restrict__ part, float* __restrict__ Y,
                                                     int64_t MN, int splits) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if ((MN & 3) == 0) {
        const float4* p4 = reinterpret_cast<const float4*>(part);
        float4* y4 = reinterpret_cast<float4*>(Y);
        const int64_t n4 = MN >> 2;
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
            // every split's load issued before the first sum (splits <= kMaxSplits)
            float4 v[kMaxSplits];
#pragma unroll
            for (int sp = 0; sp < kMaxSplits; ++sp)
                v[sp] = sp < splits ? p4[(int64_t)sp * n4 + i] : make_float4(0.f, 0.f, 0.f, 0.f);
            float4 acc = v[0];
#pragma unroll
            for (int sp = 1; sp < kMaxSplits; ++sp) {
                if (sp < splits) { acc.x += v[sp].x; acc.y += v[sp].y; acc.z += v[sp].z; acc.w += v[sp].w; }
            }
            const f32x4 o = {acc.x, acc.y, acc.z, acc.w};
            __builtin_nontemporal_store(o, reinterpret_cast<f32x4*>(&y4[i]));
        }
    } else {
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < MN; i += stride) {
            float acc = part[i];
            for (int sp = 1; sp < splits; ++sp) acc += part[(int64_t)sp * MN + i];
            Y[i] = acc;
        }
    }
}

// ---- launch plan: one launch of one tile shape, optionally split along k into partial
// outputs that reduce_kernel sums (for layers with too few output tiles to fill the CUs).
// CU count of the current device, queried once per device (every thread that races to
// fill the cache stores the same value, so relaxed atomics suffice)
int cu_count() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Modeled time (us) of a launch of one tile shape: a fixed cost (prologue, tail), plus the
// k-steps of the rounds of workgroups, each at the k-step time of as many workgroups per CU as
// the round puts there -- the workgroups of later rounds start while earlier ones finish --
// plus the output.  The numbers are fitted to 1720 forced plans of per-tensor layers over 180
// shapes (M 200 - 8192, N 320 - 10240, K 640 - 5120) on MI355X, each timed behind its quantize call
// and again with the last-level cache swept by other data; there the planner's choice takes 1.0 %
// longer than the best of the forced plans on average, 15 % at worst.  MX activations and the
// convolution take the same plans although their staging costs more: over 49 shapes, two sets of
// operands in turn, the choice takes 0.7 (E4M3), 1.0 (INT8), 2.5 (MXFP8) and 3.1 % (MXINT8) longer
// than the best on average and 7, 12, 20 and 25 % at worst; over 9 convolutions 2.0 (MXFP8), 2.4
// (E4M3) and 5.5 % (INT8), 14 % at worst.  Tiles measured and not kept, as no shape ran faster in
// them: 256 x 256 (one wavefront per SIMD: 84 us against 56 on 2048 x 10240 x 1280), 64 x 256, and
// 128 x 128 and 64 x 128 of two wavefronts.
constexpr int kMaxOcc = 4;
struct TileCost {
    int tm, tn, nw, occ;   // 32-row blocks, 32-channel blocks per wavefront, wavefronts, workgroups per CU
    double step[kMaxOcc];  // us: k-step with 1 .. occ workgroups on the CU
    double fixed;          // us per launch
    int bm() const { return 32 * tm; }
    int bn() const { return tile_width(tn, nw); }
};
constexpr int kNumTiles = 3;
constexpr TileCost kTileCosts[kNumTiles] = {{4, 2, 4, 2, {0.812, 1.338}, 5.8},
                                            {4, 1, 4, 3, {0.476, 0.780, 1.200}, 5.1},
                                            {2, 1, 4, 4, {0.305, 0.527, 0.816, 1.121}, 4.2}};

int row_tiles(int M, const TileCost& c) { return (M + c.bm() - 1) / c.bm(); }
int col_tiles(int N, const TileCost& c) { return (N + c.bn() - 1) / c.bn(); }

double launch_cost(int64_t wgs, int nsteps, const TileCost& c, int P) {
    if (wgs <= 0) return 0.0;
    const int64_t slots = (int64_t)c.occ * P;
    const int64_t full = wgs / slots, rem = wgs % slots;
    return c.fixed + (double)full * nsteps * c.step[c.occ - 1] + (rem == 0 ? 0.0 : nsteps * c.step[(rem + P - 1) / P - 1]);
}

struct Plan {
    int tile;    // index into kTileCosts
    int splits;  // k-splits (1: none)
};
// The output write: 6.3 TB/s non-temporally.  k-split: one partial output per split, written
// (5.3 TB/s) and read back with the final write by one extra launch (11 TB/s: the partials come
// from the last-level cache in part), which costs 5 us itself.
double output_cost(int64_t M, int64_t N, int splits) {
    const double mb = (double)(M * N * 4) * 1e-6;
    return splits > 1 ? 5.03 + 0.187 * splits * mb + 0.089 * (splits + 1) * mb : 0.158 * mb;
}

Plan plan_gemm(int M, int N, int K) {
    const int P = cu_count();
    const int nsteps = K / BK;
    double best = 1e300;
    Plan plan{0, 1};
    for (int b = 0; b < kNumTiles; ++b) {
        const TileCost& c = kTileCosts[b];
        const int64_t tiles = (int64_t)row_tiles(M, c) * col_tiles(N, c);
        for (int sp = 1; sp <= kMaxSplits && sp <= nsteps; ++sp) {
            const int kchunk = (nsteps + sp - 1) / sp;
            if (sp > 1 && (sp - 1) * kchunk >= nsteps) continue;  // an empty split
            const double t = launch_cost(tiles * sp, kchunk, c, P) + output_cost(M, N, sp);
            if (t < best) { best = t; plan = Plan{b, sp}; }
        }
    }
    return plan;
}

// partial-output bytes of the plan for these sizes
size_t split_bytes(int64_t M, int64_t N, int64_t K) {
    const Plan p = plan_gemm((int)M, (int)N, (int)K);
    return p.splits > 1 ? (size_t)p.splits * (size_t)M * (size_t)N * 4 : 0;
}

template <int AF, bool CONV>
void launch_gemm_af(const GemmArgs& a, int tile, unsigned grid, hipStream_t s) {
    switch (tile) {
    case 0: hipLaunchKernelGGL((gemm_kernel<4, 2, 4, AF, CONV>), dim3(grid), dim3(256), 0, s, a); break;
    case 1: hipLaunchKernelGGL((gemm_kernel<4, 1, 4, AF, CONV>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((gemm_kernel<2, 1, 4, AF, CONV>), dim3(grid), dim3(256), 0, s, a); break;
    }
}

template <bool CONV>
void launch_gemm_fmt(const GemmArgs& a, int af, int tile, unsigned grid, hipStream_t s) {
    switch (af) {
    case CHAM_A_INT8_ASYM: launch_gemm_af<CHAM_A_INT8_ASYM, CONV>(a, tile, grid, s); break;
    case CHAM_A_FP8_E4M3: launch_gemm_af<CHAM_A_FP8_E4M3, CONV>(a, tile, grid, s); break;
    case CHAM_A_FP8_E5M2: launch_gemm_af<CHAM_A_FP8_E5M2, CONV>(a, tile, grid, s); break;
    case CHAM_A_MXFP8_E4M3: launch_gemm_af<CHAM_A_MXFP8_E4M3, CONV>(a, tile, grid, s); break;
    default: launch_gemm_af<CHAM_A_MXINT8, CONV>(a, tile, grid, s); break;
    }
}

// Tile rows per group of the XCD-aware order, 0 for the row-major one.  What decides is the
// order in which the output lines reach memory: with larger groups (8 - 16 rows, which read the
// fewest operand bytes) the tiles written at one time lie in many rows and a few columns, and a
// cold 8192 x 5120 x 640 took 78 - 93 us against 61 - 66 in groups of two rows; 8192 x 640 x 2560
// 44.4 against 37.3.  Row-major puts workgroup b on XCD b % 8 and tile column b % tn: where tn
// is a multiple of 8 each XCD keeps the same eighth of the weights in its L2 and whole rows are
// written at one time (2048 x 10240 x 1280, cold: 57.6 us against 70.0 in groups of two;
// 1024 x 10240 x 1280: 32.7 against 42.2), elsewhere every XCD walks all weights and it loses
// (8192 x 3456 x 1152: 85.5 against 72.4).  From 3072 channels on, 384 per XCD, row-major wins at
// every height (1000 x 3072 x 768: 9.1 us against 12.2 in groups of two; 2048 x 3072 x 1280: 21.2
// against 24.1; 8192 x 6144 x 1280: 116 against 127; 4096 x 4096 x 640: 27.0 against 29.8); an
// XCD's share of fewer channels does not always pay for the wider spread of its activation rows
// (1000 x 2048 x 1280: 8.8 against 10.6, but 4096 x 2048 x 640, INT8: 17.4 against 16.5;
// 8192 x 1024 x 1280: 29.2 against 26.4).
int group_rows(int mt, int tn, int bn) { return tn % 8 == 0 && tn * bn >= 3072 ? 0 : std::min(2, mt); }

void launch_gemm(GemmArgs a, int tile, int af, hipStream_t s) {
    const TileCost& c = kTileCosts[tile];
    const int mt = row_tiles(a.M, c);
    a.tn = col_tiles(a.N, c);
    a.gm = group_rows(mt, a.tn, c.bn());
    a.cached = a.splits > 1 || (a.N & 31) != 0;
    const unsigned grid = (unsigned)(mt * a.tn * a.splits);
    if (a.C > 0) launch_gemm_fmt<true>(a, af, tile, grid, s);
    else launch_gemm_fmt<false>(a, af, tile, grid, s);
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }
// half-precision weights: whole blocks of 32 channels
int64_t weight_bytes(int64_t N, int64_t K) { return (N + 31) / 32 * (K / BK) * (kBlockChunks * 16); }

}  // namespace
}  // namespace cham

using namespace cham;

// Chunks of k-steps the record pre-pass splits a weight into: about one workgroup per CU per
// layer (all of a batch resident at once), at least 4 k-steps each.
static void rec_chunks(int64_t N, int64_t K, int* nkc, int* rchunk) {
    const int nblk = (int)((N + kRecChannels - 1) / kRecChannels), nst = (int)(K / BK);
    const int n = std::max(1, std::min((256 + nblk - 1) / nblk, (nst + 3) / 4));
    *rchunk = (nst + n - 1) / n;
    *nkc = (nst + *rchunk - 1) / *rchunk;
}

// The packed layout: ColPrep[N], the column-sum partials [k-chunks][N], then the half-precision
// weights.
extern "C" size_t cham_packed_bytes(int64_t N, int64_t K) {
    if (N < 1 || K < 64) return 0;
    int nkc, rchunk;
    rec_chunks(N, K, &nkc, &rchunk);
    return align256((size_t)N * sizeof(ColPrep)) + align256((size_t)nkc * (size_t)N * 4) + (size_t)weight_bytes(N, K);
}

struct Layout {
    ColPrep* cols;
    float* colsum;
    uint4* wh;
};
static Layout layout_at(void* p, int64_t N, int64_t K) {
    int nkc, rchunk;
    rec_chunks(N, K, &nkc, &rchunk);
    char* c = (char*)p;
    Layout l;
    l.cols = (ColPrep*)c;
    c += align256((size_t)N * sizeof(ColPrep));
    l.colsum = (float*)c;
    c += align256((size_t)nkc * (size_t)N * 4);
    l.wh = (uint4*)c;
    return l;
}

// One searched weight as the record pre-pass and the GEMM see it: per-channel formats
// (cham_wq) or group-scaled weights of one format (cham_gwq).
struct WView {
    int64_t N, K;
    uint32_t mask;
    int code_bits;
    const uint8_t* fmt;
    const float* scale;
    const float* zero;
    const float* nf4;
    const uint8_t* e8;
    const uint8_t* codes;
    void* packed;
    const int32_t* gsel;
    const float* gscale;
    const float* gzero;
};

static WView view_of(const cham_wq* wq) {
    return WView{wq->N, wq->K, wq->palette_mask, wq->code_bits, wq->fmt, wq->scale, wq->zero, wq->nf4_absmax,
                 wq->e8m0, wq->codes, wq->packed, nullptr, nullptr, nullptr};
}

static WView view_of(const cham_gwq* gq) {
    return WView{gq->N, gq->K, gq->palette_mask, gq->code_bits, gq->fmt, nullptr, nullptr, nullptr,
                 gq->e8m0, gq->codes, gq->packed, gq->choice, gq->gscale, gq->gzero};
}

// Record pre-pass arguments of one searched weight writing into the layout L (device),
// and the workgroups it takes.
static RecArgs record_args(const WView& v, const Layout& L, int* wgs) {
    const uint32_t mask = v.mask;
    const int N = (int)v.N, K = (int)v.K;
    const bool nf4 = (mask >> CHAM_W_NF4) & 1u;
    const bool wmx = (mask & ((1u << CHAM_W_MXINT8) | (1u << CHAM_W_MXINT4) | (1u << CHAM_W_MXFP4))) != 0u;
    const int nblk = (N + kRecChannels - 1) / kRecChannels;
    int nkc, rchunk;
    rec_chunks(N, K, &nkc, &rchunk);
    *wgs = nblk * nkc;
    // block metadata only of the enabled formats (the pre-pass reads it ahead of the format)
    return RecArgs{v.fmt, v.scale, v.zero, nf4 && !v.gsel ? v.nf4 : nullptr, wmx ? v.e8 : nullptr, v.codes,
                   mask, N, K, v.code_bits, rchunk, L.cols, L.colsum, L.wh, v.gsel, v.gscale, v.gzero};
}

static void launch_records(const WView& v, const Layout& L, hipStream_t s) {
    RecBatch B;
    B.nl = 1;
    B.ng = 0;
    int wgs = 0;
    B.r[0] = record_args(v, L, &wgs);
    B.wg_end[0] = wgs;
    hipLaunchKernelGGL(record_kernel, dim3((unsigned)wgs), dim3(256), 0, s, B);
}

// Writes the packed layout of n searched weights (the arguments checked and code_bits set),
// and with `group` also groups the channels of those that ask for perm / group_off; one
// launch per kRecBatchMax weights.
static int pack_weights(const cham_wq* const* wqs, int n, bool group, hipStream_t s) {
    for (int i0 = 0; i0 < n; i0 += kRecBatchMax) {
        RecBatch B;
        B.nl = std::min(kRecBatchMax, n - i0);
        B.ng = 0;
        int total = 0;
        for (int j = 0; j < B.nl; ++j) {
            const cham_wq* wq = wqs[i0 + j];
            int wgs = 0;
            B.r[j] = record_args(view_of(wq), layout_at(wq->packed, wq->N, wq->K), &wgs);
            total += wgs;
            B.wg_end[j] = total;
            if (group && (wq->perm || wq->group_off))
                B.g[B.ng++] = GroupArgs{wq->fmt, (int)wq->N, wq->perm, wq->group_off};
        }
        hipLaunchKernelGGL(record_kernel, dim3((unsigned)(total + B.ng)), dim3(256), 0, s, B);
        CHAM_CHECK_LAUNCH();
    }
    return CHAM_OK;
}

// The search entry points' packing step (they have checked the arguments and set code_bits).
int cham_pack_weights(const cham_wq* const* wqs, int n, hipStream_t s) { return pack_weights(wqs, n, true, s); }

extern "C" int cham_pack_weights_batch(const cham_wq* wq, int32_t n, void* stream) {
    if (!wq || n < 1) return CHAM_EINVAL;
    std::vector<const cham_wq*> p((size_t)n);
    for (int i = 0; i < n; ++i) {
        const cham_wq& w = wq[i];
        if (!w.fmt || !w.codes || !w.scale || !w.zero || !w.packed || w.N < 1) return CHAM_EINVAL;
        if ((uintptr_t)w.packed & 255u) return CHAM_EINVAL;
        const uint32_t mask = w.palette_mask;
        if (mask == 0u || (mask >> CHAM_W_NFMT) != 0u) return CHAM_EFORMAT;
        if (w.code_bits != ((mask & 0x7u) ? 8 : 4)) return CHAM_EINVAL;
        if (w.K < 64 || w.K % 64 != 0 || w.K > (1 << 20)) return CHAM_ESHAPE;
        if (((mask >> CHAM_W_NF4) & 1u) && !w.nf4_absmax) return CHAM_EINVAL;
        if ((mask & ((1u << CHAM_W_MXINT8) | (1u << CHAM_W_MXINT4) | (1u << CHAM_W_MXFP4))) && !w.e8m0)
            return CHAM_EINVAL;
        if (w.N * (w.K / 64) * 128 > (int64_t)INT32_MAX) return CHAM_EINVAL;
        p[(size_t)i] = &w;
    }
    return pack_weights(p.data(), n, false, (hipStream_t)stream);
}

// The packed layout of a group-scaled weight (called by the grouped search after its
// launches, which have checked the arguments).
int cham_pack_grouped(const cham_gwq* gq, hipStream_t s) {
    launch_records(view_of(gq), layout_at(gq->packed, gq->N, gq->K), s);
    CHAM_CHECK_LAUNCH();
    return CHAM_OK;
}

size_t cham_linear_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    return align256((size_t)M * (size_t)K * 2) + align256((size_t)M * 4) + align256(cham_packed_bytes(N, K)) +
           split_bytes(M, N, K);
}

extern "C" int cham_linear_plan(int64_t M, int64_t N, int64_t K, int32_t code_bits, int32_t* out, int32_t out_len) {
    if (!out || out_len < 10 || M < 1 || N < 1 || K < 1 || M > INT32_MAX || N > INT32_MAX || K > INT32_MAX ||
        (code_bits != 4 && code_bits != 8))
        return CHAM_EINVAL;
    const Plan p = plan_gemm((int)M, (int)N, (int)K);
    for (int i = 0; i < 10; ++i) out[i] = 0;
    out[0] = 1;
    out[1] = p.splits;
    out[3] = (int32_t)M;
    out[4] = kTileCosts[p.tile].bm();
    out[5] = kTileCosts[p.tile].bn();
    return CHAM_OK;
}

// 3x3 convolution geometry (images B x H x W, channels last)
struct ConvSpec {
    int B, H, W;
};

// Workspace of the convolution: what ws_layout reserves for activations, the weights' layout
// (no packed layout given) and the k-split partials.
static size_t conv_workspace(int64_t B, int64_t H, int64_t W, int64_t C, int64_t Co) {
    const int64_t M = B * H * W;
    return align256((size_t)(B * (H + 2) * (W + 2) * C) * 2) + align256((size_t)M * 4) + 256 +
           align256(cham_packed_bytes(Co, 9 * C)) + split_bytes(M, Co, 9 * C);
}

// What one call uses of its workspace: the weight layout (when no packed layout comes with the
// weight) and the k-split partials (when the plan splits).  MX activations and the convolution
// reserve room for a half-precision activation copy and its scales in front: nothing is written
// there, but the sizes that callers are told, and below which a call is refused, include it.
struct WsLayout {
    size_t rec, part, total;
};
static WsLayout ws_layout(bool half_copy, size_t xh_bytes, bool conv, bool packed, int64_t M, int64_t N, int64_t K,
                          int splits) {
    WsLayout l;
    l.rec = (half_copy ? align256(xh_bytes) + align256((size_t)M * 4) : 0) + (conv ? 256 : 0);
    l.part = l.rec + (packed ? 0 : align256(cham_packed_bytes(N, K)));
    l.total = l.part + (splits > 1 ? (size_t)splits * (size_t)M * (size_t)N * 4 : 0);
    return l;
}

// ws_need != NULL: only report the workspace bytes these operands need (Y and ws unused).
static int mixed_linear_impl(const cham_aq* xq, const WView& v, float* Y, void* ws, size_t ws_bytes, void* stream,
                             const ConvSpec* cv = nullptr, size_t* ws_need = nullptr) {
    const WView* wq = &v;
    if (!xq || (!Y && !ws_need) || !xq->codes || !xq->scale || !xq->zero) return CHAM_EINVAL;
    if (!wq->fmt || !wq->codes) return CHAM_EINVAL;
    if (!wq->gsel && (!wq->scale || !wq->zero)) return CHAM_EINVAL;
    if (wq->gsel && (!wq->gscale || !wq->gzero)) return CHAM_EINVAL;
    if (xq->M < 1 || wq->N < 1 || xq->K < 1 || (cv ? 9 * xq->K : xq->K) != wq->K) return CHAM_EINVAL;
    if (cv) {
        if (cv->B < 1 || cv->H < 1 || cv->W < 1 || (int64_t)cv->B * cv->H * cv->W != xq->M) return CHAM_EINVAL;
        if (xq->K % 64 != 0) return CHAM_ESHAPE;  // a k-step never straddles two taps
        const int64_t xb = (int64_t)cv->B * (cv->H + 2) * (cv->W + 2) * xq->K * 2;
        if (xb > (int64_t)INT32_MAX - 4096) return CHAM_ESHAPE;  // 32-bit buffer offsets
        if (xq->nsamples != 1 && xq->nsamples != cv->B) return CHAM_EINVAL;  // a sample is whole images
    }
    if (xq->fmt < 0 || xq->fmt >= CHAM_A_NFMT) return CHAM_EFORMAT;
    if (xq->nsamples < 1 || xq->M % xq->nsamples != 0) return CHAM_EINVAL;
    const uint32_t mask = wq->mask;
    if (mask == 0u || (mask >> CHAM_W_NFMT) != 0u) return CHAM_EFORMAT;
    const int code_bits = (mask & 0x7u) ? 8 : 4;
    if (wq->code_bits != code_bits) return CHAM_EFORMAT;
    if (wq->gsel && code_bits != 4) return CHAM_EFORMAT;  // the 8-bit group-scaled decode is not built
    if (wq->K % 64 != 0) return CHAM_ESHAPE;
    // 32-bit buffer offsets: an activation tile and an output tile of 256 rows (the tiles have 128
    // at most) and the half-precision weights stay below 2^31 bytes
    if (xq->M > INT32_MAX / 2 || wq->N > INT32_MAX / 1024 || wq->K > (1 << 20) ||
        wq->N * (wq->K / BK) * 128 > (int64_t)INT32_MAX)
        return CHAM_ESHAPE;
    const bool nf4 = (mask >> CHAM_W_NF4) & 1u;
    const bool wmx = (mask & ((1u << CHAM_W_MXINT8) | (1u << CHAM_W_MXINT4) | (1u << CHAM_W_MXFP4))) != 0u;
    if ((nf4 && !wq->gsel && !wq->nf4) || (wmx && !wq->e8)) return CHAM_EINVAL;
    const bool amx = xq->fmt == CHAM_A_MXFP8_E4M3 || xq->fmt == CHAM_A_MXINT8;
    if (amx && !xq->e8m0) return CHAM_EINVAL;
    if (((uintptr_t)xq->codes & 15u) || ((uintptr_t)wq->codes & 15u) || ((uintptr_t)wq->packed & 255u))
        return CHAM_EINVAL;
    const int M = (int)xq->M, N = (int)wq->N, K = (int)wq->K;
    const Plan plan = plan_gemm(M, N, K);
    const int kchunk = (K / BK + plan.splits - 1) / plan.splits;
    // every split holds at least one k-step (the operand ranges of the kernel rely on it)
    if (plan.splits < 1 || (plan.splits - 1) * kchunk >= K / BK) return CHAM_ESHAPE;
    const size_t xh_bytes = cv ? (size_t)cv->B * (cv->H + 2) * (cv->W + 2) * xq->K * 2 : (size_t)M * (size_t)K * 2;
    const WsLayout wl = ws_layout(amx || cv, xh_bytes, cv != nullptr, wq->packed != nullptr, M, N, K, plan.splits);
    if (ws_need) {  // the size query: nothing is checked against a buffer, nothing launched
        *ws_need = wl.total;
        return CHAM_OK;
    }
    if (wl.total > 0 && (!ws || ws_bytes < wl.total || ((uintptr_t)ws & 255u))) return CHAM_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;

    char* w = (char*)ws;
    // the search's packed layout replaces the pre-pass
    const Layout lay = layout_at(wq->packed ? wq->packed : (void*)(w + wl.rec), N, K);
    float* part = (float*)(w + wl.part);

    if (!wq->packed) launch_records(v, lay, s);
    CHAM_CHECK_LAUNCH();

    GemmArgs a;
    a.xc = xq->codes;
    a.xe8 = xq->e8m0;
    a.xs = xq->scale;
    a.xz = xq->zero;
    a.rps = M / xq->nsamples;
    a.cols = lay.cols;
    a.colsum = lay.colsum;
    {
        int rchunk;
        rec_chunks(N, K, &a.nkc, &rchunk);
    }
    a.wh = lay.wh;
    a.Y = Y;
    a.M = M;
    a.N = N;
    a.K = K;
    a.part = part;
    a.H = cv ? cv->H : 0;
    a.W = cv ? cv->W : 0;
    a.C = cv ? (int)xq->K : 0;
    a.splits = plan.splits;
    a.kchunk = kchunk;
    launch_gemm(a, plan.tile, xq->fmt, s);
    CHAM_CHECK_LAUNCH();
    if (plan.splits > 1) {
        const int64_t MN = (int64_t)M * N;
        const int64_t per = (MN & 3) == 0 ? MN / 4 : MN;
        const unsigned grid = (unsigned)std::min<int64_t>((per + 255) / 256, 4096);
        hipLaunchKernelGGL(reduce_kernel, dim3(grid), dim3(256), 0, s, part, Y, MN, plan.splits);
        CHAM_CHECK_LAUNCH();
    }
    return CHAM_OK;
}

extern "C" int cham_mixed_linear(const cham_aq* xq, const cham_wq* wq, float* Y, void* ws, size_t ws_bytes,
                                 void* stream) {
    if (!wq) return CHAM_EINVAL;
    return mixed_linear_impl(xq, view_of(wq), Y, ws, ws_bytes, stream);
}

extern "C" int cham_mixed_linear_workspace_query(const cham_aq* xq, const cham_wq* wq, size_t* bytes) {
    if (!wq || !bytes) return CHAM_EINVAL;
    return mixed_linear_impl(xq, view_of(wq), nullptr, nullptr, 0, nullptr, nullptr, bytes);
}

extern "C" int cham_mixed_linear_grouped_workspace_query(const cham_aq* xq, const cham_gwq* gq, size_t* bytes) {
    if (!gq || !gq->choice || !bytes) return CHAM_EINVAL;
    return mixed_linear_impl(xq, view_of(gq), nullptr, nullptr, 0, nullptr, nullptr, bytes);
}

extern "C" int cham_mixed_linear_grouped(const cham_aq* xq, const cham_gwq* gq, float* Y, void* ws, size_t ws_bytes,
                                         void* stream) {
    if (!gq || !gq->choice) return CHAM_EINVAL;
    return mixed_linear_impl(xq, view_of(gq), Y, ws, ws_bytes, stream);
}

extern "C" int cham_conv3x3_mixed(const cham_aq* xq, int32_t B, int32_t H, int32_t W, const cham_wq* wq, float* Y,
                                  void* ws, size_t ws_bytes, void* stream) {
    if (!wq) return CHAM_EINVAL;
    const ConvSpec cv{B, H, W};
    return mixed_linear_impl(xq, view_of(wq), Y, ws, ws_bytes, stream, &cv);
}

extern "C" size_t cham_conv3x3_workspace_bytes(int64_t B, int64_t H, int64_t W, int64_t C, int64_t Co) {
    if (B < 1 || H < 1 || W < 1 || C < 64 || Co < 1) return 0;
    return conv_workspace(B, H, W, C, Co);
}

