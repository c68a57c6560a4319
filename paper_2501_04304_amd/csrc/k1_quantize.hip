// K1: fused row statistics + pixel-class decision + group affine quantizer.
//
// Linear quantizer of Section 3.1 with the per-cell scale and offset of
// Section 3.3:  q = clamp(rne((x - z[p,g]) * inv_s[p,g]), 0, 2^b - 1).
//
// HBM-bound: every fp32 input is read once (4 B) and one code is written
// (1 B at 8 bit, 0.5 B at 4 bit), plus one class byte per row.
//
// A row belongs to one wavefront (W = 1) or to the four of a workgroup (W = 4).  It arrives in
// registers with 16-byte loads, issued one row ahead, is reduced to max / min with wave shuffles, and is
// parked in LDS.  After the class decision every lane takes 4 (8-bit) or 8 (4-bit) consecutive OUTPUT
// positions per step, gathers the inputs from LDS through the channel permutation, and writes one dword
// into the block-tiled code layout the contraction loads (64 contiguous bytes per row and chunk).
//
// What a lane needs for its output dwords -- the gather offsets (two 16-bit byte offsets to a register), the
// mask that clears padding positions of the packed word, (z, 1/s) for both classes, the place in the tiled
// row -- stays in REGISTERS for all of the wavefront's rows, read once from tables prepared with the
// handle: no table build and no barrier before the first row, a quarter less LDS traffic per position, and LDS holds
// nothing but the rows.  A row of more than 1280 channels (2560 with 4-bit codes, whose lanes take twice as many positions)
// is shared by four wavefronts instead (two row buffers and one barrier per row): the tables still fit, and a
// CU holds twelve wavefronts where one row per wavefront left it four.  So are longer rows of a launch with few of them.
//
// The loop over rows stores without conditions (a lane past the last output dword repeats that
// dword): then the wait for the prefetched row is a wait for exactly that row, while with one conditional
// store it becomes a wait for every store before it as well, a write round trip per row (the classes, too,
// are kept and stored once per wavefront).  The form that writes a convolution's shifted copies does not have this: which
// copies a pixel goes to depends on its column, and its stores wait.  Measured against the kernel that built its tables in LDS and
// stored conditionally, us: 154 x 768 4.1 -> 2.8, 512 x 1280 5.0 -> 3.2, 8192 x 320 7.5 -> 4.7, 2964 x 1280 7.0 -> 5.7,
// 65536 x 640 41.5 -> 37.0 (5.8 TB/s), 16384 x 1280 24.1 -> 21.2, 16384 x 5120 8-bit 98.8 -> 75.3 (5.6 TB/s), 4-bit
// 88.7 -> 72.3 (5.2 TB/s); a copy reaches 4.9 TB/s.
#include "dgq_internal.h"

namespace dgq {

namespace {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;

// Three-operand max / min as the instruction itself: written through the compiler's
// fmaxf they come wrapped in one canonicalising instruction per loaded value.
__device__ inline float max3(float a, float b, float c) {
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ inline float min3(float a, float b, float c) {
    float d;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// Wave-wide maximum of mx and minimum of mn without LDS traffic, both returned as
// wave-uniform values.  Four cross-lane (DPP) steps leave every 16-lane row with its own
// extreme (lane ^ 1, lane ^ 2, mirrored halves, mirrored row), two row broadcasts carry
// it on to lane 63.  The two chains alternate and one s_nop separates the steps: a DPP
// operand may be read two wait states after the register was written at the earliest.
#define DGQ_DPP_STEP(ctrl)                                 \
    "v_max_f32_dpp %0, %0, %0 " ctrl " bank_mask:0xf\n\t" \
    "v_min_f32_dpp %1, %1, %1 " ctrl " bank_mask:0xf\n\t" \
    "s_nop 0\n\t"
__device__ inline void wave_max_min(float &mx, float &mn) {
    asm("s_nop 1\n\t"
        DGQ_DPP_STEP("quad_perm:[1,0,3,2] row_mask:0xf")
        DGQ_DPP_STEP("quad_perm:[2,3,0,1] row_mask:0xf")
        DGQ_DPP_STEP("row_half_mirror row_mask:0xf")
        DGQ_DPP_STEP("row_mirror row_mask:0xf")
        DGQ_DPP_STEP("row_bcast:15 row_mask:0xa")
        DGQ_DPP_STEP("row_bcast:31 row_mask:0xc")
        : "+v"(mx), "+v"(mn));
    mx = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mx), 63));
    mn = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mn), 63));
}
#undef DGQ_DPP_STEP

// q as a float in [0, qmax]; separate subtract and multiply (no contraction).
__device__ inline float quant1(float x, float z, float inv_s, float qmax) {
    const float t = __fsub_rn(x, z);
    const float u = __fmul_rn(t, inv_s);
    return fminf(fmaxf(rintf(u), 0.0f), qmax);
}

// The same value, unrounded, for v_cvt_pk_u8_f32 to finish: that instruction rounds to
// nearest even and saturates to [0, 255] (NaN -> 0) by itself (checked against
// rint + clamp on a million values, ties and the values next to them included), so at
// 8 bit nothing is left to do, and at 4 bit only the upper clamp, which commutes with
// the rounding because the bound is an integer.  v_med3_f32 returns the minimum of its
// operands when one is NaN, i.e. 0 here, as the three-step form does.
template <int BITS>
__device__ inline float quant_pre(float x, float z, float inv_s) {
    const float t = __fsub_rn(x, z);
    const float u = __fmul_rn(t, inv_s);
    return BITS == 8 ? u : __builtin_amdgcn_fmed3f(u, 0.0f, 15.0f);
}

// NV: float4 per lane that hold the wavefront's share of a row; NS: its output dwords per lane.
// CONV: the rows are the pixels of images conv_w wide and the codes are written three times for the
// tap-gathering 3 x 3 convolution: copy 1 (codes + copy_bytes) is the map itself, copy 0 holds in row r the
// codes of the pixel left of r, copy 2 of the pixel right of r, and the code of the value 0 (fill32, one dword
// per output dword) where the image ends.
template <int BITS, int W, int NV, int NS, bool CONV>
__global__ __launch_bounds__(256) void k_quantize_act(
    const float *__restrict__ x, int64_t rows, int32_t C, int32_t n_dw, int32_t n_chunks,
    const uint32_t *__restrict__ q_off, const uint32_t *__restrict__ q_keep, const float2 *__restrict__ q_zi,
    const float *__restrict__ taus, int32_t n_tau, int8_t *__restrict__ codes,
    uint8_t *__restrict__ row_class, int32_t rows_per, int32_t conv_w, int64_t copy_bytes,
    const uint32_t *__restrict__ fill32, int64_t wg0) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    constexpr int kPer = BITS == 8 ? 4 : 8;
    constexpr int kDwPerChunk = 64 / kPer;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int part = W == 1 ? 0 : wave;  // this wave's share of a row
    float *xs = reinterpret_cast<float *>(lds_raw) + (W == 1 ? (size_t)wave * C : 0);
    float2 *zi_tab = reinterpret_cast<float2 *>(lds_raw + (size_t)C * (W == 1 ? 16 : 8));  // more than two classes
    __shared__ float2 ext[2][W];  // the waves' extremes of a row
    const uint32_t c4n = (uint32_t)C >> 2;
    const int64_t wg = wg0 + blockIdx.x;  // wg0: the workgroups of the launches before this one
    const int64_t first = (W == 1 ? wg * kWavesPerBlock + wave : wg) * rows_per;
    const int32_t n = first >= rows ? 0 : (int32_t)(rows - first < rows_per ? rows - first : rows_per);

    // An index past the end of the row is clamped to the last valid one, which re-reads a value that is
    // already part of the row, so max / min and the LDS copy are unaffected.
    float4 v[NV];
    uint32_t cidx[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const uint32_t c = lane + (k * W + part) * kWave;
        cidx[k] = c < c4n ? c : c4n - 1;
    }
    auto fetch = [&](int64_t r) __attribute__((always_inline)) {
        const float4 *x4 = reinterpret_cast<const float4 *>(x + r * C);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            // the activations are read exactly once: non-temporal, keep the caches for the codes
            typedef float v4f __attribute__((ext_vector_type(4)));
            const v4f t = __builtin_nontemporal_load(reinterpret_cast<const v4f *>(x4 + cidx[k]));
            v[k] = make_float4(t.x, t.y, t.z, t.w);
        }
    };
    if (n > 0) fetch(first);

    // the tables of this lane's output dwords travel with the first row
    uint32_t off[NS][kPer / 2], keep[NS], pos[NS];  // pos: place in the tiled row, before the row's slot swizzle
    float z0[NS], i0[NS], z1[NS], i1[NS];
    int32_t chunk[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        const uint32_t d0 = lane + 64u * (t * W + part), d = d0 < (uint32_t)n_dw ? d0 : (uint32_t)n_dw - 1;
        if constexpr (BITS == 8) {
            const uint2 o = reinterpret_cast<const uint2 *>(q_off)[d];
            off[t][0] = o.x; off[t][1] = o.y;
        } else {
            const uint4 o = reinterpret_cast<const uint4 *>(q_off)[d];
            off[t][0] = o.x; off[t][1] = o.y; off[t][kPer / 2 - 2] = o.z; off[t][kPer / 2 - 1] = o.w;
        }
        keep[t] = q_keep[d];
        chunk[t] = (int32_t)(d / kDwPerChunk);
        const float2 c0 = q_zi[chunk[t]], c1 = q_zi[n_chunks + chunk[t]];
        z0[t] = c0.x; i0[t] = c0.y; z1[t] = c1.x; i1[t] = c1.y;
        pos[t] = (d / kDwPerChunk) * 1024u + (d % kDwPerChunk) * 4u;
    }
    // lane k holds threshold k: the class of a row is the number of thresholds below its
    // range (the nearest cluster centre), counted with one compare and a mask population count
    const float tau_lane = lane < n_tau ? taus[lane] : INFINITY;
    if (n_tau > 1) {
        for (int32_t i = tid; i < (n_tau + 1) * n_chunks; i += 256) zi_tab[i] = q_zi[i];
        __syncthreads();
    }
    uint32_t cls = 0;  // lane i: the class of this wavefront's i-th row

    // a row's place in the tiled layout: scalar base, and what its slot swizzle flips in a lane's place
    auto row_base = [&](int64_t rr) -> int8_t * {
        const uint32_t t = (uint32_t)rr & (BITS == 8 ? 15u : 31u);
        return codes + (((rr >> (BITS == 8 ? 4 : 5)) * n_chunks) << 10) + t * (BITS == 8 ? 64u : 32u);
    };
    auto row_xor = [&](int64_t rr) -> uint32_t {
        const uint32_t t = (uint32_t)rr & (BITS == 8 ? 15u : 31u);
        return BITS == 8 ? (uint32_t)swz64((int)t) << 4 : ((uint32_t)swz32((int)t) << 4) | ((uint32_t)half32((int)t) << 3);
    };
    auto one_row = [&](const int32_t i, const bool more) __attribute__((always_inline)) {
        const int64_t r = first + i;
        float mx = -INFINITY, mn = INFINITY;
        float *xrow = W == 1 ? xs : xs + (i & 1) * C;
        float4 *s4 = reinterpret_cast<float4 *>(xrow);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            s4[cidx[k]] = v[k];
            mx = max3(max3(v[k].x, v[k].y, v[k].z), v[k].w, mx);
            mn = min3(min3(v[k].x, v[k].y, v[k].z), v[k].w, mn);
        }
        if (more) fetch(r + 1);
        wave_max_min(mx, mn);
        if (W > 1) {
            if (lane == 0) ext[i & 1][wave] = make_float2(mx, mn);
            // LDS only: a full barrier would also wait for the row being fetched.  One per row is enough,
            // since the next row goes to the other buffer.
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const float2 e = ext[i & 1][w];
                mx = fmaxf(mx, e.x);
                mn = fminf(mn, e.y);
            }
            mx = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, mx)));
            mn = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, mn)));
        }
        const char *xsb = reinterpret_cast<const char *>(xrow);
        const int p = __builtin_popcountll(__ballot(__fsub_rn(mx, mn) > tau_lane));
        cls = lane == i ? (uint32_t)p : cls;
        // (W = 1) the slice is private to this wave and a wave's LDS operations complete in issue order, so a
        // compiler-level fence is all that is needed
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        int8_t *out_row = row_base(r) + (CONV ? copy_bytes : 0);
        const uint32_t out_xor = row_xor(r);
        float xv[NS][kPer];
#pragma unroll
        for (int t = 0; t < NS; ++t)
#pragma unroll
            for (int k = 0; k < kPer; ++k)
                xv[t][k] = *reinterpret_cast<const float *>(xsb + ((off[t][k / 2] >> (16 * (k & 1))) & 0xffffu));
        uint32_t word[NS];
        const uint32_t second = p == 0 ? 0u : ~0u;  // a mask: a select would put the arrays in memory
        auto pick = [&](float a, float b) {
            return __uint_as_float((__float_as_uint(a) & ~second) | (__float_as_uint(b) & second));
        };
#pragma unroll
        for (int t = 0; t < NS; ++t) {
            float z = pick(z0[t], z1[t]), is = pick(i0[t], i1[t]);
            if (p > 1) {
                const float2 zi = zi_tab[p * n_chunks + chunk[t]];
                z = zi.x;
                is = zi.y;
            }
            uint32_t lo = 0, hi = 0;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const float qf = quant_pre<BITS>(xv[t][k], z, is);
                if (k < 4)
                    lo = __builtin_amdgcn_cvt_pk_u8_f32(qf, k, lo);
                else
                    hi = __builtin_amdgcn_cvt_pk_u8_f32(qf, k - 4, hi);
            }
            // 8 bit: stored code = q - 128 = q ^ 0x80 per byte.  4 bit: byte i holds position i (low
            // nibble) and position i + 4 (high nibble).  Padding positions are cleared to the stored value 0.
            word[t] = (BITS == 8 ? (lo ^ 0x80808080u) : (lo | (hi << 4))) & keep[t];
            *reinterpret_cast<uint32_t *>(out_row + (pos[t] ^ out_xor)) = word[t];
        }
        if (CONV) {
            // the shifted copies: this row's codes are the left neighbour of row r + 1 and the right
            // neighbour of row r - 1 of the same image row
            auto fill = [&](int t) { return fill32[(pos[t] >> 10) * kDwPerChunk + ((pos[t] & 1023u) >> 2)]; };
            const int32_t wcol = (int32_t)(r % conv_w);
            if (wcol + 1 < conv_w) {
                int8_t *rowL = row_base(r + 1);
                const uint32_t x2 = row_xor(r + 1);
#pragma unroll
                for (int t = 0; t < NS; ++t) *reinterpret_cast<uint32_t *>(rowL + (pos[t] ^ x2)) = word[t];
            } else {
                int8_t *rowF = row_base(r) + 2 * copy_bytes;
#pragma unroll
                for (int t = 0; t < NS; ++t) *reinterpret_cast<uint32_t *>(rowF + (pos[t] ^ out_xor)) = fill(t);
            }
            if (wcol > 0) {
                int8_t *rowR = row_base(r - 1) + 2 * copy_bytes;
                const uint32_t x2 = row_xor(r - 1);
#pragma unroll
                for (int t = 0; t < NS; ++t) *reinterpret_cast<uint32_t *>(rowR + (pos[t] ^ x2)) = word[t];
            } else {
                int8_t *rowF = row_base(r);
#pragma unroll
                for (int t = 0; t < NS; ++t) *reinterpret_cast<uint32_t *>(rowF + (pos[t] ^ out_xor)) = fill(t);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (int32_t i = 0; i + 1 < n; ++i) one_row(i, true);
    if (n > 0) one_row(n - 1, false);
    if (lane < n && part == 0) row_class[first + lane] = (uint8_t)cls;
}

// Fallback for channel counts that are not a multiple of 4 (no 16-byte loads):
// scalar loads straight into LDS, tables read from global memory.
template <int BITS>
__global__ __launch_bounds__(256) void k_quantize_act_any(
    const float *__restrict__ x, int64_t rows, int32_t C, int32_t Kp, int32_t n_chunks,
    const int32_t *__restrict__ perm, const float *__restrict__ chunk_z,
    const float *__restrict__ chunk_inv, const float *__restrict__ taus, int32_t n_tau,
    int8_t *__restrict__ codes, uint8_t *__restrict__ row_class) {
    extern __shared__ float lds[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float *xs = lds + (size_t)wave * C;
    constexpr float qmax = (float)((1 << BITS) - 1);
    constexpr int kOff = BITS == 8 ? 128 : 0;
    constexpr int kPer = BITS == 8 ? 4 : 8;  // positions per output dword
    const float tau_lane = lane < n_tau ? taus[lane] : INFINITY;

    for (int64_t r = (int64_t)blockIdx.x * kWavesPerBlock + wave; r < rows;
         r += (int64_t)gridDim.x * kWavesPerBlock) {
        const float *xr = x + r * C;
        float mx = -INFINITY, mn = INFINITY;
        for (int32_t c = lane; c < C; c += kWave) {
            const float v = xr[c];
            xs[c] = v;
            mx = fmaxf(v, mx);
            mn = fminf(v, mn);
        }
        wave_max_min(mx, mn);
        const int p = __builtin_popcountll(__ballot(__fsub_rn(mx, mn) > tau_lane));
        if (lane == 0) row_class[r] = (uint8_t)p;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int32_t jd = lane; jd < Kp / kPer; jd += kWave) {
            const int32_t ch = (jd * kPer) >> 6;
            const float z = chunk_z[p * n_chunks + ch], is = chunk_inv[p * n_chunks + ch];
            uint32_t word = 0;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int32_t c = perm[jd * kPer + k];
                uint32_t qv = 0;
                if (c >= 0) {
                    const int32_t q = (int32_t)quant1(xs[c], z, is, qmax) - kOff;
                    qv = BITS == 8 ? ((uint32_t)q & 0xffu) : (uint32_t)q;
                }
                word |= BITS == 8 ? qv << (8 * k) : qv << (k < 4 ? 8 * k : 8 * (k - 4) + 4);
            }
            const int64_t off = BITS == 8 ? tiled64_offset(r, ch, n_chunks, (jd >> 2) & 3)
                                          : tiled32_offset(r, ch, n_chunks, (jd >> 2) & 1);
            const int dw = BITS == 8 ? (jd & 3) : ((jd & 3) ^ (2 * half32((int)(r & 31))));
            *reinterpret_cast<uint32_t *>(codes + off + dw * 4) = word;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

using Kern = void (*)(const float *, int64_t, int32_t, int32_t, int32_t, const uint32_t *, const uint32_t *,
                      const float2 *, const float *, int32_t, int8_t *, uint8_t *, int32_t, int32_t, int64_t,
                      const uint32_t *, int64_t);
struct Picked {
    Kern kern;
    LdsLimit *lim;
};
template <int BITS, int W, int NV, int NS, bool CONV>
Picked picked() {
    static LdsLimit lim;
    return {k_quantize_act<BITS, W, NV, NS, CONV>, &lim};
}

// of the widest four-wavefront kernel: 8192 channels; 15360 positions at 8 bit (the padding of a 3 x 3 convolution's
// nine times sixteen groups comes to 9072), 20480 at 4 bit
constexpr int kMostFloat4 = 8;
constexpr int most_steps(int bits) { return bits == 8 ? 15 : 10; }

// The smallest kernel that holds nv float4 and ns output dwords per lane.
template <int BITS, bool CONV>
Picked pick(int W, int nv, int ns) {
#define DGQ_PICK(W_, NV, NS) \
    if (W == W_ && nv <= NV && ns <= NS) return picked<BITS, W_, NV, NS, CONV>()
    DGQ_PICK(1, 2, 2);
    DGQ_PICK(1, 3, 3);
    DGQ_PICK(1, 3, 5);
    DGQ_PICK(1, 5, 6);
    DGQ_PICK(1, 5, 8);
    if constexpr (BITS == 4) {
        DGQ_PICK(1, 8, 4);
        DGQ_PICK(1, 10, 6);
    }
    DGQ_PICK(4, 2, 2);
    DGQ_PICK(4, 3, 3);
    DGQ_PICK(4, 5, 3);
    DGQ_PICK(4, 5, 6);
    DGQ_PICK(4, 8, 5);
    DGQ_PICK(4, kMostFloat4, 10);
    if constexpr (BITS == 8 && !CONV) DGQ_PICK(4, kMostFloat4, most_steps(8));
#undef DGQ_PICK
    return {nullptr, nullptr};
}

bool vectorised(const Groups &g) { return g.info.channels % 4 == 0; }

}  // namespace

bool quantize_act_fits(const Groups &g) {
    if (!vectorised(g)) return sizeof(float) * (size_t)g.info.channels * kWavesPerBlock <= 160 * 1024;
    return g.info.channels <= 4 * 256 * kMostFloat4 && g.q_steps <= 4 * most_steps(g.info.act_bits);
}

hipError_t launch_quantize_act(const Groups &g, const float *x, int64_t rows, int8_t *codes,
                               uint8_t *row_class, hipStream_t st, int32_t conv_w, int64_t copy_bytes,
                               const uint32_t *fill32) {
    const int32_t C = g.info.channels, Kp = g.info.k_padded;
    const bool a8 = g.info.act_bits == 8;
    if (!quantize_act_fits(g)) return hipErrorInvalidValue;
    if (!vectorised(g)) {
        if (conv_w > 0) return hipErrorInvalidValue;
        const size_t lds = sizeof(float) * (size_t)C * kWavesPerBlock;
        auto kern = a8 ? k_quantize_act_any<8> : k_quantize_act_any<4>;
        if (lds > 64 * 1024) {
            const hipError_t e = a8 ? DGQ_ENSURE_LDS(k_quantize_act_any<8>, 160 * 1024) : DGQ_ENSURE_LDS(k_quantize_act_any<4>, 160 * 1024);
            if (e != hipSuccess) return e;
        }
        const int64_t blocks = (rows + kWavesPerBlock - 1) / kWavesPerBlock;
        hipLaunchKernelGGL(kern, dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(256), lds, st, x, rows, C, Kp,
                           g.n_chunks, g.d_perm, g.d_chunk_z, g.d_chunk_inv, g.d_taus, g.n_tab - 1, codes, row_class);
        return hipGetLastError();
    }
    // One wavefront per row where its registers hold the tables (1280 channels at 8 bit, 2560 at 4 bit);
    // otherwise four, and also where a row is longer than what the smallest kernels hold and all the workgroups
    // are resident at once, three to a CU with room left (us, one / four: 8-bit 512 x 704 2.67 / 2.93, 512 x 768 3.03 / 2.90,
    // 640 x 768 3.06 / 3.11, 512 x 1280 3.37 / 2.97, 704 x 1280 3.40 / 3.19, 768 x 1280 3.42 / 3.64, 2964 x 1280 5.6 / 6.4; 4-bit
    // 512 x 768 2.80 / 3.03, 512 x 800 3.58 / 3.04, 704 x 2048 4.13 / 3.65, 768 x 2560 4.20 / 4.76, 16384 x 2560 35.6 / 39.9).
    auto wave_holds = [&] {
        const int nv = (C + 255) / 256, ns = g.q_steps;
        return (nv <= 5 && ns <= 8) || (!a8 && nv <= 10 && ns <= 6);
    };
    const int W = wave_holds() && !(rows <= 704 && C >= (a8 ? 768 : 772)) ? 1 : 4;
    const int nv = (C + 256 * W - 1) / (256 * W), ns = (g.q_steps + W - 1) / W;
    // Rows per wavefront (or per workgroup of four sharing them): as many as the chip's resident wavefronts leave
    // over, which spares table reads, but at most four (more leaves the last ones uneven).  A wavefront with
    // more than three output dwords per lane holds half the registers of a SIMD's quarter again: fewer are
    // resident (8148 x 896 with 1728 positions: 14.2 us with one row each, 10.6 with four).
    const int64_t slots = W == 4 ? 512 : (ns <= 3 ? 4096 : 2048);
    const int64_t want = (rows + slots / 2) / slots;
    int32_t per = (int32_t)(want < 1 ? 1 : (want > 4 ? 4 : want));
#ifdef DGQ_TUNING  // tuning builds only
    if (const int v = tuning_value(kTuneQuantRows); v > 0) per = v;
#endif
    const Picked k = conv_w > 0 ? (a8 ? pick<8, true>(W, nv, ns) : pick<4, true>(W, nv, ns))
                                : (a8 ? pick<8, false>(W, nv, ns) : pick<4, false>(W, nv, ns));
    if (!k.kern) return hipErrorInvalidValue;
    const size_t lds = sizeof(float) * (size_t)C * (W == 1 ? kWavesPerBlock : 2) +
                       (g.n_tab > 2 ? sizeof(float2) * (size_t)g.n_tab * g.n_chunks : 0);
    if (lds > 60 * 1024) {
        const hipError_t e = raise_lds_limit(*k.lim, reinterpret_cast<const void *>(k.kern), 128 * 1024);
        if (e != hipSuccess) return e;
    }
    const int64_t per_wg = W == 1 ? (int64_t)kWavesPerBlock * per : per, wgs = (rows + per_wg - 1) / per_wg;
    constexpr int64_t kMostWgs = 1 << 23;  // a grid holds less than 2^32 threads: a launch takes 2^27 rows, or 2^25 shared ones
    for (int64_t wg0 = 0; wg0 < wgs; wg0 += kMostWgs) {
        hipLaunchKernelGGL(k.kern, dim3((unsigned)(wgs - wg0 < kMostWgs ? wgs - wg0 : kMostWgs)), dim3(256), lds, st, x, rows, C,
                           Kp / (a8 ? 4 : 8), g.n_chunks, g.d_q_off, g.d_q_keep, g.d_q_zi, g.d_taus, g.n_tab - 1, codes,
                           row_class, per, conv_w, copy_bytes, fill32, wg0);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace dgq
