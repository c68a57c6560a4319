// K2 for small launches: the same contraction as k2_linear.hip (grouped int8 x int8 -> int32, folded
// per group in fp32), for problems whose tiles do not fill the chip.
//
// There a launch is a latency chain: one workgroup per CU walks its K chunks one after the other
// through wait, barrier, LDS read, matrix instruction and fold, 0.27 us per chunk whatever the tile,
// while most of the chip idles.  So the chain is cut: the four wavefronts of a workgroup take a
// quarter of the chunks each of the SAME 32 x 32 output block, read their operand fragments straight from
// memory into registers (two chunks ahead, no LDS ring, no barrier), and add up through LDS once, at the end.
//   - The gated forms keep one wavefront per block (their layers are wide: there are blocks enough) and fold
//     whole groups in order, exactly as the ring kernel does: their results meet a quantizer next, and
//     a last bit that depends on the kernel would now and then become a different code.
//   - Otherwise every chunk is folded by itself with the scale of its group (one value per lane, read with the
//     fragments): no group bookkeeping, and a group may be cut between two wavefronts.
//   - Channels are the matrix instruction's M index (registers) and activation rows its N index
//     (lanes): a row's class then selects a per-lane scale, for any number of classes, and after
//     the sum through LDS the results leave 16 bytes per lane, 128 contiguous bytes per row.
// What bounds it beyond the smallest sizes is the vector cache: a 32 x 32 block takes 4 KB of
// fragments per chunk (16-byte pieces of 64-byte rows, about 40 bytes per clock and CU = 20 TB/s over the
// chip; wavefronts of one workgroup sharing rows or columns, wider wavefront tiles and a wave-private
// LDS ring measured the same or slower), so the ring kernel, which shares fragments through LDS, takes over once
// the chip is full.  Measured (us, before: the ring kernel): 154 x 768 -> 320 6.8 -> 3.3, 512 x 1280 -> 1280
// 9.0 -> 5.7, 32 x 1280 -> 10240 9.2 -> 4.6; convolutions 2 x 16 x 16 x 1280 -> 1280 65 -> 28, 2 x 32 x 32 x 640 -> 640
// (4-bit) 49 -> 24, 2 x 64 x 64 x 320 -> 320 29.5 -> 25.
#include "dgq_internal.h"
#include "epilogue.h"

namespace dgq {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// wavefronts that share the K range of a block (2 and 8 measured up to 10 % slower)
constexpr int slices(int geglu) { return geglu ? 1 : 4; }
constexpr int kAhead = 2;   // chunks in flight per wavefront (3 and 4 need registers that cost occupancy: slower)

__global__ __launch_bounds__(256) void k_clear(int32_t *__restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0;
}

// GEGLU as in k_linear: 0 plain, 1 gated, 2 gated and requantized for the next layer.
// DUMP: the int32 sums of every (row, channel, group), added up over the group's chunks in acc_dump
// (which starts at zero); the results keep their bits.
template <int ABITS, int GEGLU, bool MULTI, bool CONV, bool DUMP>
__global__ __launch_bounds__(64 * slices(GEGLU) * (GEGLU ? 2 : 1), 4) void k_linear_direct(
    const int8_t *__restrict__ codes, const uint8_t *__restrict__ row_class,
    const int8_t *__restrict__ wq, const float *__restrict__ sw, const float *__restrict__ zb,
    const float *__restrict__ chunk_s, const float *__restrict__ zoff_tab, int64_t rows, int32_t O,
    int32_t O_pad, int32_t n_chunks, int32_t tiles_r, int32_t tiles_o, int32_t per_xcd,
    float *__restrict__ y, const float2 *__restrict__ rq_zi, const uint8_t *__restrict__ rq_keep,
    uint8_t *__restrict__ rq_cls, int32_t rq_bits, ConvGather cv, int32_t *__restrict__ acc_dump,
    const int32_t *__restrict__ gchunk, int32_t NG, int32_t n_tab) {
    constexpr int kSlices = slices(GEGLU);
    constexpr int WO = GEGLU ? 2 : 1;       // column blocks of a workgroup: the channels, or value and gate
    constexpr int kThreads = 64 * kSlices * WO;
    constexpr int PITCH = 32 * WO + 4;      // floats per row of a slice's partial sums
    constexpr int NA = ABITS == 8 ? 2 : 1;  // 16-byte activation fragments per chunk
    __shared__ __attribute__((aligned(16))) float part[kSlices][32 * PITCH];

    // ---- workgroup w runs on XCD w % 8: contiguous tile ranges per XCD, in bands of 8 row tiles
    constexpr int32_t kBand = 8;
    const int32_t t = (int32_t)(blockIdx.x & 7) * per_xcd + (int32_t)(blockIdx.x >> 3);
    if (t >= tiles_r * tiles_o) return;
    const int32_t first_r = t / (kBand * tiles_o) * kBand, in_band = t % (kBand * tiles_o);
    const int32_t band = tiles_r - first_r < kBand ? tiles_r - first_r : kBand;
    const int32_t tile_r = first_r + in_band % band, tile_o = in_band / band;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int slice = wave / WO, wo = wave % WO;
    const int m32 = lane & 31, kh = lane >> 5;
    const int64_t r0 = (int64_t)tile_r * 32;
    const int32_t o0 = tile_o * 32;  // first output (value) channel
    const int32_t c_begin = n_chunks * slice / kSlices, c_end = n_chunks * (slice + 1) / kSlices;

    // ---- fragment addresses: uniform block pointers plus one lane offset per operand.  8-bit codes:
    // a lane reads slots kh and kh + 2 of its row (k-steps 0 and 1).  Packed 4-bit codes: one slot holds
    // both k-steps of a lane, positions 32 kh .. + 31, so the weights come from slots 2 kh and 2 kh + 1.
    constexpr int kARows = ABITS == 8 ? 16 : 32;
    const int64_t n_ablocks = (rows + kARows - 1) / kARows, a_blk0 = r0 / kARows;
    int64_t a_blk = a_blk0 + (ABITS == 8 ? m32 >> 4 : 0);
    a_blk = a_blk < n_ablocks ? a_blk : n_ablocks - 1;  // rows past the end are never stored
    const uint32_t a_in = ABITS == 8 ? (m32 & 15) * 64 + ((kh ^ swz64(m32 & 15)) << 4)
                                     : m32 * 32 + ((kh ^ swz32(m32)) << 4);
    const int8_t *a_base = codes + ((a_blk0 * n_chunks) << 10);
    const uint32_t a_off = (uint32_t)(a_blk - a_blk0) * (uint32_t)n_chunks * 1024u + a_in;
    const int32_t ch0 = GEGLU && wo ? O / 2 + o0 : o0;  // first channel of the wave's block
    const int8_t *b_base = wq + (((int64_t)(ch0 >> 4) * n_chunks) << 10);
    const uint32_t b_off = (uint32_t)(m32 >> 4) * (uint32_t)n_chunks * 1024u + (m32 & 15) * 64 +
                           (((ABITS == 8 ? kh : 2 * kh) ^ swz64(m32 & 15)) << 4);
    constexpr uint32_t kBStep = ABITS == 8 ? 32 : 16;  // between the two k-steps' slots (XOR)

    int32_t cls = row_class[r0 + m32 < rows ? r0 + m32 : rows - 1];
    // a class the layer does not have reads the last one's scale, never past the tables
    if (MULTI) cls = cls < n_tab ? cls : n_tab - 1;
    else cls = cls != 0;
    const float *s_row = chunk_s + (int64_t)cls * n_chunks;

    // CONV: the lane's row block in the centre tap of copy 0, and which of the image rows above, at
    // and below it exist; the tap and the chunk inside it of the next chunk to load are running counters
    const int8_t *cv_row = nullptr;
    uint32_t cv_ok = 0;
    int32_t cv_c = 0, cv_dx = 0, cv_dy = 0;
    if (CONV) {
        const int32_t tap = c_begin / cv.chunks;
        cv_c = c_begin - tap * cv.chunks;
        cv_dy = tap / 3;
        cv_dx = tap - 3 * cv_dy;
        const int32_t h = (int32_t)((a_blk / cv.w_blocks) % cv.height);
        cv_ok = 2u | (h > 0 ? 1u : 0u) | (h + 1 < cv.height ? 4u : 0u);
        cv_row = codes + ((a_blk * cv.chunks) << 10) + a_in;
    }

    struct Frag {
        v4i a[NA], b[2];
        float s;
    };
    auto load = [&](Frag &f, int32_t c) __attribute__((always_inline)) {
        const int64_t co = (int64_t)c << 10;
        if (CONV) {
            const int64_t shift = cv_dx * cv.copy_bytes +
                                  (((int64_t)(cv_dy - 1) * cv.w_blocks * cv.chunks + cv_c) << 10);
            const int8_t *p = (cv_ok >> cv_dy) & 1 ? cv_row + shift : cv.fill + ((uint32_t)cv_c << 10) + a_in;
            f.a[0] = *reinterpret_cast<const v4i *>(p);
            if (NA == 2)  // blocks are 1 KiB aligned: the other slot is one address bit away
                f.a[NA - 1] = *reinterpret_cast<const v4i *>(p + (int32_t)(a_in ^ 32u) - (int32_t)a_in);
            if (++cv_c == cv.chunks) {
                cv_c = 0;
                if (++cv_dx == 3) {
                    cv_dx = 0;
                    ++cv_dy;
                }
            }
        } else {
            f.a[0] = *reinterpret_cast<const v4i *>(a_base + co + a_off);
            if (NA == 2) f.a[NA - 1] = *reinterpret_cast<const v4i *>(a_base + co + (a_off ^ 32u));
        }
        f.b[0] = *reinterpret_cast<const v4i *>(b_base + co + b_off);
        f.b[1] = *reinterpret_cast<const v4i *>(b_base + co + (b_off ^ kBStep));
        f.s = s_row[c];
    };
    Frag f[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
        if (c_begin + u < c_end) load(f[u], c_begin + u);

    // ---- the epilogue's constants travel with the first fragments: a thread finishes four
    // consecutive channels (of the value half, and the same four of the gate half)
    const int piece = tid & 7;
    const int32_t oc = o0 + 4 * piece;  // < O_pad always
    float4 c_sw[WO], c_z0[WO], c_z1[WO];
#pragma unroll
    for (int w = 0; w < WO; ++w) {
        const int32_t o = oc + w * (O / 2);
        c_sw[w] = *reinterpret_cast<const float4 *>(sw + o);
        c_z0[w] = *reinterpret_cast<const float4 *>(zb + o);
        c_z1[w] = *reinterpret_cast<const float4 *>(zb + O_pad + o);
    }

    float sum[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) sum[i] = 0.0f;
    auto a_operand = [&](const Frag &fr, int ks) __attribute__((always_inline)) {
        if (ABITS == 8) return fr.a[ks % NA];
        // 16 unsigned nibbles, byte i of a dword holds positions i and i + 4; rows 16..31 keep the
        // 8-byte halves of a slot swapped
        const bool low = (ks == 0) != (half32(m32) != 0);
        const uint32_t p = (uint32_t)(low ? fr.a[0].x : fr.a[0].z), q = (uint32_t)(low ? fr.a[0].y : fr.a[0].w);
        return v4i{(int)(p & 0x0f0f0f0fu), (int)((p >> 4) & 0x0f0f0f0fu), (int)(q & 0x0f0f0f0fu),
                   (int)((q >> 4) & 0x0f0f0f0fu)};
    };
    const v16i zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    v16i acc = zero;
    int32_t g = 0, g_end = GEGLU ? gchunk[1] : 0;  // whole groups: the running one and its end
    auto step = [&](const bool more, Frag &fr, int32_t c) __attribute__((always_inline)) {
        const float s = fr.s;
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr.b[0], a_operand(fr, 0), GEGLU ? acc : zero, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(fr.b[1], a_operand(fr, 1), acc, 0, 0, 0);
        if (DUMP) {
            int32_t gd = 0;
            while (gd + 1 < NG && gchunk[gd + 1] <= c) ++gd;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int32_t o = ch0 + 8 * (i >> 2) + 4 * kh + (i & 3);
                if (r0 + m32 < rows && o < O) atomicAdd(acc_dump + ((r0 + m32) * O + o) * NG + gd, acc[i]);
            }
        }
        if (more) load(fr, c + kAhead);
        // left alone the compiler interleaves several steps and runs out of registers
        __builtin_amdgcn_sched_barrier(0);
        if (!GEGLU || c + 1 == g_end) {
#pragma unroll
            for (int i = 0; i < 16; ++i) sum[i] = fmaf((float)acc[i], s, sum[i]);
            if (GEGLU) {
                acc = zero;
                g_end = ++g < NG ? gchunk[g + 1] : 0;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    int32_t c = c_begin;
    for (; c + 2 * kAhead <= c_end; c += kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) step(true, f[u], c + u);
    }
#pragma unroll
    for (int u = 0; u < 2 * kAhead; ++u)
        if (c + u < c_end) step(u < kAhead && c + u + kAhead < c_end, f[u % kAhead], c + u);

    // ---- the slices' sums meet in LDS (register i: channel 8 (i / 4) + 4 kh + i % 4 of row m32)
#pragma unroll
    for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4 *>(&part[slice][m32 * PITCH + 32 * wo + 8 * q + 4 * kh]) =
            make_float4(sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]);
    __syncthreads();

#pragma unroll
    for (int rl = tid >> 3; rl < 32; rl += kThreads / 8) {  // row of the block
        const int64_t row = r0 + rl;
        const bool live = row < rows;
        float h[WO][4];
        if (live) {
            int32_t cl = row_class[row];
            if (MULTI) cl = cl < n_tab ? cl : n_tab - 1;
            const float zo = MULTI ? zoff_tab[cl] : 0.0f;
#pragma unroll
            for (int w = 0; w < WO; ++w) {
                const float *p = &part[0][rl * PITCH + 32 * w + 4 * piece];
                float4 v = *reinterpret_cast<const float4 *>(p);
#pragma unroll
                for (int k = 1; k < kSlices; ++k) {
                    const float4 u = *reinterpret_cast<const float4 *>(p + k * 32 * PITCH);
                    v = make_float4(v.x + u.x, v.y + u.y, v.z + u.z, v.w + u.w);
                }
                const float4 z0 = c_z0[w], z1 = c_z1[w];
                const float4 z = MULTI ? make_float4(fmaf(zo, z0.x, z1.x), fmaf(zo, z0.y, z1.y), fmaf(zo, z0.z, z1.z), fmaf(zo, z0.w, z1.w))
                                       : (cl ? z1 : z0);
                h[w][0] = fmaf(c_sw[w].x, v.x, z.x);
                h[w][1] = fmaf(c_sw[w].y, v.y, z.y);
                h[w][2] = fmaf(c_sw[w].z, v.z, z.z);
                h[w][3] = fmaf(c_sw[w].w, v.w, z.w);
            }
            if (GEGLU) {
#pragma unroll
                for (int e = 0; e < 4; ++e) h[0][e] *= gelu(h[WO - 1][e]);
            }
        }
        if (GEGLU == 2) {
            // the next layer's quantizer, as in k_linear: the channels are that layer's positions
            const int32_t chunk = oc >> 6, nch2 = O >> 7;
            const float2 zi = rq_zi[chunk];
            uint32_t pk = 0;
            if (live) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float u = __fmul_rn(__fsub_rn(h[0][e], zi.x), zi.y);
                    if (rq_bits == 4) u = __builtin_amdgcn_fmed3f(u, 0.0f, 15.0f);
                    pk = __builtin_amdgcn_cvt_pk_u8_f32(u, e, pk);
                }
                if (rq_bits == 8) pk ^= 0x80808080u;
                pk &= *reinterpret_cast<const uint32_t *>(rq_keep + oc);
            }
            int8_t *out = reinterpret_cast<int8_t *>(y);
            if (rq_bits == 4) {  // a dword holds eight positions: byte i those of i (low nibble) and i + 4
                const uint32_t high = (uint32_t)__shfl_down((int)pk, 1, 64);
                const int e8 = (oc & 63) >> 3;
                if (live && !(piece & 1))
                    *reinterpret_cast<uint32_t *>(out + tiled32_offset(row, chunk, nch2, e8 >> 2) +
                                                  (((e8 & 3) ^ (2 * half32((int)(row & 31)))) << 2)) = pk | (high << 4);
            } else if (live) {
                const int e4 = (oc & 63) >> 2;
                *reinterpret_cast<uint32_t *>(out + tiled64_offset(row, chunk, nch2, e4 >> 2) + ((e4 & 3) << 2)) = pk;
            }
            if (tile_o == 0 && live && piece == 0) rq_cls[row] = 0;
            continue;
        }
        if (!live) continue;
        const int32_t width = GEGLU ? O / 2 : O;
        float *dst = y + row * width + oc;
        if ((width & 3) == 0) {
            if (oc < width) *reinterpret_cast<float4 *>(dst) = make_float4(h[0][0], h[0][1], h[0][2], h[0][3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (oc + e < width) dst[e] = h[0][e];
        }
    }
}

template <int ABITS, int GEGLU, bool MULTI, bool CONV, bool DUMP = false>
hipError_t launch(const Groups &g, const Weight &w, const int8_t *codes, const uint8_t *row_class, int64_t rows,
                  float *y, uint8_t *rq_cls, const ConvGather &cv, int32_t *acc_dump, hipStream_t st) {
    const int32_t tiles_r = (int32_t)((rows + 31) / 32), tiles_o = ((GEGLU ? w.O / 2 : w.O) + 31) / 32;
    const int32_t per_xcd = (int32_t)(((int64_t)tiles_r * tiles_o + 7) / 8);
    if (DUMP) {
        const int64_t n = rows * w.O * g.info.n_groups;
        hipLaunchKernelGGL(k_clear, dim3((unsigned)(n > 2048 * 256 ? 2048 : (n + 255) / 256)), dim3(256), 0, st, acc_dump, n);
    }
    hipLaunchKernelGGL((k_linear_direct<ABITS, GEGLU, MULTI, CONV, DUMP>), dim3((unsigned)(per_xcd * 8)),
                       dim3(64 * slices(GEGLU) * (GEGLU ? 2 : 1)), 0, st, codes, row_class, w.d_wq, w.d_sw, w.d_zb,
                       g.d_chunk_s, g.d_zoff, rows, w.O, w.O_pad, g.n_chunks, tiles_r, tiles_o, per_xcd, y,
                       w.d_rq_zi, w.d_rq_keep, rq_cls, w.next_bits, cv, acc_dump, g.d_gchunk, g.info.n_groups, g.n_tab);
    return hipGetLastError();
}

}  // namespace

// Both kernels' times in ns, fitted to a sweep over 19 .. 16384 rows, 128 .. 11520 channels and 64 .. 10240
// outputs (linear layers and convolutions, 80 shapes), for T tiles of 64 x 64 with n chunks and g groups:
// this kernel takes its traffic, T (4 + 0.66 n) (4-bit codes: 0.53), the ring kernel 1000 more to
// start and then its latency chain, 130 per chunk and 100 per group (a convolution's tables: 80 more per
// chunk), or its throughput, per tile 1.5 + 0.25 n + 0.35 g (convolution: 0.1 n more), whichever is longer.
// Unfolded and gathered convolutions take the same kernel, so that their results have the same bits.
bool linear_direct_pays(const Groups &g, int64_t rows, int64_t out_channels) {
#ifdef DGQ_TUNING
    if (const int v = tuning_value(kTuneLinearCfg); v > 0) return v == 1;
#endif
    const int64_t tiles = ((rows + 63) / 64) * ((out_channels + 63) / 64);
    if (tiles > 1024) return false;  // the chip is full (this also keeps the kernel's tile counts in range)
    const double T = (double)tiles, n = g.n_chunks, ng = g.info.n_groups;
    const double direct = T * (4.0 + (g.info.act_bits == 8 ? 0.66 : 0.53) * n);
    const double chain = (g.conv_taps ? 210.0 : 130.0) * n + 100.0 * ng;
    const double flow = T * (1.5 + (g.conv_taps ? 0.35 : 0.25) * n + 0.35 * ng);
    return direct < 1000.0 + (chain > flow ? chain : flow);
}

hipError_t launch_linear_direct(const Groups &g, const Weight &w, const int8_t *codes, const uint8_t *row_class,
                                int64_t rows, float *y, int geglu, uint8_t *rq_cls, const ConvGather *cv,
                                int32_t *acc_dump, hipStream_t st) {
    const bool a8 = g.info.act_bits == 8, multi = g.n_tab > 2;
#define DGQ_DIRECT(GEGLU, MULTI, CONV, SRC)                                                              \
    return a8 ? launch<8, GEGLU, MULTI, CONV>(g, w, codes, row_class, rows, y, rq_cls, SRC, nullptr, st) \
              : launch<4, GEGLU, MULTI, CONV>(g, w, codes, row_class, rows, y, rq_cls, SRC, nullptr, st)
    if (cv) DGQ_DIRECT(0, false, true, *cv);
    if (geglu == 2) DGQ_DIRECT(2, false, false, ConvGather());
    if (geglu == 1) DGQ_DIRECT(1, false, false, ConvGather());
    if (acc_dump)
        return a8 ? launch<8, 0, false, false, true>(g, w, codes, row_class, rows, y, rq_cls, ConvGather(), acc_dump, st)
                  : launch<4, 0, false, false, true>(g, w, codes, row_class, rows, y, rq_cls, ConvGather(), acc_dump, st);
    if (multi) DGQ_DIRECT(0, true, false, ConvGather());
    DGQ_DIRECT(0, false, false, ConvGather());
#undef DGQ_DIRECT
}

}  // namespace dgq
