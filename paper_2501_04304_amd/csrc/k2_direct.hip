// K2 for small launches: the same contraction as k2_linear.hip (grouped int8 x int8 -> int32, folded
// per group in fp32), for problems whose tiles do not fill the chip.
//
// There a launch is a latency chain: one workgroup per CU walks its K chunks one after the other
// through wait, barrier, LDS read, matrix instruction and fold, 0.27 us per chunk whatever the tile,
// while most of the chip idles.  Here a wavefront owns a small block outright: it reads its operand fragments
// straight from memory into registers, several chunks ahead, and there is no LDS and no barrier.
//   - Groups are summed whole in int32 and folded in order, so every result has the bits that the ring
//     kernel gives it: a row's result does not depend on how many rows are in the call, and never
//     becomes a different code in the quantizer that it meets next.  (Cutting a block's chunks among
//     four wavefronts is 0-15 % faster, but then groups are cut, or folded in another order, or the wavefronts
//     meet at a barrier every four chunks, which costs 20-60 %.)
//   - The matrix instruction is the 16 x 16 x 64 one: its operand is one code block (16 rows x 64 bytes = 1 KiB
//     of contiguous memory per load), and a block of 16 x 16 leaves a group's fold eight vector
//     instructions, so that a chunk is a short link of the chain: about 40 ns, 20 instructions.
//   - Channels are its M index (four consecutive ones per lane) and activation rows its N index
//     (lanes): a row's class selects a per-lane scale, for any number of classes, and results
//     leave 16 bytes per lane.
// What bounds it: the instructions that one wavefront issues per chunk while the launch has less than one per
// SIMD, beyond that its operand traffic (1 KiB per 16 rows or channels, chunk and wavefront), which is why larger
// launches take larger blocks and the ring kernel, whose wavefronts share operands through LDS, the
// largest.  Measured (us, ring kernel / this one): 154 x 768 -> 320 6.4 / 3.4, 512 x 1280 -> 1280 7.7 / 6.6,
// 32 x 1280 -> 10240 8.0 / 5.0, 512 x 5120 -> 1280 17.8 / 14.5; convolutions 2 x 16 x 16 x 1280 -> 1280 67 / 31,
// 2 x 32 x 32 x 640 -> 640 40 / 25, 2 x 64 x 64 x 320 -> 320 31 / 26.
#include <type_traits>

#include "dgq_internal.h"
#include "epilogue.h"

namespace dgq {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));

// Tables and operands read by index from a uniform pointer: scalar loads, and vector loads with a scalar base
// and one 32-bit lane offset for all blocks (the compiler's plain loads spend a 64-bit add per lane and load).
#define DGQ_CONST __attribute__((address_space(4)))
typedef __amdgpu_buffer_rsrc_t Rsrc;
__device__ inline Rsrc rsrc_of(const int8_t *p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(p), 0, 0x7fffffff, 0x00020000);
}

// GEGLU as in k_linear: 0 plain, 1 gated, 2 gated and requantized for the next layer.
// DUMP: the int32 sum of every (row, channel, group), as it is folded.
// A wavefront's block: 16 RB rows x 16 OB channels (gated: OB of the values and the same of the gates); it is a
// workgroup by itself (four with neighbouring blocks measured 5-40 % slower).  AHEAD: chunks in flight.
// EACH: every chunk is a group of its own.
template <int ABITS, int GEGLU, bool MULTI, bool CONV, bool EACH, bool DUMP, int RB, int OB, int AHEAD>
__global__ __launch_bounds__(64, RB * OB * (GEGLU ? 2 : 1) >= 4 ? 3 : 4) void k_linear_direct(
    const int8_t *__restrict__ codes, const uint8_t *__restrict__ row_class,
    const int8_t *__restrict__ wq, const float *__restrict__ sw, const float *__restrict__ zb,
    const float *__restrict__ chunk_s, const uint32_t *__restrict__ chunk_ends, const float *__restrict__ s_tab,
    const float *__restrict__ zoff_tab, int64_t rows, int32_t O, int32_t O_pad, int32_t n_chunks, int32_t tiles_r,
    int32_t tiles_o, int32_t per_xcd,
    float *__restrict__ y, const float2 *__restrict__ rq_zi, const uint8_t *__restrict__ rq_keep,
    uint8_t *__restrict__ rq_cls, int32_t rq_bits, ConvGather cv, int32_t *__restrict__ acc_dump, int32_t NG,
    int32_t n_tab) {
    constexpr int NB = GEGLU ? 2 * OB : OB;        // weight blocks: values, then gates
    constexpr int kARows = ABITS == 8 ? 16 : 32;   // rows per code block

    // ---- workgroup w runs on XCD w % 8: contiguous tile ranges per XCD, in bands of 8 row tiles
    constexpr int32_t kBand = 8;
    const int32_t t = (int32_t)(blockIdx.x & 7) * per_xcd + (int32_t)(blockIdx.x >> 3);
    if (t >= tiles_r * tiles_o) return;
    const int32_t first_r = t / (kBand * tiles_o) * kBand, in_band = t % (kBand * tiles_o);
    const int32_t band = tiles_r - first_r < kBand ? tiles_r - first_r : kBand;
    const int32_t tile_r = first_r + in_band % band, tile_o = in_band / band;
    const int lane = threadIdx.x, n16 = lane & 15, kq = lane >> 4;
    const int64_t r0 = (int64_t)tile_r * (16 * RB);
    const int32_t width = GEGLU ? O / 2 : O;
    const int32_t o0 = tile_o * (16 * OB);  // first output (value) channel

    // ---- fragment addresses: a uniform block pointer plus one lane offset per operand.  Lane (n16, kq) holds
    // positions 16 kq .. + 15 of row n16: a 16-byte slot of 8-bit codes and weights, half a slot of packed codes
    // (whose rows 16..31 keep the halves of a slot swapped).
    const int64_t n_ablocks = (rows + kARows - 1) / kARows;
    int64_t a_blk[RB];
    uint32_t a_in[RB];
    int32_t cls[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const int64_t r = r0 + 16 * b;
        a_blk[b] = r / kARows < n_ablocks ? r / kARows : n_ablocks - 1;  // rows past the end are never stored
        const int tr = (int)(r & 31) + n16;  // row of a 32-row block
        a_in[b] = ABITS == 8 ? n16 * 64 + ((kq ^ swz64(n16)) << 4)
                             : tr * 32 + (((kq >> 1) ^ swz32(tr)) << 4) + (((kq & 1) ^ half32(tr)) << 3);
        cls[b] = row_class[r + n16 < rows ? r + n16 : rows - 1];
    }
    const uint32_t b_in = n16 * 64 + ((kq ^ swz64(n16)) << 4);
    Rsrc a_rsrc[RB], w_rsrc[NB];
    // CONV: one tap's blocks, such that the offset of a weight chunk is that of its codes too; a tap outside the
    // image reads the code of 0
    int32_t cv_h[RB], cv_dx = 0, cv_dy = 0, cv_base = 0, cv_next = CONV ? cv.chunks << 10 : 0;
    auto set_tap = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int64_t blk = a_blk[b] + (int64_t)(cv_dy - 1) * cv.w_blocks;
            a_rsrc[b] = rsrc_of(((uint32_t)(cv_h[b] + cv_dy - 1) < (uint32_t)cv.height
                                     ? codes + cv_dx * cv.copy_bytes + ((blk * cv.chunks) << 10) : cv.fill) - cv_base);
        }
    };
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        cv_h[b] = CONV ? (int32_t)((a_blk[b] / cv.w_blocks) % cv.height) : 0;
        if (!CONV) a_rsrc[b] = rsrc_of(codes + ((a_blk[b] * n_chunks) << 10));
    }
    if (CONV) set_tap();
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int32_t o = b < OB ? o0 + 16 * b : O / 2 + o0 + 16 * (b - OB);  // < O_pad
        w_rsrc[b] = rsrc_of(wq + (((int64_t)(o >> 4) * n_chunks) << 10));
    }

    struct Frag {
        v4i a[RB], w[NB];  // (packed codes: in a's first half)
    };
    // Loads are not conditional (the wait for a chunk is then exact): behind the last chunk they repeat it.
    // A lone wavefront issues an instruction every five clocks or so, whatever its kind: addresses cost one
    // scalar add and minimum per chunk.
    int32_t off = 0;
    const int32_t last_off = (n_chunks - 1) << 10;
    auto load = [&](Frag &f) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            if (ABITS == 8) {
                f.a[b] = __builtin_amdgcn_raw_buffer_load_b128(a_rsrc[b], a_in[b], off, 0);
            } else {
                const v2i q = __builtin_amdgcn_raw_buffer_load_b64(a_rsrc[b], a_in[b], off, 0);
                f.a[b].x = q.x;
                f.a[b].y = q.y;
            }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) f.w[b] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc[b], b_in, off, 0);
        off = off + 1024 < last_off ? off + 1024 : last_off;
        if (CONV && off == cv_next) {
            cv_base = cv_next;
            cv_next += cv.chunks << 10;
            if (++cv_dx == 3) {
                cv_dx = 0;
                ++cv_dy;
            }
            set_tap();
        }
    };
    // The classes first, then the chunks in their order: a wait in the loop is otherwise one for the whole lot.
    Frag f[AHEAD];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
        load(f[u]);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        // a class the layer does not have reads the last one's scale, never past the tables
        const int32_t c = cls[b];
        cls[b] = MULTI ? (c < n_tab ? c : n_tab - 1) : c != 0;
        asm volatile("" : "+v"(cls[b]));
    }

    // Two sets of int32 sums take turns: while the matrix instructions of a chunk run, the sums of a group that
    // ended with the chunk before are folded.
    v4i acc[2][RB][NB];
    float sum[RB][NB][4];
    const v4i zero = {0, 0, 0, 0};
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            acc[1][a][b] = zero;
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[a][b][e] = 0.0f;
        }
    float s_multi[RB];  // MULTI: one group
#pragma unroll
    for (int a = 0; a < RB; ++a) s_multi[a] = MULTI ? s_tab[cls[a]] : 0.0f;
    // rows of one class throughout (almost always: outlier rows are rare) take their scale from a scalar register
    bool any1 = false, all1 = true;
#pragma unroll
    for (int a = 0; a < RB; ++a) {
        const uint64_t m = MULTI || CONV ? 0 : __ballot(cls[a] != 0);
        any1 = any1 || m != 0;
        all1 = all1 && m == ~0ull;
    }
    const DGQ_CONST uint32_t *ends_of = (const DGQ_CONST uint32_t *)(uintptr_t)chunk_ends;

    auto contract = [&](auto mixed_tag) __attribute__((always_inline)) {
        constexpr bool MIXED = decltype(mixed_tag)::value;
        const DGQ_CONST float *scales0 = (const DGQ_CONST float *)(uintptr_t)(chunk_s + (!MIXED && any1 ? n_chunks + Groups::kReadAhead : 0));
        const DGQ_CONST float *scales1 = (const DGQ_CONST float *)(uintptr_t)(chunk_s + n_chunks + Groups::kReadAhead);
        int32_t g = 0;
        auto fold = [&](const v4i (&v)[RB][NB], const float s0, const float s1) __attribute__((always_inline)) {
#pragma unroll
            for (int a = 0; a < RB; ++a) {
                const float s = MULTI ? s_multi[a] : (MIXED && cls[a] ? s1 : s0);
#pragma unroll
                for (int b = 0; b < NB; ++b) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[a][b][e] = fmaf((float)v[a][b][e], s, sum[a][b][e]);
                    if (DUMP) {
                        const int64_t row = r0 + 16 * a + n16;
                        const int32_t o = o0 + 16 * b + 4 * kq;
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (row < rows && o + e < O) acc_dump[(row * O + o + e) * NG + g] = v[a][b][e];
                    }
                }
            }
            if (DUMP) ++g;
        };
        // The scales of a trip's chunks (AHEAD of them) are read a trip ahead: a scalar load takes longer than a chunk.
        static_assert(AHEAD % 2 == 0, "the two sets of sums take turns within a trip");
        struct Scales {
            float s0[AHEAD], s1[AHEAD];
            uint32_t ends;  // bit k: chunk k ends its group
        };
        auto read_scales = [&](Scales &v, int32_t c) __attribute__((always_inline)) {
            if (MULTI) return;
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                v.s0[u] = scales0[c + u];
                if (MIXED) v.s1[u] = scales1[c + u];
            }
            if (!EACH) v.ends = ends_of[c];
        };
        Scales cur, nxt;
        read_scales(nxt, 0);
        // of the chunk before: its group's scales, and (not zero) whether the group ended there
        float last0 = 0.0f, last1 = 0.0f;
        uint32_t ended = 0;
        auto chunk = [&](const int u) __attribute__((always_inline)) {
            v4i (&now)[RB][NB] = acc[u & 1], (&before)[RB][NB] = acc[1 - (u & 1)];
            v4i av[RB];
#pragma unroll
            for (int a = 0; a < RB; ++a) {
                const v4i q = f[u].a[a];
                av[a] = q;
                if (ABITS == 4)  // 16 unsigned nibbles, byte i of a dword holds positions i and i + 4
                    av[a] = v4i{q.x & 0x0f0f0f0f, (int)((uint32_t)q.x >> 4) & 0x0f0f0f0f, q.y & 0x0f0f0f0f,
                                (int)((uint32_t)q.y >> 4) & 0x0f0f0f0f};
            }
            // whether the chunk before ended its group
            const uint32_t end = EACH ? 1 : (MULTI ? 0 : (u > 0 ? cur.ends & (1u << (u - 1)) : ended));
            auto product = [&](auto from) __attribute__((always_inline)) {
#pragma unroll
                for (int a = 0; a < RB; ++a)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        now[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[u].w[b], av[a], from(before[a][b]), 0, 0, 0);
            };
            if (EACH) {
                product([&](const v4i &) { return zero; });
                fold(before, last0, last1);  // (before the first chunk: 0 with scale 0)
            } else if (MULTI) {
                product([&](const v4i &v) { return v; });
            } else if (RB * NB == 1) {  // four masks are less than a second branch
                const int32_t keep = end ? 0 : -1;
                product([&](const v4i &v) { return v & keep; });
                if (end) fold(before, last0, last1);
            } else if (end) {
                product([&](const v4i &) { return zero; });
                fold(before, last0, last1);
            } else {
                product([&](const v4i &v) { return v; });
            }
            if (MULTI) return;
            last0 = cur.s0[u];
            if (MIXED) last1 = cur.s1[u];
            if (!EACH && u == AHEAD - 1) ended = cur.ends & (1u << u);
        };
        int32_t c = 0;
        for (; c + AHEAD <= n_chunks; c += AHEAD) {
            cur = nxt;
            read_scales(nxt, c + AHEAD);
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                chunk(u);
                load(f[u]);
                // left alone the compiler interleaves several chunks and runs out of registers
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        cur = nxt;
#pragma unroll
        for (int u = 0; u < AHEAD - 1; ++u)
            if (c + u < n_chunks) chunk(u);
        if (n_chunks & 1)
            fold(acc[0], last0, last1);
        else
            fold(acc[1], last0, last1);
    };
    if constexpr (MULTI || CONV) {
        contract(std::false_type{});
    } else if constexpr (RB * NB > 1) {
        contract(std::true_type{});  // (the selection is a smaller part of a larger block's fold)
    } else {
        if (any1 && !all1)
            contract(std::true_type{});
        else
            contract(std::false_type{});
    }

    // ---- register e of a block: channel 4 kq + e of row n16
#pragma unroll
    for (int a = 0; a < RB; ++a) {
        const int64_t row = r0 + 16 * a + n16;
        const bool live = row < rows;
        const float zo = MULTI ? zoff_tab[cls[a]] : 0.0f;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int32_t o = (b < OB ? o0 + 16 * b : O / 2 + o0 + 16 * (b - OB)) + 4 * kq;  // < O_pad
            const float4 w4 = *reinterpret_cast<const float4 *>(sw + o);
            float4 z = *reinterpret_cast<const float4 *>(zb + (!MULTI && cls[a] ? O_pad : 0) + o);
            if (MULTI) {
                const float4 z1 = *reinterpret_cast<const float4 *>(zb + O_pad + o);
                z = make_float4(fmaf(zo, z.x, z1.x), fmaf(zo, z.y, z1.y), fmaf(zo, z.z, z1.z), fmaf(zo, z.w, z1.w));
            }
            sum[a][b][0] = fmaf(w4.x, sum[a][b][0], z.x);
            sum[a][b][1] = fmaf(w4.y, sum[a][b][1], z.y);
            sum[a][b][2] = fmaf(w4.z, sum[a][b][2], z.z);
            sum[a][b][3] = fmaf(w4.w, sum[a][b][3], z.w);
        }
#pragma unroll
        for (int b = 0; b < OB; ++b) {
            float(&h)[4] = sum[a][b];
            const int32_t oc = o0 + 16 * b + 4 * kq;
            if (GEGLU) {
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] *= gelu(sum[a][GEGLU ? OB + b : b][e]);
            }
            if (GEGLU == 2) {
                // the next layer's quantizer, as in k_linear: the channels are that layer's positions
                const int32_t chunk = oc >> 6, nch2 = O >> 7;
                const float2 zi = rq_zi[chunk];
                uint32_t pk = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float u = __fmul_rn(__fsub_rn(h[e], zi.x), zi.y);
                    if (rq_bits == 4) u = __builtin_amdgcn_fmed3f(u, 0.0f, 15.0f);
                    pk = __builtin_amdgcn_cvt_pk_u8_f32(u, e, pk);
                }
                if (rq_bits == 8) pk ^= 0x80808080u;
                pk &= *reinterpret_cast<const uint32_t *>(rq_keep + oc);
                int8_t *out = reinterpret_cast<int8_t *>(y);
                if (rq_bits == 4) {  // a dword holds eight positions: byte i those of i (low nibble) and i + 4
                    const uint32_t high = (uint32_t)__shfl_down((int)pk, 16, 64);
                    const int e8 = (oc & 63) >> 3;
                    if (live && !(kq & 1))
                        *reinterpret_cast<uint32_t *>(out + tiled32_offset(row, chunk, nch2, e8 >> 2) +
                                                      (((e8 & 3) ^ (2 * half32((int)(row & 31)))) << 2)) = pk | (high << 4);
                } else if (live) {
                    const int e4 = (oc & 63) >> 2;
                    *reinterpret_cast<uint32_t *>(out + tiled64_offset(row, chunk, nch2, e4 >> 2) + ((e4 & 3) << 2)) = pk;
                }
                if (o0 == 0 && b == 0 && kq == 0 && live) rq_cls[row] = 0;
            } else if (live) {
                float *dst = y + row * width + oc;
                if ((width & 3) == 0) {
                    if (oc < width) *reinterpret_cast<float4 *>(dst) = make_float4(h[0], h[1], h[2], h[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (oc + e < width) dst[e] = h[e];
                }
            }
        }
    }
}

struct Call {
    int block;
    const Groups &g;
    const Weight &w;
    const int8_t *codes;
    const uint8_t *row_class;
    int64_t rows;
    float *y;
    uint8_t *rq_cls;
    ConvGather cv;
    int32_t *acc_dump;
    hipStream_t st;
};

template <int ABITS, int GEGLU, bool MULTI, bool CONV, bool EACH, bool DUMP, int RB, int OB, int AHEAD>
hipError_t launch(const Call &c) {
    static_assert(AHEAD <= Groups::kReadAhead, "the tables are read a trip ahead");
    constexpr int TR = 16 * RB, TO = 16 * OB;
    const Groups &g = c.g;
    const Weight &w = c.w;
    const int32_t tiles_r = (int32_t)((c.rows + TR - 1) / TR), tiles_o = ((GEGLU ? w.O / 2 : w.O) + TO - 1) / TO;
    const int32_t per_xcd = (int32_t)(((int64_t)tiles_r * tiles_o + 7) / 8);
    hipLaunchKernelGGL((k_linear_direct<ABITS, GEGLU, MULTI, CONV, EACH, DUMP, RB, OB, AHEAD>), dim3((unsigned)(per_xcd * 8)),
                       dim3(64), 0, c.st, c.codes, c.row_class, w.d_wq, w.d_sw, w.d_zb, g.d_chunk_s, g.d_chunk_ends,
                       g.d_s, g.d_zoff, c.rows, w.O, w.O_pad, g.n_chunks, tiles_r, tiles_o, per_xcd, c.y, w.d_rq_zi,
                       w.d_rq_keep, c.rq_cls, w.next_bits, c.cv, c.acc_dump, g.info.n_groups, g.n_tab);
    return hipGetLastError();
}

template <int ABITS, int GEGLU, bool MULTI, bool CONV, bool EACH, bool DUMP>
hipError_t launch_block(const Call &c) {
#define DGQ_BLOCK(...) return launch<ABITS, GEGLU, MULTI, CONV, EACH, DUMP, __VA_ARGS__>(c)
    if (c.block == 0) DGQ_BLOCK(1, 1, 6);
    if constexpr (GEGLU) {
        DGQ_BLOCK(2, 1, 4);
    } else {
        if (c.block == 1) DGQ_BLOCK(1, 2, 4);
        DGQ_BLOCK(2, 2, 4);
    }
#undef DGQ_BLOCK
}

template <int GEGLU, bool MULTI, bool CONV, bool DUMP>
hipError_t launch_kind(const Call &c) {
    const bool a8 = c.g.info.act_bits == 8;
    if constexpr (!MULTI && !DUMP) {
        if (c.g.info.n_groups == c.g.n_chunks)
            return a8 ? launch_block<8, GEGLU, MULTI, CONV, true, DUMP>(c) : launch_block<4, GEGLU, MULTI, CONV, true, DUMP>(c);
    }
    return a8 ? launch_block<8, GEGLU, MULTI, CONV, false, DUMP>(c) : launch_block<4, GEGLU, MULTI, CONV, false, DUMP>(c);
}

}  // namespace

// Which block, or -1 where the ring kernel is the faster one.  For T blocks of 32 x 32 outputs, n chunks and g groups
// the times in ns, fitted to a sweep over 19 .. 16384 rows, 64 .. 11520 channels and 128 .. 10240 outputs (linear
// layers, gated ones and convolutions, both code widths, 280 launches: the rule's choice is 0.5 % off the fastest of all
// blocks and tiles on average, 20 % at most): this kernel takes its chain of chunks (and a branch per group where groups are
// longer than a chunk) or its traffic, whichever is longer, and a third of the other; the ring kernel takes 1.3 us
// more to start, then its chain of chunks and folds or its throughput per 64 x 64 tile.
// The blocks by T: 16 x 16 up to 384, i.e. 1.5 wavefronts per SIMD (512 x 2560 -> 640, T = 320: 6.8 us against 7.8 with 16 x 32;
// 300 x 320 -> 1280, T = 400: 4.04 / 4.00), 16 x 32 up to 1024 (1024 x 2560 -> 640, T = 640: 8.9 against 10.4 with 32 x 32; 2 x 32 x 32 x
// 320 -> 640 convolution, T = 1280: 18.8 / 16.0).  One group leaves the loop without folds: 32 x 32 from 512 on (512 x 5120 ->
// 1280, T = 640: 14.1 / 10.7).  A gated layer's 16 x 16 blocks come with their gates, and their epilogue wants more
// wavefronts: up to 1024 (300 x 640 -> 2560, T = 800: 5.4 / 5.7 with 32 x 16; 512 x 320 -> 2560, T = 1280: 6.5 / 5.8).
int direct_block(const LinearShape &s) {
    const int64_t t32 = ((s.rows + 31) / 32) * ((s.out_channels + 31) / 32);
    const int64_t t64 = ((s.rows + 63) / 64) * ((s.out_channels + 63) / 64);
    int block = s.gated ? (t32 <= 1024 ? 0 : 2) : (t32 <= 384 ? 0 : (t32 <= (s.multi ? 512 : 1024) ? 1 : 2));
#ifdef DGQ_TUNING
    if (const int v = tuning_value(kTuneSuperRows); v > 0) block = v - 1;
    if (const int v = tuning_value(kTuneLinearCfg); v > 0) return v == 1 ? block : -1;
#endif
    // the chip is full (this also keeps the tile counts in range); 32-bit offsets into a row of code blocks
    if (t64 > 1024 || s.n_chunks > (1 << 20)) return -1;
    const double per_chunk[3] = {42.0, 35.0, 47.0}, traffic[3] = {0.22, 0.20, 0.15};
    const double n = s.n_chunks, g = s.n_groups;
    const double chain = per_chunk[block] * n + (g == n ? 0.0 : 12.0 * g);
    const double flow = (double)t32 * (1.37 + traffic[block] * n);
    const double ring_chain = (s.conv ? 197.0 : 115.0) * n + 141.0 * g;
    const double ring_flow = (double)t64 * (1.08 + (s.conv ? 0.50 : 0.28) * n + 0.23 * g);
    const double direct = 2830.0 + (chain > flow ? chain + 0.35 * flow : flow + 0.35 * chain);
    return direct < 4190.0 + (ring_chain > ring_flow ? ring_chain : ring_flow) ? block : -1;
}

hipError_t launch_linear_direct(int block, const Groups &g, const Weight &w, const int8_t *codes, const uint8_t *row_class,
                                int64_t rows, float *y, int geglu, uint8_t *rq_cls, const ConvGather *cv,
                                int32_t *acc_dump, hipStream_t st) {
    const Call c{block, g, w, codes, row_class, rows, y, rq_cls, cv ? *cv : ConvGather(), acc_dump, st};
    if (cv) return launch_kind<0, false, true, false>(c);
    if (geglu == 2) return launch_kind<2, false, false, false>(c);
    if (geglu == 1) return launch_kind<1, false, false, false>(c);
    if (acc_dump) return launch_kind<0, false, false, true>(c);
    return g.n_tab > 2 ? launch_kind<0, true, false, false>(c) : launch_kind<0, false, false, false>(c);
}

}  // namespace dgq
