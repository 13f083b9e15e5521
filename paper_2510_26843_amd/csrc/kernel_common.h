// Device helpers shared by the gfx950 kernels (kernels.hip, prefill.hip):
// reductions, activation conversion, MFMA steps, the GEMM epilogues, and the
// attention's softmax and merge steps.
#pragma once
#include "cas_internal.h"
#include <type_traits>

#include <hip/hip_runtime.h>
#include <math.h>

namespace cas {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

template <typename AT> struct Act;
template <> struct Act<float> {
    static __device__ __forceinline__ float ld(const float* p, size_t i) { return p[i]; }
    static __device__ __forceinline__ void st(float* p, size_t i, float v) { p[i] = v; }
    static __device__ __forceinline__ float round(float v) { return v; }
};
template <> struct Act<uint16_t> {
    static __device__ __forceinline__ float ld(const uint16_t* p, size_t i) { return bf2f(p[i]); }
    static __device__ __forceinline__ void st(uint16_t* p, size_t i, float v) { p[i] = f2bf(v); }
    static __device__ __forceinline__ float round(float v) { return bf2f(f2bf(v)); }
};

// ---------------------------------------------------------------- reductions

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
// Block-wide maximum for 256 threads.
__device__ __forceinline__ float block_max256(float v, float* sh) {
    v = wave_max(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[w] = v;
    __syncthreads();
    return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

// Reductions over a workgroup of W waves (sh: W floats of LDS); the wave
// partials are combined in wave order, so every thread gets the same value.
template <int W>
__device__ __forceinline__ float block_sum(float v, float* sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = sh[0];
#pragma unroll
    for (int w = 1; w < W; ++w) r += sh[w];
    return r;
}
template <int W>
__device__ __forceinline__ float block_max(float v, float* sh) {
    v = wave_max(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = sh[0];
#pragma unroll
    for (int w = 1; w < W; ++w) r = fmaxf(r, sh[w]);
    return r;
}

// Code of x at scale sc in [-qm, qm] (qm 127: int8, 7: int4).
__device__ __forceinline__ float qcode(float x, float sc, float qm) {
    return sc != 0.f ? fminf(fmaxf(rintf(x / sc), -qm), qm) : 0.f;
}
// Largest magnitude of 8 bf16 values (16 bytes).
__device__ __forceinline__ float amax_bf8(const i32x4 v) {
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t w = (uint32_t)v[i];
        m = fmaxf(m, fmaxf(fabsf(__uint_as_float(w << 16)), fabsf(__uint_as_float(w & 0xffff0000u))));
    }
    return m;
}

// The attention output of one query row of one head at 4 consecutive d: the
// KV splits' partial states merged in split order with a running max
// (online softmax), eight splits' (m, l) pairs and partial outputs loaded at
// a time (one round of loads for contexts up to 2048 slots), then
// normalised.  row = head * T + t.
__device__ __forceinline__ f32x4 attn_merge_row_hd(const AttnArgs& a, int S, size_t row, int d4, int HD) {
#pragma clang fp contract(off)
    const size_t sstride = (size_t)a.H * a.T;  // rows between splits
    float M = -1e30f, L = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < S; s0 += 8) {
        float2 ml[8];
        f32x4 po[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const size_t r = row + (size_t)min(s0 + k, S - 1) * sstride;
            ml[k] = *(const float2*)(a.part_ml + r * 2);
            po[k] = *(const f32x4*)(a.part_o + r * HD + d4);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (s0 + k < S) {
                const float mn = fmaxf(M, ml[k].x);
                const float fo = exp2f(M - mn), fn = exp2f(ml[k].x - mn);
                acc = acc * fo + po[k] * fn;
                L = L * fo + ml[k].y * fn;
                M = mn;
            }
        }
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    return acc * inv;
}
template <int HD>
__device__ __forceinline__ f32x4 attn_merge_row(const AttnArgs& a, int S, size_t row, int d4) {
    return attn_merge_row_hd(a, S, row, d4, HD);
}

// ---------------------------------------------------------------- GEMM

template <int WT> struct WTr;
template <> struct WTr<ET_F32> { static constexpr int E = 4, EB = 4; using acc_t = f32x4; };
template <> struct WTr<ET_BF16> { static constexpr int E = 8, EB = 2; using acc_t = f32x4; };
template <> struct WTr<ET_I8> { static constexpr int E = 16, EB = 1; using acc_t = i32x4; };
// int4 weights run on the int8 MFMA: same steps (16 k per lane), half the bytes
template <> struct WTr<ET_I4> { static constexpr int E = 16, EB = 1; using acc_t = i32x4; };
template <int WT> constexpr bool is_int() { return WT == ET_I8 || WT == ET_I4; }
// 1 KB weight blocks per 16-row tile and chunk (int4: two steps per block)
template <int WT> constexpr int wblocks() { return WT == ET_I4 ? FRAG_U / 2 : FRAG_U; }
// steps per stage: int4 stages hold whole blocks
template <int WT, int UC> constexpr int stage_uc() { return WT == ET_I4 && UC < 2 ? 2 : UC; }

// Four packed nibbles-with-offset (q + 8, one per byte) -> four int8 codes q:
// ((u | 0x80) - 8) ^ 0x80 per byte, no borrow crosses a byte.
__device__ __forceinline__ uint32_t sext_nib4(uint32_t x) { return ((x | 0x80808080u) - 0x08080808u) ^ 0x80808080u; }
// The int8 A-fragment of step h (0, 1) of a packed int4 block (wt4_byte layout).
__device__ __forceinline__ i32x4 i4_step(const i32x4 blk, int h) {
    const uint32_t w0 = (uint32_t)(h ? blk[2] : blk[0]), w1 = (uint32_t)(h ? blk[3] : blk[1]);
    return i32x4{(int)sext_nib4(w0 & 0x0f0f0f0fu), (int)sext_nib4(w1 & 0x0f0f0f0fu),
                 (int)sext_nib4((w0 >> 4) & 0x0f0f0f0fu), (int)sext_nib4((w1 >> 4) & 0x0f0f0f0fu)};
}

// GEMV-style step of one activation row: the lane's 16 weight bytes (8 bf16
// or 16 int8 k of one weight row) times the same k of the row, accumulated in
// the lane (fp32 fma, or exact int32 dot4).  The four lanes of a weight row
// (one per k-group) are summed once, at the end of the stream.
__device__ __forceinline__ float gv_dot(const i32x4 w, const i32x4 x, float acc) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t a = (uint32_t)w[i], b = (uint32_t)x[i];
        acc = fmaf(__uint_as_float(a << 16), __uint_as_float(b << 16), acc);
        acc = fmaf(__uint_as_float(a & 0xffff0000u), __uint_as_float(b & 0xffff0000u), acc);
    }
    return acc;
}
__device__ __forceinline__ int gv_dot(const i32x4 w, const i32x4 x, int acc) {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_sdot4(w[i], x[i], acc, false);
    return acc;
}

// A VALU read of an MFMA result needs a number of wait states after the MFMA
// (8 for the bf16 and int8 16x16 forms, 10 for the fp32 one).  The compiler
// pads straight-line code, but a drain that branches right after its MFMAs
// has been compiled with the accumulators read back at the join two
// instructions later (the last stage's contribution lost for part of a
// tile).  16 wait states after each conditional MFMA group close every such
// path; they cost a few cycles per drain stage.
__device__ __forceinline__ void mfma_result_pad() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7\n\ts_nop 7");
    __builtin_amdgcn_sched_barrier(0);
}

template <int WT>
__device__ __forceinline__ typename WTr<WT>::acc_t mfma_step(i32x4 a, i32x4 b, typename WTr<WT>::acc_t c) {
    if constexpr (WT == ET_BF16) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                        __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    } else if constexpr (is_int<WT>()) {
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
    } else {
        const f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[0], fb[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[1], fb[1], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[2], fb[2], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[3], fb[3], c, 0, 0, 0);
        return c;
    }
}

// Per-lane operands of the QKV epilogue of one weight tile, loaded at kernel
// start so that they sit in registers when the weight stream ends: each
// row's KV slot and, for q and k rows, the RoPE cos/sin of the lane's two
// rotation pairs at the row's position.  Loads are unconditional (indices
// clamped into their arrays).
template <int NT>
struct QkvPre {
    int slot[NT];
    float cs[NT][2], sn[NT][2];
    __device__ __forceinline__ void load(const GemmArgs& a, int tile, int lane, int row0 = 0) {
        const int r = lane & 15, g = lane >> 4, nb = tile * 16 + 4 * g;
        const int hd = a.hd, qrows = a.H * hd, krows = a.Hkv * hd, half = hd / 2;
        const bool rot = nb < qrows + krows;
        const int p0 = ((nb - (nb < qrows ? 0 : qrows)) % hd) / 2;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int t = min(row0 + 16 * j + r, a.T - 1);
            slot[j] = a.row_slot[t];
            int pos = a.row_pos[t];
            if (!dcheck(a.chk, pos >= 0 && pos < a.ctx_cap, CHK_POSITION)) pos = 0;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const size_t idx = rot ? (size_t)pos * half + p0 + p : 0;
                cs[j][p] = a.rope_cos[idx];
                sn[j][p] = a.rope_sin[idx];
            }
        }
    }
};

// The rotation of a pair, with its fused step spelled out: left to the
// compiler, each instantiation fuses one product of the sum or the other, and
// one bf16 key or query element in some 100 000 rounds differently.  The forms
// are those that the kernels have had from the start, so logits and KV keep
// their bits: fma(x1, cos, x0 sin) for fp32 accumulators (every tree size and
// the prefill alike) and for integer ones of two tiles per wave; the integer
// kernels of one tile per wave (X0) fuse the other product.
__device__ __forceinline__ float rope_lo(float x0, float x1, float cs, float sn) { return fmaf(x0, cs, -(x1 * sn)); }
template <bool X0 = false> __device__ __forceinline__ float rope_hi(float x0, float x1, float cs, float sn) {
    return X0 ? fmaf(x0, sn, x1 * cs) : fmaf(x1, cs, x0 * sn);
}

// Two consecutive activation values (4-byte aligned for bf16, 8 for fp32).
__device__ __forceinline__ void st2(uint16_t* p, size_t o, float x, float y) {
    *(uint32_t*)(p + o) = (uint32_t)f2bf(x) | ((uint32_t)f2bf(y) << 16);
}
__device__ __forceinline__ void st2(float* p, size_t o, float x, float y) { *(float2*)(p + o) = make_float2(x, y); }

// Epilogue of one 16-row weight tile: lane holds y[n = 16*tile + 4g + i][t = row0 + 16j + r].
// qp: the tile's preloaded QKV operands (EPI_QKV only).  TPW: tiles per wave.
// ROWS: a prefill's rows (row_tiles).
template <int WT, int NT, int EPI, typename AT, int TPW = 1, bool ROWS = false>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, const typename WTr<WT>::acc_t (&acc)[NT], int tile,
                                              int last_tile, int lane, const QkvPre<NT>& qp, int row0 = 0) {
    const int r = lane & 15, g = lane >> 4, T = a.T;
    const int nb = tile * 16 + 4 * g;
    // column tiles of a tiled output (NT, or 1 held for a wider layout)
    const int nto = ROWS ? row_tiles(T) : col_tiles(T);
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int t = row0 + 16 * j + r;
        if (t >= T) continue;
        float v[4];
        if constexpr (is_int<WT>()) {
            if constexpr (EPI == EPI_RAW) {
                int* o = (int*)a.out + (size_t)t * a.ldo + nb;
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = acc[j][i];
                continue;
            } else {
                const float xs = a.xs[t];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float y = (float)acc[j][i] * xs;
                    v[i] = y * a.ws[nb + i];
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = acc[j][i];
        }
        if constexpr (EPI == EPI_STORE) {
            float* o = (float*)a.out + (size_t)t * a.ldo + nb;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = v[i];
        } else if constexpr (EPI == EPI_RESID) {
            float* o = (float*)a.out + (size_t)t * a.ldo + nb;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] += v[i];
        } else if constexpr (EPI == EPI_SWIGLU) {
            constexpr int EO = 16 / sizeof(AT);
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const float gt = v[2 * p], up = v[2 * p + 1];
                Act<AT>::st((AT*)a.out, xt_off(t, nb / 2 + p, nto, EO), gt / (1.0f + expf(-gt)) * up);
            }
        } else if constexpr (EPI == EPI_QKV) {
            const int hd = a.hd, qrows = a.H * hd, krows = a.Hkv * hd;
            const int slot = qp.slot[j];
            if (nb < qrows + krows) {
                const bool isq = nb < qrows;
                const int rel = nb - (isq ? 0 : qrows);
                const int head = rel / hd, p0 = (rel % hd) / 2, half = hd / 2;
                float lo[2], hi[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const float cs = qp.cs[j][p], sn = qp.sn[j][p];
                    const float x0 = v[2 * p], x1 = v[2 * p + 1];
                    lo[p] = rope_lo(x0, x1, cs, sn);
                    hi[p] = rope_hi<is_int<WT>() && TPW == 1>(x0, x1, cs, sn);
                }
                // the pairs p0, p0 + 1 (p0 even) are adjacent in q and in both K layouts
                if (isq) {
                    AT* o = (AT*)a.out + ((size_t)t * a.H + head) * hd;
                    st2(o, p0, lo[0], lo[1]);
                    st2(o, p0 + half, hi[0], hi[1]);
                } else if (dcheck(a.chk, slot >= 0 && slot < a.ctx_cap, CHK_KV_WRITE)) {
                    constexpr int ET = sizeof(AT) == 2 ? ET_BF16 : ET_F32;
                    AT* o = (AT*)a.kc + (size_t)head * a.ctx_cap * hd;
                    st2(o, kv_k_off(ET, slot, p0, hd, a.ctx_cap), lo[0], lo[1]);
                    st2(o, kv_k_off(ET, slot, p0 + half, hd, a.ctx_cap), hi[0], hi[1]);
                }
            } else if (dcheck(a.chk, slot >= 0 && slot < a.ctx_cap, CHK_KV_WRITE)) {
                constexpr int ET = sizeof(AT) == 2 ? ET_BF16 : ET_F32;
                const int rel = nb - qrows - krows;
                const int head = rel / hd, dd = rel % hd;
                AT* o = (AT*)a.vt + (size_t)head * a.ctx_cap * hd;
#pragma unroll
                for (int i = 0; i < 4; ++i) Act<AT>::st(o, kv_v_off(ET, slot, dd + i, hd, a.ctx_cap), v[i]);
            }
        }
    }
    if constexpr (EPI == EPI_SWIGLU) {
        // the last tile also zeroes the pad columns of the output rows
        constexpr int EO = 16 / sizeof(AT);
        if (tile == last_tile) {
            const int kp = (a.out_k + 16 * EO - 1) / (16 * EO) * (16 * EO);
            const int w = kp - a.out_k;
            const int rows = ROWS ? min(T - row0, 16 * NT) : T;
            for (int idx = lane; idx < rows * w; idx += 64)
                Act<AT>::st((AT*)a.out, xt_off(row0 + idx / w, a.out_k + idx % w, nto, EO), 0.f);
        }
    }
}

// ---------------------------------------------------------------- activations

// Element e of a 16-byte piece of activations (bf16 bits or fp32), as fp32.
template <typename AT> __device__ __forceinline__ float piece_val(const i32x4 v, int e);
template <> __device__ __forceinline__ float piece_val<uint16_t>(const i32x4 v, int e) {
    const uint32_t w = (uint32_t)v[e >> 1];
    return __uint_as_float((e & 1) ? (w & 0xffff0000u) : (w << 16));
}
template <> __device__ __forceinline__ float piece_val<float>(const i32x4 v, int e) { return __int_as_float(v[e]); }

// Store 4 consecutive k (k4 a multiple of 4) of one row into tiled
// activations: they are contiguous inside one fragment.
__device__ __forceinline__ void st4(float* out, size_t o, float a, float b, float c, float d) {
    *(float4*)(out + o) = make_float4(a, b, c, d);
}
__device__ __forceinline__ void st4(uint16_t* out, size_t o, float a, float b, float c, float d) {
    const uint32_t lo = (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16);
    const uint32_t hi = (uint32_t)f2bf(c) | ((uint32_t)f2bf(d) << 16);
    *(uint2*)(out + o) = make_uint2(lo, hi);
}

__device__ __forceinline__ void st4q(int8_t* q, size_t o, float a, float b, float c, float d) {
    const uint32_t v = (uint32_t)(uint8_t)(int8_t)a | ((uint32_t)(uint8_t)(int8_t)b << 8) |
                       ((uint32_t)(uint8_t)(int8_t)c << 16) | ((uint32_t)(uint8_t)(int8_t)d << 24);
    *(uint32_t*)(q + o) = v;
}

// ---------------------------------------------------------------- attention

// A workgroup covers 4 waves x ATT_TPW key tiles of 32 slots.
static constexpr int ATT_WAVES = 4;
static constexpr int ATT_TPW = 2;
static constexpr int ATT_SPLIT = ATT_WAVES * ATT_TPW * 32;
static constexpr int ATT_MAX_SPLITS = 64;  // contexts up to 16384 slots

// Key tiles of a windowed forward: the tiles holding the sink slots, then the
// tiles from the window's first slot to the last tree slot.  Logical tile lt
// is physical tile lt (lt < st) or lt - st + pt0.  Without a window every
// committed slot is visible (csink = wstart = Lc) and the map is the identity.
struct AttnWindow {
    int csink, wstart, st, pt0, n_log;
    __host__ __device__ AttnWindow(int Lc, int n_tree, int win_sink, int win_len) {
        const int n_tiles = (Lc + n_tree + 31) >> 5;
        if (win_len > 0) {
            csink = win_sink < Lc ? win_sink : Lc;
            wstart = Lc - win_len > csink ? Lc - win_len : csink;
            st = (csink + 31) >> 5;
            pt0 = (wstart >> 5) > st ? (wstart >> 5) : st;
            n_log = st + (n_tiles - pt0);
        } else {
            csink = wstart = Lc;
            st = n_tiles;
            pt0 = 0;
            n_log = n_tiles;
        }
    }
    __host__ __device__ int phys(int lt) const { return lt < st ? lt : lt - st + pt0; }
};

// Butterfly max / sum with the lane 16 and lane 32 apart, through the
// cross-lane swap instructions (no LDS round trip).  Both lanes of a pair get
// the same operands in the same order, so their results are bit-identical.
__device__ __forceinline__ float pair_max16(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_max32(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum16(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float pair_sum32(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ bool anc_bit(uint64_t a0, uint64_t a1, int node) {
    return node < 64 ? ((a0 >> node) & 1ull) : ((a1 >> (node - 64)) & 1ull);
}

// Softmax state of one part (NTL key tiles) for the rows of a 16-row query
// tile, in two steps: attn_part_max gives the scores of visible slots
// scaled to log2 units and their maximum m (at least -1e30, so an empty part
// gives exp2 weights of 0); attn_part_probs gives the probabilities as bf16
// hi + lo pairs in the P-operand order and their sum l.  Both attention
// kernels use these and the merge helpers below with FP contraction off, so
// they round every row the same way.
// Bits e in [lo, hi) of an 8-bit mask.
__device__ __forceinline__ uint32_t bits8(int lo, int hi) {
    lo = max(lo, 0);
    hi = min(hi, 8);
    return lo < hi ? (0xffu >> (8 - (hi - lo))) << lo : 0u;
}
// Visibility of the 8 slots base .. base + 7 for one query row: committed
// slots in [0, csink) or [wstart, Lc), tree slots whose node is an
// ancestor-or-self (bit of the row's 128-bit mask), nothing at or past
// n_slots.  Shifts and range masks instead of a test per slot.
__device__ __forceinline__ uint32_t attn_vis8(int base, int Lc, int n_slots, const AttnWindow& win, uint64_t an0,
                                              uint64_t an1) {
    const uint32_t c = bits8(-base, win.csink - base) | bits8(win.wstart - base, Lc - base);
    const int n0 = base - Lc;  // tree node of bit 0 (negative: bit -n0 holds node 0)
    uint32_t t = 0;
    if (n0 >= 64 && n0 < 128) t = (uint32_t)(an1 >> (n0 - 64));
    else if (n0 > 0 && n0 < 64) t = (uint32_t)((an0 >> n0) | (an1 << (64 - n0)));
    else if (n0 == 0) t = (uint32_t)an0;
    else if (n0 > -8 && n0 < 0) t = (uint32_t)(an0 << (-n0));
    return c | (t & bits8(Lc - base, n_slots - base));
}
// Scaled scores of one key tile, -inf where the visibility bit is clear.
__device__ __forceinline__ void attn_tile_scores(const f32x4 (&S)[2], uint32_t vm, float scale_log2, float (&x)[8]) {
#pragma clang fp contract(off)
    if (__all(vm == 0xffu)) {  // a tile every lane sees whole (all committed tiles without a window)
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[4 * h2 + i] = S[h2][i] * scale_log2;
    } else {
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[4 * h2 + i] = (vm >> (4 * h2 + i)) & 1u ? S[h2][i] * scale_log2 : -INFINITY;
    }
}
template <int NTL>
__device__ __forceinline__ void attn_part_scores(const f32x4 (&S)[NTL][2], const int* ptile, const bool* live, int g,
                                                 int Lc, int n_slots, const AttnWindow& win, uint64_t an0,
                                                 uint64_t an1, float scale_log2, float (&x)[NTL][8]) {
#pragma unroll
    for (int tt = 0; tt < NTL; ++tt) {
        const uint32_t vm = live[tt] ? attn_vis8(ptile[tt] * 32 + 8 * g, Lc, n_slots, win, an0, an1) : 0u;
        attn_tile_scores(S[tt], vm, scale_log2, x[tt]);
    }
}
template <int NTL>
__device__ __forceinline__ float attn_part_max(const float (&x)[NTL][8]) {
    float mt = -INFINITY;
#pragma unroll
    for (int tt = 0; tt < NTL; ++tt)
#pragma unroll
        for (int e = 0; e < 8; ++e) mt = fmaxf(mt, x[tt][e]);
    return fmaxf(-1e30f, pair_max32(pair_max16(mt)));
}
template <int NTL>
__device__ __forceinline__ float attn_part_probs(const float (&x)[NTL][8], float mn, i32x4 (&Pf)[NTL],
                                                 i32x4 (&Pl)[NTL]) {
#pragma clang fp contract(off)
    float ps = 0.f;
#pragma unroll
    for (int tt = 0; tt < NTL; ++tt) {
        uint16_t pb[8], pl[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float p = __builtin_amdgcn_exp2f(x[tt][e] - mn);
            ps += p;
            pb[e] = f2bf(p);
            pl[e] = f2bf(p - bf2f(pb[e]));  // exact difference, rounded: p = hi + lo to ~2^-17
        }
        Pf[tt] = i32x4{(int)(pb[0] | ((uint32_t)pb[1] << 16)), (int)(pb[2] | ((uint32_t)pb[3] << 16)),
                       (int)(pb[4] | ((uint32_t)pb[5] << 16)), (int)(pb[6] | ((uint32_t)pb[7] << 16))};
        Pl[tt] = i32x4{(int)(pl[0] | ((uint32_t)pl[1] << 16)), (int)(pl[2] | ((uint32_t)pl[3] << 16)),
                       (int)(pl[4] | ((uint32_t)pl[5] << 16)), (int)(pl[6] | ((uint32_t)pl[7] << 16))};
    }
    return pair_sum32(pair_sum16(ps));
}

// The in-order merge of part states under the common maximum M: weight
// exp2(m - M) of a part, then acc = fma(weight, o, acc), L = fma(weight, l, L).
__device__ __forceinline__ float attn_merge_weight(float m, float M) { return exp2f(m - M); }
__device__ __forceinline__ void attn_merge_o(f32x4& acc, const f32x4 o, float f) {
    acc = f32x4{fmaf(o[0], f, acc[0]), fmaf(o[1], f, acc[1]), fmaf(o[2], f, acc[2]), fmaf(o[3], f, acc[3])};
}
__device__ __forceinline__ void attn_merge_l(float& L, float l, float f) { L = fmaf(l, f, L); }

// Query rows of a kv head: its G query heads x T tokens, each head's rows
// padded to Rp and packed into 16-row tiles, row p = 16 tile + r holding
// token p % Rp of head p / Rp of the group.  Up to 16 tokens Rp = T, so the
// heads' rows follow each other (a one-node call of a 4-head group fills one
// tile instead of four, and the group's K/V pass serves every head; a head's
// rows may straddle two tiles); above, Rp rounds T up to 16.  A row's
// arithmetic does not depend on where it sits in its tile.
__host__ __device__ inline int attn_head_rows(int T) { return T <= 16 ? T : (T + 15) & ~15; }
__host__ __device__ inline int attn_query_tiles(int T, int G) { return (G * attn_head_rows(T) + 15) / 16; }

// One step of the in-order merge of split partials (attn_merge_row_hd's), the
// running state in registers.
template <int NDT>
__device__ __forceinline__ void attn_merge_split(f32x4 (&acc)[NDT], float& L, float& M, const f32x4 (&o)[NDT], float l,
                                                 float m) {
#pragma clang fp contract(off)
    const float mn = fmaxf(M, m);
    const float fo = exp2f(M - mn), fn = exp2f(m - mn);
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) acc[dt] = acc[dt] * fo + o[dt] * fn;
    L = L * fo + l * fn;
    M = mn;
}

}  // namespace cas
