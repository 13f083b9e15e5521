// gfx950 kernels of a prefill: the layers over hundreds to thousands of
// consecutive tokens, with the values of the tree kernels (kernels.hip).
#include "kernel_common.h"
#include <algorithm>

namespace cas {

// ---------------------------------------------------------------- GEMM of many rows

// Prefill: the same linear layers over hundreds to thousands of rows, where
// the weights are reused and the matrix cores are what counts.  A workgroup
// computes (16 NW WN) weight rows x (16 TW WT_) activation rows; its WN x WT_
// waves own NW x TW MFMA tiles each.  Both operands lie in memory as 1 KB
// fragments, so a stage (two k-steps of every tile) goes to LDS with
// direct-to-LDS loads, 1 KB per wave instruction, and every MFMA operand is
// one conflict-free 16-byte LDS read; no register passes through, no swizzle.
// Two stages alternate: the next one's loads are in flight while the current
// one is multiplied, and __syncthreads() both waits for them and frees the
// buffer (four separate arrays, so that the reads of one stage do not wait
// for the loads of the other).
//
// The k order of a sum is that of k_gemm / k_gemm_wide: the same MFMA, steps
// in order; where those split K over waves or workgroups (RNG: a.ksplit
// ranges) each range is summed from zero and added to the total in order.  A
// row's result therefore has the same bits in a prefill, a verify and a
// one-row call.
//
// Measured, prefill of 1024 tokens on the 7B shapes (blocks of 256 x 256,
// or 128 x 128 with ranges): QKV 139 us, gate/up 229 us (805 TFLOP/s), O 64,
// down 157; before, eight passes of the weight-streaming kernels at 128 rows
// took 8 x (43, 45, 15, 30) us, and each pass its own LM head.
template <int WT, int NW, int TW, int WN, int WT_, int EPI, typename AT, bool KM, bool RNG>
__global__ void __launch_bounds__(64 * WN * WT_, 2) k_gemm_rows(const GemmArgs a) {
    using ACC = typename WTr<WT>::acc_t;
    constexpr int E = WTr<WT>::E, W = WN * WT_, BN = NW * WN, BT = TW * WT_, US = 2;
    constexpr int LA = BN * US / W, LB = BT * US / W;  // 1 KB loads per wave and stage
    static_assert(!is_int<WT>(), "fp32 and bf16 weights");
    static_assert(LA * W == BN * US && LB * W == BT * US && FRAG_U == 2 * US, "stage shape");
    __shared__ __attribute__((aligned(16))) char sa0[BN * US * 1024], sb0[BT * US * 1024];
    __shared__ __attribute__((aligned(16))) char sa1[BN * US * 1024], sb1[BT * US * 1024];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave / WT_, wt = wave % WT_;
    const int ntiles = a.N >> 4, nto = col_tiles(a.T);
    // Workgroups go to the XCDs round robin; each XCD takes a run of
    // consecutive (weight block, row block) pairs, rows fastest, so that the
    // workgroups sharing a weight block share an L2.
    const int nT = ((a.T + 15) / 16 + BT - 1) / BT, nb = gridDim.x;
    const int xcd = blockIdx.x % 8, per = nb / 8, rem = nb % 8;
    const int lin = xcd * per + min(xcd, rem) + blockIdx.x / 8;
    const int tn0 = (lin / nT) * BN, tt0 = (lin % nT) * BT;  // first weight / row tile
    const int C = a.Kp / (16 * E), NS = 2 * C;               // chunks, stages

    // 1 KB blocks of this wave: block i of a stage is step i / BN of tile i % BN
    const size_t ast = (KM ? (size_t)ntiles : 1) * 1024, bst = (size_t)nto * 1024;  // bytes per step
    const char* pa[LA];
    const char* pb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int b = wave * LA + i, tile = min(tn0 + b % BN, ntiles - 1);
        pa[i] = (const char*)a.W + (KM ? (size_t)tile : (size_t)tile * C * FRAG_U) * 1024 + (b / BN) * ast + lane * 16;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int b = wave * LB + i, tile = min(tt0 + b % BT, nto - 1);
        pb[i] = (const char*)a.X + (size_t)tile * 1024 + (b / BT) * bst + lane * 16;
    }
    ACC acc[NW][TW], tot[RNG ? NW : 1][RNG ? TW : 1];
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j) {
            acc[i][j] = ACC{0, 0, 0, 0};
            if constexpr (RNG) tot[i][j] = ACC{0, 0, 0, 0};
        }
    auto stage = [&](char* sa, char* sb, int s) {
#pragma unroll
        for (int i = 0; i < LA; ++i) lds_load16(pa[i] + (size_t)s * US * ast, sa + (wave * LA + i) * 1024);
#pragma unroll
        for (int i = 0; i < LB; ++i) lds_load16(pb[i] + (size_t)s * US * bst, sb + (wave * LB + i) * 1024);
        __builtin_amdgcn_sched_barrier(0);  // the loads go first, not behind the LDS reads
    };
    auto mma = [&](const char* sa, const char* sb) {
#pragma unroll
        for (int u = 0; u < US; ++u) {
            i32x4 A[NW], B[TW];
#pragma unroll
            for (int i = 0; i < NW; ++i) A[i] = *(const i32x4*)(sa + (u * BN + wn * NW + i) * 1024 + lane * 16);
#pragma unroll
            for (int j = 0; j < TW; ++j) B[j] = *(const i32x4*)(sb + (u * BT + wt * TW + j) * 1024 + lane * 16);
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int j = 0; j < TW; ++j) acc[i][j] = mfma_step<WT>(A[i], B[j], acc[i][j]);
        }
    };
    // first chunk of the next range with any (K shorter than ksplit chunks leaves some empty)
    int range = 0, bound = 0;
    auto next_bound = [&](int c) {
        while (bound <= c && range < a.ksplit) bound = (int)(((long)++range * C) / a.ksplit);
    };
    if constexpr (RNG) next_bound(0);
    stage(sa0, sb0, 0);
    __syncthreads();
    for (int c = 0; c < C; ++c) {
        stage(sa1, sb1, 2 * c + 1);
        mma(sa0, sb0);
        __syncthreads();
        if (c + 1 < C) stage(sa0, sb0, 2 * c + 2);
        mma(sa1, sb1);
        if constexpr (RNG) {
            if (c + 1 == bound) {
                mfma_result_pad();
#pragma unroll
                for (int i = 0; i < NW; ++i)
#pragma unroll
                    for (int j = 0; j < TW; ++j) {
                        tot[i][j] += acc[i][j];
                        acc[i][j] = ACC{0, 0, 0, 0};
                    }
                next_bound(c + 1);
            }
        }
        __syncthreads();
    }
    mfma_result_pad();
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const int tile = tn0 + wn * NW + i, row0 = (tt0 + wt * TW) * 16;
        if (tile >= ntiles || row0 >= a.T) continue;
        QkvPre<TW> qp;
        if constexpr (EPI == EPI_QKV) qp.load(a, tile, lane, row0);
        if constexpr (RNG) gemm_epilogue<WT, TW, EPI, AT>(a, tot[i], tile, ntiles - 1, lane, qp, row0);
        else gemm_epilogue<WT, TW, EPI, AT>(a, acc[i], tile, ntiles - 1, lane, qp, row0);
    }
}

int gemm_sum_ranges(int wtype, int N, int Kp, int resid) {
    if (resid) {
        const int ks = gemm_parts_count(wtype, N, Kp, 1);
        if (ks > 1) return ks;
    }
    // the wide kernel streams the whole range in each wave; k_gemm splits it four ways
    return N >= 8192 && ((N / 16) % 4 == 0 || (N / 16) % 3 == 0) ? 1 : 4;
}

template <int WT, int NW, int TW, int WN, int WT_, int EPI, typename AT, bool KM, bool RNG>
static hipError_t gemm_rows_launch(const GemmArgs& a, hipStream_t s) {
    const int nT = ((a.T + 15) / 16 + TW * WT_ - 1) / (TW * WT_), nN = (a.N / 16 + NW * WN - 1) / (NW * WN);
    hipLaunchKernelGGL((k_gemm_rows<WT, NW, TW, WN, WT_, EPI, AT, KM, RNG>), dim3(nT * nN), dim3(64 * WN * WT_), 0, s, a);
    return hipGetLastError();
}

template <int WT, int EPI, typename AT, bool KM>
static hipError_t gemm_rows_go(const GemmArgs& a, hipStream_t s) {
    if (a.kmaj != (int)KM) return hipErrorInvalidValue;
    if (a.ksplit > 1) return gemm_rows_launch<WT, 4, 4, 2, 2, EPI, AT, KM, true>(a, s);
    return gemm_rows_launch<WT, 8, 4, 2, 4, EPI, AT, KM, false>(a, s);
}

template <int WT, typename AT>
static hipError_t gemm_rows_epi(int epi, const GemmArgs& a, hipStream_t s) {
    switch (epi) {
    case EPI_RESID: return gemm_rows_go<WT, EPI_RESID, AT, false>(a, s);
    case EPI_SWIGLU: return gemm_rows_go<WT, EPI_SWIGLU, AT, true>(a, s);
    case EPI_QKV: return gemm_rows_go<WT, EPI_QKV, AT, false>(a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_rows(int wtype, int epi, const GemmArgs& a, hipStream_t s) {
    if (a.N < 16 || a.N % 16 || a.Kp % chunk_k(wtype) || a.Kp < chunk_k(wtype) || a.T <= 128 || a.ksplit < 1 ||
        a.ksplit > 8 || a.qx || a.mx_o)
        return hipErrorInvalidValue;
    if (wtype == ET_BF16) return gemm_rows_epi<ET_BF16, uint16_t>(epi, a, s);
    if (wtype == ET_F32) return gemm_rows_epi<ET_F32, float>(epi, a, s);
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- attention

// Causal attention of a prefill.  Workgroup = (kv head, QW query tiles of 16
// rows; the G heads of a group at the same rows follow each other, so its
// waves need about the same slots).  It walks the splits of 256 slots that
// its rows see; a split's K and then its V pass once through LDS (64 KB each
// at head_dim 128, direct-to-LDS loads: V arrives under the scores, the next
// K under the softmax and P V), and each wave computes the split's partial of
// its rows exactly as k_attn_rows does and merges it into its running state
// exactly as k_attn_merge does, in split order: the same bits as a forward of
// up to 128 rows, without the partials' trip through memory.  Parts wholly
// past a tile's last row would add zero and are left out.
template <int HD, int QW>
__global__ void __launch_bounds__(64 * QW, 2) k_attn_causal(const AttnArgs a, float scale_log2) {
    constexpr int UD = HD / 32, DG = HD / 4, NDT = HD / 16, TE = 32 * HD;
    constexpr int NP = ATT_WAVES, NTS = NP * ATT_TPW, KF = 2 * UD, LP = NTS * KF / QW;
    static_assert(KF == NDT && LP * QW == NTS * KF, "K and V stages must match");
    __shared__ i32x4 ks[NTS * KF * 64], vs[NTS * NDT * 64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int Lc = a.sp->Lc, T = a.T, G = a.H / a.Hkv;
    if (!dcheck(a.chk, Lc >= 0 && Lc + T <= a.sp->cap && a.sp->cap <= a.ctx_cap, CHK_ATTN_SLOTS)) return;
    const int n_tiles = (Lc + T + 31) >> 5;
    // the last rows see the most slots: their workgroups start first
    const int kvh = blockIdx.x % a.Hkv, blk = (int)(gridDim.x / a.Hkv) - 1 - (int)(blockIdx.x / a.Hkv);
    const int ct = blk * QW + wave, hg = ct % G, t0 = ct / G * 16, head = kvh * G + hg;
    const int blast = min(T, ((blk * QW + QW - 1) / G + 1) * 16);     // rows below it need the workgroup's walk
    const int nsplit = (Lc + blast + ATT_SPLIT - 1) / ATT_SPLIT;
    const int wslots = t0 < T ? Lc + min(t0 + 16, T) : 0;             // slots the wave's rows see
    const int vl = t0 + r < T ? Lc + t0 + r + 1 : 0;                  // slots the lane's row sees
    const uint16_t* q = (const uint16_t*)a.q;
    i32x4 Qf[UD];
    {
        const int t = min(t0 + r, T - 1);
#pragma unroll
        for (int u = 0; u < UD; ++u) Qf[u] = *(const i32x4*)(q + ((size_t)t * a.H + head) * HD + g * DG + u * 8);
    }
    const uint16_t* kbase = (const uint16_t*)a.kc + (size_t)kvh * a.ctx_cap * HD + lane * 8;
    const uint16_t* vbase = (const uint16_t*)a.vt + (size_t)kvh * a.ctx_cap * HD + lane * 8;
    auto load = [&](const uint16_t* base, i32x4* dst, int split) {
#pragma unroll
        for (int i = 0; i < LP; ++i) {
            const int f = wave * LP + i, tile = min(split * NTS + f / KF, n_tiles - 1);
            lds_load16(base + (size_t)tile * TE + (f % KF) * 512, dst + f * 64);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x4 acc[NDT];
    float L = 0.f, M = -1e30f;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    load(kbase, ks, 0);
    __syncthreads();
    for (int split = 0; split < nsplit; ++split) {
        const int base = split * ATT_SPLIT;
        load(vbase, vs, split);
        float x[NP][ATT_TPW][8], m[NP], Ms = -1e30f;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            m[p] = -1e30f;
            if (base + p * 32 * ATT_TPW < wslots) {
#pragma unroll
                for (int tt = 0; tt < ATT_TPW; ++tt) {
                    f32x4 S[2];
#pragma unroll
                    for (int h2 = 0; h2 < 2; ++h2) {
                        S[h2] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int u = 0; u < UD; ++u)
                            S[h2] = mfma_step<ET_BF16>(ks[((p * ATT_TPW + tt) * KF + h2 * UD + u) * 64 + lane], Qf[u], S[h2]);
                    }
                    attn_tile_scores(S, bits8(0, vl - (base + (p * ATT_TPW + tt) * 32 + 8 * g)), scale_log2, x[p][tt]);
                }
                m[p] = attn_part_max<ATT_TPW>(x[p]);
                Ms = fmaxf(Ms, m[p]);
            }
        }
        __syncthreads();  // V is there, K is read
        if (split + 1 < nsplit) load(kbase, ks, split + 1);
        if (base < wslots) {
            f32x4 o[NDT];
            float l = 0.f;
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                if (base + p * 32 * ATT_TPW >= wslots) continue;
                i32x4 Pf[ATT_TPW], Pl[ATT_TPW];
                const float lp = attn_part_probs<ATT_TPW>(x[p], m[p], Pf, Pl);
                const float f = attn_merge_weight(m[p], Ms);
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    f32x4 po = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int tt = 0; tt < ATT_TPW; ++tt) {
                        const i32x4 v = vs[((p * ATT_TPW + tt) * NDT + dt) * 64 + lane];
                        po = mfma_step<ET_BF16>(v, Pf[tt], po);
                        po = mfma_step<ET_BF16>(v, Pl[tt], po);
                    }
                    attn_merge_o(o[dt], po, f);
                }
                attn_merge_l(l, lp, f);
            }
            attn_merge_split<NDT>(acc, L, M, o, l, Ms);
        }
        __syncthreads();  // the next K is there, V is read
    }
    const int t = t0 + r;
    if (t < T) {
        const float inv = L > 0.f ? 1.f / L : 0.f;
        const int nto = col_tiles(T);
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
            st4((uint16_t*)a.out, xt_off(t, head * HD + 16 * dt + 4 * g, nto, 8), acc[dt][0] * inv, acc[dt][1] * inv,
                acc[dt][2] * inv, acc[dt][3] * inv);
    }
}

hipError_t launch_attention_causal(int atype, const AttnArgs& a, hipStream_t s) {
    if (a.T < 1 || a.Hkv < 1 || a.H % a.Hkv || (a.hd != 64 && a.hd != 128) || !a.out_tiled || a.win_len)
        return hipErrorInvalidValue;
    if (atype == ET_F32) return launch_attention_f32(a, 1, s);
    if (a.ctx_cap % 32) return hipErrorInvalidValue;
    constexpr int QW = 8;
    const int nct = (a.T + 15) / 16 * (a.H / a.Hkv), nblk = (nct + QW - 1) / QW;
    const float scale_log2 = (1.0f / sqrtf((float)a.hd)) * 1.4426950408889634f;
    if (a.hd == 128) hipLaunchKernelGGL((k_attn_causal<128, QW>), dim3(nblk * a.Hkv), dim3(64 * QW), 0, s, a, scale_log2);
    else hipLaunchKernelGGL((k_attn_causal<64, QW>), dim3(nblk * a.Hkv), dim3(64 * QW), 0, s, a, scale_log2);
    return hipGetLastError();
}

// ---------------------------------------------------------------- embedding

// Rows of a prefill: row t is token tok[t] at slot and position Lc + t.
template <typename AT>
__global__ void __launch_bounds__(256) k_embed_chain(const AT* E, int d, int vocab, const int* toks,
                                                     const StepParams* sp, float* h, int* row_pos, int* row_slot,
                                                     int* chk) {
    const int t = blockIdx.x, Lc = sp->Lc;
    int tok = toks[t];
    if (!dcheck(chk, tok >= 0 && tok < vocab, CHK_TOKEN)) tok = 0;
    constexpr int EV = 16 / sizeof(AT);
    const AT* er = E + (size_t)tok * d;
    float* hr = h + (size_t)t * d;
    for (int k = threadIdx.x * EV; k < d; k += 256 * EV) {
        const i32x4 pc = *(const i32x4*)(er + k);
#pragma unroll
        for (int e = 0; e < EV; e += 4)
            *(float4*)(hr + k + e) = make_float4(piece_val<AT>(pc, e), piece_val<AT>(pc, e + 1),
                                                 piece_val<AT>(pc, e + 2), piece_val<AT>(pc, e + 3));
    }
    if (threadIdx.x == 0) {
        row_pos[t] = Lc + t;
        row_slot[t] = dcheck(chk, Lc >= 0 && Lc + (int)gridDim.x <= sp->cap, CHK_SLOTS) ? Lc + t : -1;
    }
}

hipError_t launch_embed_chain(int atype, const void* embed, int d, int vocab, const int* tok, const StepParams* sp,
                              int T, float* h, int* row_pos, int* row_slot, int* chk, hipStream_t s) {
    if (T < 1 || d % 16) return hipErrorInvalidValue;
    if (atype == ET_BF16)
        hipLaunchKernelGGL(k_embed_chain<uint16_t>, dim3(T), dim3(256), 0, s, (const uint16_t*)embed, d, vocab, tok, sp,
                           h, row_pos, row_slot, chk);
    else
        hipLaunchKernelGGL(k_embed_chain<float>, dim3(T), dim3(256), 0, s, (const float*)embed, d, vocab, tok, sp, h,
                           row_pos, row_slot, chk);
    return hipGetLastError();
}

}  // namespace cas
