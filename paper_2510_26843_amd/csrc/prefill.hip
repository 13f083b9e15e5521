// gfx950 kernels of a prefill: the layers over hundreds to thousands of
// consecutive tokens, with the values of the tree kernels (kernels.hip).
#include "kernel_common.h"
#include <algorithm>

namespace cas {

// ---------------------------------------------------------------- GEMM of many rows

// Direct-to-LDS load of one wave: 16 bytes per lane from base + voff (base
// uniform, voff per lane) to LDS byte lds + 16 lane.  Written out because the
// compiler, which cannot tell the ring's stages apart, would wait for every
// load in flight before each LDS read; stage_wait() below is the wait.  (No
// register is written; s_nop: the wait state between m0 and its use.)
__device__ __forceinline__ void lds_load16(const char* base, uint32_t voff, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds)
                 : "memory");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}
// All but the last N of this wave's direct-to-LDS loads have landed and its
// LDS reads are done; then the same holds for every wave of the workgroup.
template <int N>
__device__ __forceinline__ void stage_wait() {
    static_assert(N >= 0 && N <= 63, "vmcnt");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// 4 x 4 transpose over the lane groups g = lane / 16: lane group g's v[j]
// becomes v[g] of lane group j.
__device__ __forceinline__ void lane_transpose4(uint32_t (&v)[4]) {
    const auto a = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
    const auto lo = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
    v[0] = lo[0];
    v[1] = lo[1];
    v[2] = hi[0];
    v[3] = hi[1];
}
__device__ __forceinline__ uint32_t pack_bf(float x, float y) { return (uint32_t)f2bf(x) | ((uint32_t)f2bf(y) << 16); }

// The bf16 SwiGLU and QKV epilogues of one weight tile over four row tiles
// (gemm_epilogue's arithmetic) with 16-byte stores: its lanes hold 2- and
// 4-byte pieces of a row that are 8 consecutive elements of the output, so
// the four lane groups exchange them, each ending with one row tile's 16
// bytes; V tiles, whose output runs along the slots, turn through LDS.  The
// piecewise stores cost the 7B QKV 131 us and gate/up 199 us at
// 1024 rows, these 115 and 189 (3001 tokens of the 8B shape: 115 -> 99, 317 -> 289).
constexpr int EP_LDS = 16 * 72;  // 2-byte elements of a wave's V tile: 16 d, 64 slots, padded
struct RowsPre {
    int pos[4], slot, vslot;  // RoPE positions of rows 16j + r; slot of row 16g + r, of row 8 (lane % 8)
    __device__ __forceinline__ void load(const GemmArgs& a, int row0, int lane) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            pos[j] = a.row_pos[min(row0 + 16 * j + (lane & 15), a.T - 1)];
            if (!dcheck(a.chk, pos[j] >= 0 && pos[j] < a.ctx_cap, CHK_POSITION)) pos[j] = 0;
        }
        slot = a.row_slot[min(row0 + lane, a.T - 1)];  // 16 g + r = lane
        vslot = a.row_slot[min(row0 + 8 * (lane & 7), a.T - 1)];
    }
};
struct RopePre {
    float2 cs[4], sn[4];  // the lane's two rotation pairs at rows 16j + r
    __device__ __forceinline__ void load(const GemmArgs& a, int tile, int lane, const RowsPre& rp) {
        const int hd = a.hd, nb = tile * 16 + 4 * (lane >> 4), p0 = nb % hd / 2, half = hd / 2;
        const bool rot = tile * 16 < (a.H + a.Hkv) * hd;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const size_t i = rot ? (size_t)rp.pos[j] * half + p0 : 0;
            cs[j] = *(const float2*)(a.rope_cos + i);
            sn[j] = *(const float2*)(a.rope_sin + i);
        }
    }
};
template <int EPI>
__device__ __forceinline__ void rows_epilogue(const GemmArgs& a, const f32x4 (&v)[4], int tile, int last_tile, int lane,
                                              int row0, const RowsPre& rp, const RopePre& ro, uint16_t* ep) {
    static_assert(EPI == EPI_SWIGLU || EPI == EPI_QKV, "bf16 outputs");
    const int T = a.T, t = row0 + lane;  // row of the lane's stores
    if constexpr (EPI == EPI_SWIGLU) {
        uint32_t w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            w[j] = pack_bf(v[j][0] / (1.0f + expf(-v[j][0])) * v[j][1], v[j][2] / (1.0f + expf(-v[j][2])) * v[j][3]);
        lane_transpose4(w);
        const int nto = row_tiles(T);
        if (t < T) *(uint4*)((uint16_t*)a.out + xt_off(t, tile * 8, nto, 8)) = make_uint4(w[0], w[1], w[2], w[3]);
        if (tile == last_tile) {  // and the pad columns
            const int pad = (a.out_k + 127) / 128 * 128 - a.out_k, rows = min(T - row0, 64);
            for (int i = lane; i < rows * pad; i += 64)
                ((uint16_t*)a.out)[xt_off(row0 + i / pad, a.out_k + i % pad, nto, 8)] = 0;
        }
    } else {
        const int hd = a.hd, half = hd / 2, qrows = a.H * hd, krows = a.Hkv * hd, n0 = tile * 16;
        if (n0 < qrows + krows) {
            uint32_t lo[4], hi[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float2 cs = ro.cs[j], sn = ro.sn[j];
                lo[j] = pack_bf(rope_lo(v[j][0], v[j][1], cs.x, sn.x), rope_lo(v[j][2], v[j][3], cs.y, sn.y));
                hi[j] = pack_bf(rope_hi(v[j][0], v[j][1], cs.x, sn.x), rope_hi(v[j][2], v[j][3], cs.y, sn.y));
            }
            lane_transpose4(lo);
            lane_transpose4(hi);
            const bool isq = n0 < qrows;
            const int rel = n0 - (isq ? 0 : qrows), head = rel / hd, d0 = rel % hd / 2;
            uint16_t *pl, *ph;
            bool ok = t < T;
            if (isq) {
                pl = (uint16_t*)a.out + ((size_t)t * a.H + head) * hd + d0;
                ph = pl + half;
            } else {
                ok = ok && dcheck(a.chk, rp.slot >= 0 && rp.slot < a.ctx_cap, CHK_KV_WRITE);
                uint16_t* o = (uint16_t*)a.kc + (size_t)head * a.ctx_cap * hd;
                pl = o + kv_k_tiled(rp.slot, d0, hd);
                ph = o + kv_k_tiled(rp.slot, d0 + half, hd);
            }
            if (ok) {
                *(uint4*)pl = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                *(uint4*)ph = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            }
        } else {
            const int rel = n0 - qrows - krows, head = rel / hd, d0 = rel % hd;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) ep[(4 * (lane >> 4) + i) * 72 + 16 * j + (lane & 15)] = f2bf(v[j][i]);
            asm volatile("" ::: "memory");  // (one wave's LDS operations stay in order)
            // eight rows of one d per lane: consecutive slots, one 16-byte
            // piece of the cache where the first is a multiple of 8
            const int tg = 8 * (lane & 7), n = min(8, T - row0 - tg);
            uint16_t* o = (uint16_t*)a.vt + (size_t)head * a.ctx_cap * hd;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int d = (lane >> 3) + 8 * h;
                const uint16_t* e = ep + d * 72 + tg;
                if (n < 1 || !dcheck(a.chk, rp.vslot >= 0 && rp.vslot + n <= a.ctx_cap, CHK_KV_WRITE)) continue;
                if (n == 8 && (rp.vslot & 7) == 0) *(i32x4*)(o + kv_v_tiled(rp.vslot, d0 + d, hd)) = *(const i32x4*)e;
                else
                    for (int k = 0; k < n; ++k) o[kv_v_tiled(rp.vslot + k, d0 + d, hd)] = e[k];
            }
            asm volatile("" ::: "memory");
        }
    }
}

// Prefill: the same linear layers over hundreds to thousands of rows, where
// the weights are reused and the matrix cores are what counts.  A workgroup
// computes (16 NW WN) weight rows x (16 TW WT_) activation rows; its WN x WT_
// waves own NW x TW MFMA tiles each.  Both operands lie in memory as 1 KB
// fragments, so a k-step of every tile goes to LDS with direct-to-LDS loads,
// 1 KB per wave instruction, and every MFMA operand is one conflict-free
// 16-byte LDS read; no register passes through, no swizzle.  D one-step
// stages form a ring: while step s is multiplied out of registers, the
// fragments of s + 1 are read into the other register set and the loads of
// s + 2 .. s + D are in flight; one barrier per step.
//
// The k order of a sum is that of k_gemm / k_gemm_wide: the same MFMA, steps
// in order; where those split K over waves or workgroups (RNG: a.ksplit
// ranges) each range is summed from zero and added to the total in order, or,
// with few workgroups, computed by a workgroup of its own (SPL: gridDim.y =
// a.ksplit, range k's sums stored at a.out + k * a.part_stride for the next
// norm to add).  A row's result therefore has the same bits in a prefill, a
// verify and a one-row call.
template <int WT, int NW, int TW, int WN, int WT_, int D, int EPI, typename AT, bool KM, bool RNG, bool SPL>
__global__ void __launch_bounds__(64 * WN * WT_, 2) k_gemm_rows(GemmArgs a) {
    using ACC = typename WTr<WT>::acc_t;
    constexpr int E = WTr<WT>::E, W = WN * WT_, BN = NW * WN, BT = TW * WT_;
    constexpr int LA = BN / W, LB = BT / W, LD = LA + LB;  // 1 KB loads per wave and step
    constexpr int SB = (BN + BT) * 1024;                   // bytes of a stage
    static_assert(!is_int<WT>() && !(RNG && SPL), "fp32 and bf16 weights; one way with the ranges");
    static_assert(LA * W == BN && LB * W == BT, "stage shape");
    static_assert(D == FRAG_U, "a round of the ring is a chunk, so that no step is past the last");
    constexpr bool BFX = sizeof(AT) == 2 && (EPI == EPI_SWIGLU || EPI == EPI_QKV);  // the 16-byte epilogues
    static_assert(!BFX || (TW == 4 && 2 * W * EP_LDS <= D * SB), "epilogue shape");
    __shared__ __attribute__((aligned(16))) char sm[D * SB];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave / WT_, wt = wave % WT_;
    const int ntiles = a.N >> 4, nto = row_tiles(a.T);
    // Workgroups go to the XCDs round robin; each XCD takes a run of
    // consecutive (weight block, row block) pairs, rows fastest, so that the
    // workgroups sharing a weight block share an L2.
    const int nT = ((a.T + 15) / 16 + BT - 1) / BT, nb = gridDim.x;
    const int xcd = blockIdx.x % 8, per = nb / 8, rem = nb % 8;
    const int lin = xcd * per + min(xcd, rem) + blockIdx.x / 8;
    const int tn0 = (lin / nT) * BN, tt0 = (lin % nT) * BT;  // first weight / row tile
    const int CW = a.Kp / (16 * E);                          // chunks of the matrix
    const int c0 = SPL ? (int)(((long)blockIdx.y * CW) / gridDim.y) : 0;
    const int C = SPL ? (int)(((long)(blockIdx.y + 1) * CW) / gridDim.y) - c0 : CW;  // chunks of this workgroup
    const int NS = C * FRAG_U;                                                       // steps
    if constexpr (SPL) a.out = (float*)a.out + blockIdx.y * a.part_stride;

    // 1 KB blocks of this wave: LA weight tiles, LB row tiles of each step
    const size_t ast = (KM ? (size_t)ntiles : 1) * 1024, bst = (size_t)nto * 1024;  // bytes per step
    const char* pa[LA];
    const char* pb[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) {
        const int tile = min(tn0 + wave * LA + i, ntiles - 1);
        pa[i] = (const char*)a.W + (KM ? (size_t)tile : (size_t)tile * CW * FRAG_U) * 1024 + c0 * FRAG_U * ast;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i)
        pb[i] = (const char*)a.X + (size_t)min(tt0 + wave * LB + i, nto - 1) * 1024 + c0 * FRAG_U * bst;
    const uint32_t vo = lane * 16;
    const uint32_t la = lds_addr(sm) + wave * LA * 1024, lb = lds_addr(sm) + (BN + wave * LB) * 1024;
    // the next step's loads; past the last step the pointers stay (a reload
    // into a stage that is not read again), so that the counts of loads in
    // flight hold to the end
    auto load = [&](int stg, bool more) {
#pragma unroll
        for (int i = 0; i < LA; ++i) {
            lds_load16(pa[i], vo, la + stg * SB + i * 1024);
            pa[i] += more ? ast : 0;
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            lds_load16(pb[i], vo, lb + stg * SB + i * 1024);
            pb[i] += more ? bst : 0;
        }
    };
    RowsPre rp;
    if constexpr (BFX && EPI == EPI_QKV) rp.load(a, (tt0 + wt * TW) * 16, lane);
    ACC acc[NW][TW], tot[RNG ? NW : 1][RNG ? TW : 1];
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j) {
            acc[i][j] = ACC{0, 0, 0, 0};
            if constexpr (RNG) tot[i][j] = ACC{0, 0, 0, 0};
        }
    i32x4 A[2][NW], B[2][TW];
    auto read = [&](int p, int stg) {
        const char* sb = sm + stg * SB;
#pragma unroll
        for (int i = 0; i < NW; ++i) A[p][i] = *(const i32x4*)(sb + (wn * NW + i) * 1024 + lane * 16);
#pragma unroll
        for (int j = 0; j < TW; ++j) B[p][j] = *(const i32x4*)(sb + (BN + wt * TW + j) * 1024 + lane * 16);
    };
    // end of the first K range with any chunk (K shorter than ksplit chunks leaves some empty)
    int range = 0, bound = 0;
    auto next_bound = [&](int c) {
        while (bound <= c && range < a.ksplit) bound = (int)(((long)++range * C) / a.ksplit);
    };
    if constexpr (RNG) next_bound(0);
#pragma unroll
    for (int q = 0; q < D; ++q) load(q, q + 1 < NS);
    stage_wait<(D - 1) * LD>();
    read(0, 0);
    for (int s0 = 0; s0 < NS; s0 += D) {
#pragma unroll
        for (int q = 0; q < D; ++q) {
            const int s = s0 + q, p = q & 1;
            // stage q is read by every wave, stage q + 1 has landed
            stage_wait<(D - 2) * LD>();
            load(q, s + D + 1 < NS);
            __builtin_amdgcn_sched_barrier(0);  // the loads go first, not behind the LDS reads
            read(p ^ 1, (q + 1) % D);
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int j = 0; j < TW; ++j) acc[i][j] = mfma_step<WT>(A[p][i], B[p][j], acc[i][j]);
            if constexpr (NW * TW == 32) {
                // two MFMAs per LDS read (left to itself the compiler puts the
                // reads in front): 256 x 256 blocks 201 -> 193 us for the 7B
                // gate/up at 1024 rows in a copy of the loop that only stores;
                // 128 x 128 blocks were slower this way
#pragma unroll
                for (int k = 0; k < NW + TW; ++k) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x8, 2, 0);
                }
            }
            if constexpr (RNG) {
                if (q % FRAG_U == FRAG_U - 1 && s / FRAG_U + 1 == bound) {
                    mfma_result_pad();
#pragma unroll
                    for (int i = 0; i < NW; ++i)
#pragma unroll
                        for (int j = 0; j < TW; ++j) {
                            tot[i][j] += acc[i][j];
                            acc[i][j] = ACC{0, 0, 0, 0};
                        }
                    next_bound(bound);
                }
            }
        }
        asm volatile("" ::: "memory");  // the last step's reads stay before the next round's barrier
    }
    stage_wait<0>();
    mfma_result_pad();
    const int row0 = (tt0 + wt * TW) * 16, tile0 = tn0 + wn * NW;
    if (row0 >= a.T) return;
    if constexpr (BFX) {
        RopePre ro[2];
        if constexpr (EPI == EPI_QKV) ro[0].load(a, min(tile0, ntiles - 1), lane, rp);
        uint16_t* ep = (uint16_t*)sm + wave * EP_LDS;  // every wave is done with the ring
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            if (EPI == EPI_QKV && i + 1 < NW) ro[(i + 1) & 1].load(a, min(tile0 + i + 1, ntiles - 1), lane, rp);
            if (tile0 + i >= ntiles) continue;
            if constexpr (RNG) rows_epilogue<EPI>(a, tot[i], tile0 + i, ntiles - 1, lane, row0, rp, ro[i & 1], ep);
            else rows_epilogue<EPI>(a, acc[i], tile0 + i, ntiles - 1, lane, row0, rp, ro[i & 1], ep);
        }
    } else {
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            if (tile0 + i >= ntiles) continue;
            QkvPre<TW> qp;
            if constexpr (EPI == EPI_QKV) qp.load(a, tile0 + i, lane, row0);
            if constexpr (RNG) gemm_epilogue<WT, TW, EPI, AT, 1, true>(a, tot[i], tile0 + i, ntiles - 1, lane, qp, row0);
            else gemm_epilogue<WT, TW, EPI, AT, 1, true>(a, acc[i], tile0 + i, ntiles - 1, lane, qp, row0);
        }
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

template <int WT, int NW, int TW, int WN, int WT_, int EPI, typename AT, bool KM, bool RNG, bool SPL = false>
static hipError_t gemm_rows_launch(const GemmArgs& a, hipStream_t s) {
    const int nT = ((a.T + 15) / 16 + TW * WT_ - 1) / (TW * WT_), nN = (a.N / 16 + NW * WN - 1) / (NW * WN);
    hipLaunchKernelGGL((k_gemm_rows<WT, NW, TW, WN, WT_, 4, EPI, AT, KM, RNG, SPL>), dim3(nT * nN, SPL ? a.ksplit : 1),
                       dim3(64 * WN * WT_), 0, s, a);
    return hipGetLastError();
}

// Blocks of 128 x 128 as eight waves of 32 x 64 (64 KB: two workgroups per CU),
// 128 x 256 as eight of 64 x 64, or 256 x 256 as eight of 128 x 64.  The larger
// ones read less LDS per MFMA but come one per CU: in a copy of the loop that
// only stores its sums, at K = 4096, a CU's first 128 x 128 block took 40 us and
// each further one 32-36, a round of 128 x 256 blocks 57-65 us, one of 256 x 256
// blocks 90-105.  The block with the least cost in these units is taken, at
// every K.  These kernels in a prefill, by events, the three blocks in turn
// (* the rule's):
//   QKV      7B 1024 rows *108 / 123 / 102 us, 2048 rows 207 / *198 / 208;
//            13B 1024 168 / 152 / *135; 8B (K ranges) 1504 *98 / 120
//   gate/up  7B 512 rows 100 / 111 / *86, 1024 *182 / 166 / 182, 2048 340 / 334 /
//            *286; 13B 1024 268 / 270 / *229; 8B 2048 436 / 396 / *380
//   down     7B 1024 *101 / 138, 2048 186 / *159; 8B 1504 225 / *184
// The rule misses the best one at 1024 rows of 7B (QKV by 6%, gate/up by 9%).
// (In the same copy of the loop, the 7B down projection: 128 x 128 as eight
// waves 88 us, as four 96; rings of eight stages 113.)
// Small matrices: up to 64 blocks of 128 x 128 would leave most CUs without
// one, so blocks of 64 x 64 (four waves of 16 x 64).  1000 rows, 128 x 128
// against 64 x 64 blocks: QKV of the 512-wide decoder 13.2 -> 7.7 us, its
// down projection 16.8 -> 11.7, that of the 1024-wide one 27.2 -> 18.7,
// QKV of the 256-wide fp32 decoder 30.6 -> 12.7.
RowsBlock gemm_rows_block(int N, int T, int ksplit) {
    const int tt = (T + 15) / 16, tn = N / 16;
    auto blocks = [&](int bn, int bt) { return (long)((tt + bt - 1) / bt) * ((tn + bn - 1) / bn); };
    const long n1 = blocks(8, 8), n2 = blocks(8, 16), n4 = blocks(16, 16);
    const double c1 = n1 <= 256 ? 1.2 : std::max(2.0, n1 / 256.0);
    const double c2 = 1.8 * ((n2 + 255) / 256), c4 = 3.0 * ((n4 + 255) / 256);
    if (n1 <= 64) return RB_64_64;
    if (ksplit == 1 && c4 < c1 && c4 < c2) return RB_256_256;
    return c2 < c1 ? RB_128_256 : RB_128_128;
}

template <int WT, int EPI, typename AT, bool KM, bool RNG>
static hipError_t gemm_rows_shape(const GemmArgs& a, hipStream_t s) {
    switch (gemm_rows_block(a.N, a.T, a.ksplit)) {
    case RB_64_64:  // (a matrix whose K range is whole has 8192 rows or more)
        if constexpr (RNG) return gemm_rows_launch<WT, 1, 4, 4, 1, EPI, AT, KM, true>(a, s);
        break;
    case RB_128_128: return gemm_rows_launch<WT, 2, 4, 4, 2, EPI, AT, KM, RNG>(a, s);
    case RB_128_256: return gemm_rows_launch<WT, 4, 4, 2, 4, EPI, AT, KM, RNG>(a, s);
    case RB_256_256:  // (both accumulators of a range would not fit the registers)
        if constexpr (!RNG) return gemm_rows_launch<WT, 8, 4, 2, 4, EPI, AT, KM, false>(a, s);
        break;
    }
    return hipErrorInvalidValue;
}
template <int WT, int EPI, typename AT, bool KM>
static hipError_t gemm_rows_go(const GemmArgs& a, hipStream_t s) {
    if (a.kmaj != (int)KM) return hipErrorInvalidValue;
    return a.ksplit > 1 ? gemm_rows_shape<WT, EPI, AT, KM, true>(a, s) : gemm_rows_shape<WT, EPI, AT, KM, false>(a, s);
}

// Residual projections of few rows (up to 128 blocks of 128 x 128: 512 rows of
// the 7B shapes) leave most of the chip idle and hand each K range to a
// workgroup of its own.
bool gemm_rows_split(int wtype, int N, int Kp, int T) {
    return T <= PF_SPLIT_ROWS && gemm_parts_count(wtype, N, Kp, 1) > 1 && (long)((T + 127) / 128) * ((N + 127) / 128) <= 128;
}

template <int WT, typename AT>
static hipError_t gemm_rows_epi(int epi, const GemmArgs& a, hipStream_t s) {
    switch (epi) {
    case EPI_STORE:  // split partial sums
        if (a.kmaj || a.ksplit < 2 || a.part_stride < (size_t)a.T * a.ldo) return hipErrorInvalidValue;
        return gemm_rows_launch<WT, 2, 4, 4, 2, EPI_STORE, AT, false, false, true>(a, s);
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

// The same through the builtin, for stages the compiler can tell apart
// (separate arrays): it waits for a wave's own loads before that wave's reads.
// The other waves' reads are what stage_wait<0>() is for: every wave's loads
// have landed before the barrier lets any of them read.
__device__ __forceinline__ void lds_load16_b(const void* src, void* dst) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

// Causal attention of a prefill.  Workgroup = (kv head, four query tiles of 16
// rows; the G heads of a group at the same rows follow each other, so its
// waves need about the same slots).  It walks the splits of 256 slots that
// its rows see; a split's K and then its V pass through LDS in halves (32 KB
// each at head_dim 128, two buffers, direct-to-LDS loads: each half arrives
// while the previous one is used), and each wave computes the split's partial of
// its rows exactly as k_attn_rows does and merges it into its running state
// exactly as k_attn_merge does, in split order: the same bits as a forward of
// up to 128 rows, without the partials' trip through memory.  Parts wholly
// past a tile's last row would add zero and are left out.
// Most of what it issues is the softmax: by counters 1280 VALU instructions
// against 192 MFMAs per wave and split, and the matrix cores are 15% busy (7B,
// 1024 tokens).  Two workgroups of 64 rows per CU even out the rows' unequal
// walks: eight waves on 128 KB of whole K and V stages, one workgroup per CU,
// took 38 us per layer for 1024 tokens of the 7B shape and 93 for 1501 of 8B
// (after 1500); these take 32 and 86.
template <int HD>
__global__ void __launch_bounds__(256, 2) k_attn_causal(const AttnArgs a, float scale_log2) {
    constexpr int UD = HD / 32, DG = HD / 4, NDT = HD / 16, TE = 32 * HD, QW = 4;
    constexpr int NP = ATT_WAVES, NTS = NP * ATT_TPW, NTH = NTS / 2, KF = 2 * UD, LP = NTH * KF / QW;
    static_assert(KF == NDT && LP * QW == NTH * KF, "K and V stages must match");
    __shared__ i32x4 sa[NTH * KF * 64], sb[NTH * KF * 64];
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
    auto load = [&](const uint16_t* base, i32x4* dst, int split, int half) {
#pragma unroll
        for (int i = 0; i < LP; ++i) {
            const int f = wave * LP + i, tile = min(split * NTS + half * NTH + f / KF, n_tiles - 1);
            lds_load16_b(base + (size_t)tile * TE + (f % KF) * 512, dst + f * 64);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x4 acc[NDT];
    float L = 0.f, M = -1e30f;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float x[NP][ATT_TPW][8], m[NP], Ms, l;
    f32x4 o[NDT];
    auto scores = [&](const i32x4* ks, int base, int half) {
#pragma unroll
        for (int ph = 0; ph < NP / 2; ++ph) {
            const int p = half * (NP / 2) + ph;
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
                            S[h2] = mfma_step<ET_BF16>(ks[((ph * ATT_TPW + tt) * KF + h2 * UD + u) * 64 + lane], Qf[u], S[h2]);
                    }
                    attn_tile_scores(S, bits8(0, vl - (base + (p * ATT_TPW + tt) * 32 + 8 * g)), scale_log2, x[p][tt]);
                }
                m[p] = attn_part_max<ATT_TPW>(x[p]);
                Ms = fmaxf(Ms, m[p]);
            }
        }
    };
    auto values = [&](const i32x4* vs, int base, int half) {
#pragma unroll
        for (int ph = 0; ph < NP / 2; ++ph) {
            const int p = half * (NP / 2) + ph;
            if (base + p * 32 * ATT_TPW >= wslots) continue;
            i32x4 Pf[ATT_TPW], Pl[ATT_TPW];
            const float lp = attn_part_probs<ATT_TPW>(x[p], m[p], Pf, Pl);
            const float f = attn_merge_weight(m[p], Ms);
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt) {
                f32x4 po = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int tt = 0; tt < ATT_TPW; ++tt) {
                    const i32x4 v = vs[((ph * ATT_TPW + tt) * NDT + dt) * 64 + lane];
                    po = mfma_step<ET_BF16>(v, Pf[tt], po);
                    po = mfma_step<ET_BF16>(v, Pl[tt], po);
                }
                attn_merge_o(o[dt], po, f);
            }
            attn_merge_l(l, lp, f);
        }
    };
    load(kbase, sa, 0, 0);
    stage_wait<0>();
    for (int split = 0; split < nsplit; ++split) {
        const int base = split * ATT_SPLIT;
        Ms = -1e30f;
        l = 0.f;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        load(kbase, sb, split, 1);
        scores(sa, base, 0);
        stage_wait<0>();  // what was loaded is there, what was used is free
        load(vbase, sa, split, 0);
        scores(sb, base, 1);
        stage_wait<0>();
        load(vbase, sb, split, 1);
        values(sa, base, 0);
        stage_wait<0>();
        if (split + 1 < nsplit) load(kbase, sa, split + 1, 0);
        values(sb, base, 1);
        if (base < wslots) attn_merge_split<NDT>(acc, L, M, o, l, Ms);
        stage_wait<0>();
    }
    const int t = t0 + r;
    if (t < T) {
        const float inv = L > 0.f ? 1.f / L : 0.f;
        const int nto = row_tiles(T);
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
    const int nct = (a.T + 15) / 16 * (a.H / a.Hkv), nblk = (nct + 3) / 4;
    const float scale_log2 = (1.0f / sqrtf((float)a.hd)) * 1.4426950408889634f;
    if (a.hd == 128) hipLaunchKernelGGL(k_attn_causal<128>, dim3(nblk * a.Hkv), dim3(256), 0, s, a, scale_log2);
    else hipLaunchKernelGGL(k_attn_causal<64>, dim3(nblk * a.Hkv), dim3(256), 0, s, a, scale_log2);
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
