// evidence.hip -- evidence kernel: the frontier pass plus, per boundary, the runner-up gap and
// the tie-set size (localization evidence, Sec. 4) and max_r d / sum_r d
// (the per-stage terms of the max and mean baselines, Props. 1 and 2).
//
// One workgroup per step (WG = 64 or 128 threads).  Each lane accumulates,
// over its ranks of a tile, the two largest packed keys, the number of its
// ranks whose prefix equals that of its largest key, and the max and sum of
// the stage's durations.  The wave reduces these with DPP lane moves.  Sums
// and counts are not idempotent, so every move used gives each receiving lane
// a distinct partner; lanes a row broadcast does not reach hold partial
// values that are never read.  The full result is in lane 63.

#include "sf_device.h"
#include "sf_host.h"

namespace sfk {

struct EvAcc {
    u64 k1, k2;      // largest and second-largest packed key
    int64_t smax;    // max of d over ranks
    int64_t ssum;    // sum of d over ranks
    uint32_t c;      // ranks whose prefix equals that of k1
};

__device__ __forceinline__ void ev_merge(EvAcc& a, const EvAcc& b)
{
    const u64 pa = a.k1 >> kRankBits, pb = b.k1 >> kRankBits;
    a.c = pa > pb ? a.c : (pb > pa ? b.c : a.c + b.c);
    a.k2 = umax64(umin64(a.k1, b.k1), umax64(a.k2, b.k2));
    a.k1 = umax64(a.k1, b.k1);
    a.smax = a.smax > b.smax ? a.smax : b.smax;
    a.ssum += b.ssum;
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ EvAcc ev_move(const EvAcc& a)
{
    EvAcc b;
    b.k1 = dpp_move<CTRL, ROW_MASK>(a.k1);
    b.k2 = dpp_move<CTRL, ROW_MASK>(a.k2);
    b.smax = (int64_t)dpp_move<CTRL, ROW_MASK>((u64)a.smax);
    b.ssum = (int64_t)dpp_move<CTRL, ROW_MASK>((u64)a.ssum);
    b.c = (uint32_t)__builtin_amdgcn_update_dpp((int)a.c, (int)a.c, CTRL, ROW_MASK, 0xF, false);
    return b;
}

// Merge over aligned groups of SUB lanes (a power of two <= 64); the result
// is valid in the last lane of each group.
template <int SUB>
__device__ __forceinline__ EvAcc ev_group_reduce(EvAcc a)
{
    if (SUB >= 2) ev_merge(a, ev_move<0xB1, 0xF>(a));   // quad_perm [1,0,3,2]: lane ^ 1
    if (SUB >= 4) ev_merge(a, ev_move<0x4E, 0xF>(a));   // quad_perm [2,3,0,1]: lane ^ 2
    if (SUB >= 8) ev_merge(a, ev_move<0x141, 0xF>(a));  // row_half_mirror: other quad of 8
    if (SUB >= 16) ev_merge(a, ev_move<0x140, 0xF>(a)); // row_mirror: other half of the row
    if (SUB >= 32) ev_merge(a, ev_move<0x142, 0xA>(a)); // row_bcast:15: row 0 -> 1, row 2 -> 3
    if (SUB >= 64) ev_merge(a, ev_move<0x143, 0xC>(a)); // row_bcast:31: rows 0-1 -> row 3
    return a;
}

__device__ __forceinline__ void ev_store(int64_t i, const EvAcc& a, u64 kprev, int R,
                                         int64_t* inc, int32_t* lead, int64_t* gap,
                                         int32_t* ties, int64_t* stage_max, int64_t* stage_sum)
{
    const int64_t F = (int64_t)(a.k1 >> kRankBits);
    inc[i] = F - (int64_t)(kprev >> kRankBits);
    lead[i] = (int32_t)(kRankMask - (a.k1 & kRankMask));
    gap[i] = R > 1 ? F - (int64_t)(a.k2 >> kRankBits) : -1;
    ties[i] = (int32_t)a.c;
    stage_max[i] = a.smax;
    stage_sum[i] = a.ssum;
}

// Same step/lane layout as k_frontier: G lanes per step, K ranks per lane,
// WG / G steps per workgroup.  When one group of at most 64 lanes covers all
// R ranks of its step, the group's last lane writes each boundary's outputs
// as soon as the stage is reduced (groups of up to 16 lanes: G boundaries at a
// time, a lane each; one lane's 8-byte stores leave the L2 partly filled lines
// of more steps than it holds: 16 ranks x 74 x 75909 668 -> 232 us);
// otherwise partial results go through LDS
// (5 arrays of [WG / min(G, 64)][S]) and the workgroup writes them at the end.
// GTAB (stage counts past what LDS holds; G <= 64): the group's last lane
// keeps the partial results of its step in the step's own output rows (the
// largest key in out_increment, the runner-up key in out_gap, the tie count,
// max and sum in their final rows), and after the last tile the workgroup
// decodes the increment, leader and gap in place, chunk by chunk from the
// end, each chunk read before any of it is written.
//
// The ranks are loaded in pairs, 16 bytes at any 8-byte alignment (V: 1 where
// R == 1, 2 for even R, 3 for odd).  Slots past R, and at odd R the first slot of the last pair
// (it overlaps the pair before), load ranks that other slots hold: their
// duration counts as 0 and their key stays 0, below every real key.
// D: stage rows in flight (as in k_frontier).
template <int V, int K, int G, int WG, bool GTAB, int D>
__global__ __launch_bounds__(WG) void k_frontier_evidence(
    const int64_t* __restrict__ d, int64_t T, int R, int S, int64_t* __restrict__ inc,
    int32_t* __restrict__ lead, int64_t* __restrict__ gap, int32_t* __restrict__ ties,
    int64_t* __restrict__ stage_max, int64_t* __restrict__ stage_sum)
{
    constexpr int VEC = V == 1 ? 1 : 2;
    constexpr bool ODD = V == 3;
    static_assert(K % VEC == 0 && (WG % G == 0 || G == WG), "shape");
    static_assert(!GTAB || G <= 64, "GTAB: one writer lane per step");
    constexpr int SUB = G < 64 ? G : 64;
    constexpr int SPW = WG / G;
    constexpr int SPS = G / SUB;
    constexpr int NSLOT = WG / SUB;
    constexpr int NLD = K / VEC;
    constexpr int RT = G * K;

    extern __shared__ u64 evtab[];
    u64* t_k1 = evtab;
    u64* t_k2 = t_k1 + NSLOT * S;
    u64* t_c = t_k2 + NSLOT * S;
    u64* t_max = t_c + NSLOT * S;
    u64* t_sum = t_max + NSLOT * S;

    const bool direct = SPS == 1 && R <= RT;  // uniform over the launch
    const int tid = threadIdx.x;
    const int gl = tid % G;
    const int slot = tid / SUB;
    const bool writer = (tid % SUB) == SUB - 1;
    const int64_t tb = xcd_block() * SPW;
    // wave-uniform where a wave holds one step: the row base in SGPRs
    const int64_t t = tb + (G >= 64 ? __builtin_amdgcn_readfirstlane(tid / G) : tid / G);

    if (t < T) {  // uniform over the step group
        const int64_t* dt = d + t * (int64_t)S * R;
        for (int r0 = 0; r0 < R; r0 += RT) {
            // (a tile of one rank starts one below it)
            const int rb = r0 < R - VEC ? r0 : R - VEC;
            const int last = R - VEC - rb;  // the last pair's place in the tile
            u64 q[K];
            bool ok[NLD], ok0[NLD];  // the pair's second (or only), first slot holds a rank
#pragma unroll
            for (int l = 0; l < NLD; ++l) {
                const int r = r0 + (l * G + gl) * VEC;
                ok[l] = r < R;
                ok0[l] = ODD ? r <= R - VEC : ok[l];
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const int at = ok0[l] ? r + e : R - VEC + e;
                    q[l * VEC + e] = (ODD && e == 0 ? ok0[l] : ok[l]) ? (kRankMask - (u64)at) : 0ull;
                }
            }
            int64_t v[D][K];
            auto load_row = [&](int c, int s) {
                const int64_t* row = dt + (int64_t)s * R + rb;
#pragma unroll
                for (int l = 0; l < NLD; ++l) {
                    const uint32_t idx = (uint32_t)(ok0[l] ? (l * G + gl) * VEC : last);
                    if (VEC == 2) {
                        const v2i64_a8 x = __builtin_nontemporal_load(reinterpret_cast<const v2i64_a8*>(row + idx));
                        v[c][2 * l] = x.x;
                        v[c][2 * l + 1] = x.y;
                    } else {
                        v[c][l] = __builtin_nontemporal_load(row + idx);
                    }
                }
            };
            u64 kprev = 0, hprev = 0;
            EvAcc a, held = {};
            auto advance = [&](int c) {
                a.k1 = 0;
                a.k2 = 0;
                a.smax = 0;
                a.ssum = 0;
                a.c = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int64_t dv = (ODD && k % 2 == 0 ? ok0[k / VEC] : ok[k / VEC]) ? v[c][k] : 0;
                    q[k] += (u64)dv << kRankBits;
                    a.k2 = umax64(a.k2, umin64(a.k1, q[k]));
                    a.k1 = umax64(a.k1, q[k]);
                    a.smax = a.smax > dv ? a.smax : dv;
                    a.ssum += dv;
                }
#pragma unroll
                for (int k = 0; k < K; ++k)
                    a.c += ((ODD && k % 2 == 0 ? ok0[k / VEC] : ok[k / VEC]) && ((q[k] ^ a.k1) >> kRankBits) == 0) ? 1u : 0u;
            };
            auto reduce = [&](int s) {
                a = ev_group_reduce<SUB>(a);
                if (G <= 16 && direct) {
                    // every lane has the result: lane s % G keeps it, and G
                    // boundaries are written at once
                    const int own = s % G;
                    if (gl == own) {
                        held = a;
                        hprev = kprev;
                    }
                    kprev = a.k1;
                    if ((own == G - 1 || s == S - 1) && gl <= own)
                        ev_store(t * S + s - own + gl, held, hprev, R, inc, lead, gap, ties, stage_max, stage_sum);
                } else if (writer) {
                    if (direct) {
                        ev_store(t * S + s, a, kprev, R, inc, lead, gap, ties, stage_max, stage_sum);
                        kprev = a.k1;
                    } else if (GTAB) {
                        // the step's own output rows, read back by this lane
                        // only until the decode below
                        const int64_t i = t * S + s;
                        if (r0 > 0) {
                            EvAcc b;
                            b.k1 = (u64)inc[i];
                            b.k2 = (u64)gap[i];
                            b.c = (uint32_t)ties[i];
                            b.smax = stage_max[i];
                            b.ssum = stage_sum[i];
                            ev_merge(a, b);
                        }
                        inc[i] = (int64_t)a.k1;
                        gap[i] = (int64_t)a.k2;
                        ties[i] = (int32_t)a.c;
                        stage_max[i] = a.smax;
                        stage_sum[i] = a.ssum;
                    } else {
                        const int i = slot * S + s;
                        if (r0 > 0) {
                            EvAcc b;
                            b.k1 = t_k1[i];
                            b.k2 = t_k2[i];
                            b.c = (uint32_t)t_c[i];
                            b.smax = (int64_t)t_max[i];
                            b.ssum = (int64_t)t_sum[i];
                            ev_merge(a, b);
                        }
                        t_k1[i] = a.k1;
                        t_k2[i] = a.k2;
                        t_c[i] = a.c;
                        t_max[i] = (u64)a.smax;
                        t_sum[i] = (u64)a.ssum;
                    }
                }
            };
            if constexpr (D == 1) {
                load_row(0, 0);
                for (int s = 0; s < S; ++s) {
                    advance(0);
                    if (s + 1 < S) load_row(0, s + 1);
                    reduce(s);
                }
            } else {
#pragma unroll
                for (int c = 0; c < D; ++c)
                    if (c < S) load_row(c, c);
                int s = 0;
                for (; s + 2 * D <= S; s += D) {
#pragma unroll
                    for (int c = 0; c < D; ++c) {
                        advance(c);
                        load_row(c, s + c + D);
                        reduce(s + c);
                    }
                }
                for (; s < S; s += D) {
#pragma unroll
                    for (int c = 0; c < D; ++c) {
                        if (s + c < S) {
                            advance(c);
                            if (s + c + D < S) load_row(c, s + c + D);
                            reduce(s + c);
                        }
                    }
                }
            }
        }
    }
    if (direct) return;
    __syncthreads();

    if constexpr (GTAB) {
        // the workgroup's steps are contiguous rows; a chunk of WG entries
        // reads its keys and the key before each (in the same chunk or the
        // one below, not yet decoded), waits for every thread's reads, then
        // writes.  The tie count, max and sum are final already.
        const int64_t steps = T - tb < SPW ? T - tb : SPW;
        const int64_t n = steps * S;
        const int64_t base = tb * S;
        for (int64_t c = (n - 1) / WG; c >= 0; --c) {
            const int64_t i = c * WG + tid;
            const bool ok = i < n;
            u64 key = 0, kprev = 0, key2 = 0;
            if (ok) {
                key = (u64)inc[base + i];
                key2 = (u64)gap[base + i];
                if (i % S != 0) kprev = (u64)inc[base + i - 1];
            }
            __syncthreads();
            if (ok) {
                const int64_t F = (int64_t)(key >> kRankBits);
                inc[base + i] = F - (int64_t)(kprev >> kRankBits);
                lead[base + i] = (int32_t)(kRankMask - (key & kRankMask));
                gap[base + i] = R > 1 ? F - (int64_t)(key2 >> kRankBits) : -1;
            }
        }
        return;
    }

    for (int i = tid; i < SPW * S; i += WG) {
        const int jj = i / S;
        const int s = i - jj * S;
        const int64_t tt = tb + jj;
        if (tt >= T) break;
        EvAcc a, p;
        const int i0 = jj * SPS * S + s;
        a.k1 = t_k1[i0];
        a.k2 = t_k2[i0];
        a.c = (uint32_t)t_c[i0];
        a.smax = (int64_t)t_max[i0];
        a.ssum = (int64_t)t_sum[i0];
        u64 kp = s > 0 ? t_k1[i0 - 1] : 0;
#pragma unroll(SPS <= 4 ? SPS : 2)
        for (int qd = 1; qd < SPS; ++qd) {
            const int iq = (jj * SPS + qd) * S + s;
            p.k1 = t_k1[iq];
            p.k2 = t_k2[iq];
            p.c = (uint32_t)t_c[iq];
            p.smax = (int64_t)t_max[iq];
            p.ssum = (int64_t)t_sum[iq];
            ev_merge(a, p);
            if (s > 0) kp = umax64(kp, t_k1[iq - 1]);
        }
        ev_store(tt * S + s, a, kp, R, inc, lead, gap, ties, stage_max, stage_sum);
    }
}

struct EvidenceVariant {
    const void* fn;
    int K, G, WG;
    int per_cu;  // resident workgroups per CU to allow (0: no cap)
};

template <int V, int K, int G, int WG, bool GTAB = false, int D = 1>
EvidenceVariant ev_variant(int per_cu)
{
    return EvidenceVariant{reinterpret_cast<const void*>(&k_frontier_evidence<V, K, G, WG, GTAB, D>),
                           K, G, WG, per_cu};
}

// LDS bytes a variant needs: none when one group of <= 64 lanes covers the
// step's ranks or the partial results live in the output rows, else 5
// arrays of [WG / min(G, 64)][S] u64.
size_t ev_lds_need(const EvidenceVariant& v, int R, int S, bool gtab)
{
    const int sub = v.G < 64 ? v.G : 64;
    if (gtab || (v.G <= 64 && R <= v.G * v.K)) return 0;
    return (size_t)5 * (v.WG / sub) * S * 8;
}

// Few steps (measured on MI355X): a wave or more per step and four rows in
// flight, where the shapes below leave the chip idle (1023 ranks x 8 x 128 26 ->
// 12 us, 130 x 60 x 128 120 -> 41).  Up to 1 MB of stage rows over all steps (at 8
// MB 27 -> 36); at 129 to 256 ranks, where the shapes below take two tiles, up
// to 1536 steps (200 x 12 x 1200 26 -> 22, 129 x 6 x 2000 14.3 -> 15.6); up to 128
// ranks, one wave per step, up to 1024 steps (100 x 12: 600 steps 13.8 -> 10.8,
// 1200 14.7 -> 16.1).  Past 8192 ranks all 1024 lanes, one workgroup per CU, up
// to 256 steps (16384 x 8: 150 steps 46 -> 40, 300 74 -> 86) and where the last
// tile is half full at least (24576 x 8 x 50 66 -> 74, 32768 88 -> 81; at 128
// VGPRs they spill 4, at odd ranks 7).  From 1025
// to 8192 ranks the reductions of so many waves cost more than they hide.
static bool ev_deep(int64_t T, int R, int S)
{
    if (R > 8192) return T <= 256 && (R - 1) % 16384 >= 8192;
    if (R <= 64 || R > 1024) return false;
    if (R <= 128) return T <= 1024 && S >= 4;
    if (R <= 256) return T <= 1536;
    return T * R * 8 <= 1 << 20 && (R > 512 || S >= 4);
}

template <int V>
EvidenceVariant pick_evidence_deep(int R)
{
    if (R <= 128) return ev_variant<V, 2, 64, 64, false, 4>(0);
    if (R <= 256) return ev_variant<V, 2, 128, 128, false, 4>(0);
    if (R <= 512) return ev_variant<V, 2, 256, 256, false, 4>(0);
    if (R <= 1024) return ev_variant<V, 2, 512, 512, false, 4>(0);
    return ev_variant<V, 16, 1024, 1024>(0);
}

// Launch shape by rank count, measured on MI355X: the pass is bound by its VALU
// work as much as by HBM (about 20 instructions per slot, ranks or not), so
// the tile is close to R, and its groups are as few lanes as hold it at 12 to
// 16 ranks each, since a reduction costs as much as 8 to 10 slots (1500 x 10
// x 8192: 356 -> 164 us, 671 x 8 x 8192 85 -> 63, 1024 x 12 x 8192 149 -> 128,
// 6001 x 10 x 1024 133 -> 84; 250 ranks on 32 lanes level, 256 110 against
// 115, 240 x 12 x 16000 72 against 67; 8192 ranks at 16 each, 32 MB of rows and more, 126 against 130).  A
// shape whose LDS would exceed 64 KB at this S falls back to half as many lanes
// (512 lanes past 204 stages: 8192 x 260, one step 1523 -> 600 us), else to two
// 64-lane slots per step (80 * S bytes, at most 64 KB).
template <int V>
EvidenceVariant pick_evidence(int64_t T, int R, int S)
{
    if (ev_deep(T, R, S)) {
        const EvidenceVariant v = pick_evidence_deep<V>(R);
        if (ev_lds_need(v, R, S, false) <= kLdsMaxPerWg) return v;
    }
    EvidenceVariant v;
    if (R == 1) v = ev_variant<1, 2, 4, 64>(0);
    else if (R <= 8) v = S < 8 ? ev_variant<V, 2, 4, 64>(0) : ev_variant<V, 2, 4, 64, false, 4>(0);
    else if (R <= 16) v = S < 8 ? ev_variant<V, 2, 8, 64>(0) : ev_variant<V, 2, 8, 64, false, 4>(0);
    else if (R <= 32) v = ev_variant<V, 4, 8, 64>(0);
    else if (R <= 64) v = ev_variant<V, 4, 16, 64>(0);
    else if (R <= 128) v = ev_variant<V, 8, 16, 256>(8);
    else if (R <= 240 && (R <= 144 || T * R * 8 < 24 << 20)) v = ev_variant<V, 8, 32, 64>(0);
    else if (R <= 256) v = ev_variant<V, 8, 16, 256>(8);
    else if (R <= 384) v = ev_variant<V, 12, 32, 64>(0);
    else if (R <= 512) v = ev_variant<V, 16, 32, 64>(0);
    else if (R <= 768) v = ev_variant<V, 12, 64, 64>(0);
    else if (R <= 1024) v = ev_variant<V, 16, 64, 64>(0);
    else if (R <= 1536) v = ev_variant<V, 12, 128, 128>(0);
    else if (R <= 2048) v = ev_variant<V, 16, 128, 128>(0);
    else if (R <= 3072) v = ev_variant<V, 12, 256, 256>(2);
    else if (R <= 4096) v = ev_variant<V, 16, 256, 256>(2);
    else if (R <= 6144) v = ev_variant<V, 12, 512, 512>(0);
    else if (R <= 8192 && T < 400) v = ev_variant<V, 16, 512, 512>(0);
    else if (R > 8192 && R <= 12288) v = ev_variant<V, 24, 512, 512>(0);
    else v = ev_variant<V, 32, 256, 256>(0);
    if (v.WG == 512 && ev_lds_need(v, R, S, false) > kLdsMaxPerWg) v = ev_variant<V, 32, 256, 256>(0);
    if (ev_lds_need(v, R, S, false) > kLdsMaxPerWg) v = ev_variant<V, 16, 128, 128>(0);
    return v;
}

// Stage counts whose LDS table would not fit even the two-slot fallback
// (more than 819 stages): one group of at most 64 lanes per step, the
// partial results in the output rows.
template <int V>
EvidenceVariant pick_evidence_gtab(int R)
{
    if (R == 1) return ev_variant<1, 2, 4, 64, true>(0);
    if (R <= 8) return ev_variant<V, 2, 4, 64, true>(0);
    if (R <= 16) return ev_variant<V, 2, 8, 64, true>(0);
    if (R <= 32) return ev_variant<V, 4, 8, 64, true>(0);
    if (R <= 64) return ev_variant<V, 4, 16, 64, true>(0);
    if (R <= 512) return ev_variant<V, 16, 32, 64, true>(0);
    return ev_variant<V, 16, 64, 64, true>(0);
}

}  // namespace sfk

using namespace sfk;

SF_API int sf_frontier_evidence(const int64_t* durations, int64_t T, int32_t R, int32_t S,
                                int64_t* out_increment, int32_t* out_leader, int64_t* out_gap,
                                int32_t* out_ties, int64_t* out_stage_max,
                                int64_t* out_stage_sum, sf_stream_t stream)
{
    if (T < 0 || R < 1 || R > SF_MAX_R || S < 1) return SF_EINVAL;
    if (!fits(T, S, R, 8)) return SF_EINVAL;
    if (T == 0) return SF_OK;
    if (T > INT32_MAX) return SF_EINVAL;
    const void* bufs[7] = {durations, out_increment, out_leader, out_gap,
                           out_ties, out_stage_max, out_stage_sum};
    const uintptr_t align[7] = {8, 8, 4, 8, 4, 8, 8};
    const int64_t ts = T * S;
    const int64_t sizes[7] = {ts * R * 8, ts * 8, ts * 4, ts * 8, ts * 4, ts * 8, ts * 8};
    for (int a = 0; a < 7; ++a)
        if (!bufs[a] || !aligned(bufs[a], align[a])) return SF_EINVAL;
    for (int a = 0; a < 7; ++a)
        for (int b = (a < 1 ? 1 : a + 1); b < 7; ++b)
            if (!disjoint(bufs[a], sizes[a], bufs[b], sizes[b])) return SF_EINVAL;

    const bool odd = R & 1;
    EvidenceVariant v = odd ? pick_evidence<3>(T, R, S) : pick_evidence<2>(T, R, S);
    const bool gtab = ev_lds_need(v, R, S, false) > kLdsMaxPerWg;
    if (gtab) v = odd ? pick_evidence_gtab<3>(R) : pick_evidence_gtab<2>(R);
    const int spw = v.WG / v.G;
    const size_t lds = lds_request(ev_lds_need(v, R, S, gtab), v.per_cu);
    const int64_t blocks = (T + spw - 1) / spw;
    int Ri = R, Si = S;
    void* args[] = {(void*)&durations, (void*)&T, (void*)&Ri, (void*)&Si,
                    (void*)&out_increment, (void*)&out_leader, (void*)&out_gap,
                    (void*)&out_ties, (void*)&out_stage_max, (void*)&out_stage_sum};
    return launch(v.fn, dim3((unsigned)blocks), dim3(v.WG), args, lds, stream);
}
