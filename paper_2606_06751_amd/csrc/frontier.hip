// frontier.hip -- sf_frontier: per-step frontier advances and leaders
// (Sec. 3, Eq. (1)) on gfx950.
//
// Data layout in HBM: durations [T][S][R] int64 (rank fastest), outputs
// [T][S].
//
// Frontier kernel.  Every step is independent (Sec. 3 streams one step at a
// time), so the grid walks the step axis; inside a step, a group of G lanes
// owns the step and each lane owns K ranks of a tile of G*K ranks.  The lane
// keeps the running prefix of each of its ranks in registers as a packed key
//     q = (P << 16) | (0xFFFF - r)
// so that an unsigned 64-bit max over keys yields the largest prefix and, on
// equal prefixes, the lowest rank.  Adding a duration shifted left by 16
// advances P without touching the rank field, so the key is built once per
// rank and then only added to.  Per stage, a lane takes the max of its K
// keys, the group reduces with DPP lane moves (quad_perm, row mirrors,
// row broadcasts: no LDS traffic), and the last lane of each 64-lane (or
// smaller) sub-group stores the partial max in LDS.  After the last stage
// the workgroup decodes F and the leader per (step, stage), takes the
// advance F[s] - F[s-1] and writes [T][S] rows with contiguous stores.
// Durations are read exactly once, in 16-byte loads of rank pairs at any
// 8-byte alignment (odd R shifts every other row by half a load).
//
// The large shapes keep one stage row per lane group in flight and rely on
// many steps at once to fill the memory system.  With few steps the pass is
// bound by latency instead: the deep shapes spread a step over more lanes
// (2 to 16 ranks each) and keep D stage rows in flight.
//
// Stage counts beyond what LDS holds (the gradient-accumulation expansion of
// Sec. 3 multiplies S by the number of micro-steps) take the GTAB variant:
// one group of at most 64 lanes owns a step, and its last lane keeps the
// step's per-stage partial maxima in the step's own out_increment row (the
// caller's output, so no extra memory); after the last tile the workgroup
// decodes those rows in place, chunk by chunk from the end, each chunk read
// before any of it is written.
//
// The checked variant also verifies the data contract on the way: every
// duration in [0, 2^47) (its high word below 2^15) and every prefix below
// 2^47 (the top bit of every key clear: while all durations are below 2^47
// a prefix that first reaches 2^47 is still below 2^48, so its key's top bit
// is set at that stage).  A wave that sees a violation ORs SF_ERANGE into the
// caller's status word.
//

#include "sf_device.h"
#include "sf_host.h"

namespace sfk {

// VEC: int64 elements per load (2, or 1 where R == 1); K: ranks per lane per
//      tile; G: lanes per step;
// WG:  threads per workgroup (WG / G steps per workgroup); CHECK: verify the
//      data contract into *status; GTAB: partial maxima in the out_increment
//      rows instead of LDS (any S; G <= 64); D: stage rows in flight.
template <int VEC, int K, int G, int WG, bool CHECK, bool GTAB, int D>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(K == 16 && G == 32 && !CHECK ? 4 : 1))) void k_frontier(const int64_t* __restrict__ d, int64_t T,
                                                 int R, int S, int64_t* __restrict__ inc,
                                                 int32_t* __restrict__ lead,
                                                 uint32_t* __restrict__ status)
{
    static_assert(K % VEC == 0, "K must be a multiple of VEC");
    static_assert(WG % G == 0 || G == WG, "a workgroup holds whole steps");
    static_assert(!GTAB || G <= 64, "GTAB: one writer lane per step");
    constexpr int SUB = G < 64 ? G : 64;  // lanes per DPP reduction group
    constexpr int SPW = WG / G;           // steps per workgroup
    constexpr int SPS = G / SUB;          // LDS slots per step
    constexpr int NLD = K / VEC;          // loads per lane per stage row
    constexpr int RT = G * K;             // ranks per tile

    extern __shared__ u64 tab[];          // [WG / SUB][S] partial maxima

    const int tid = threadIdx.x;
    const int gl = tid % G;
    // wave-uniform where a wave holds one step: the row base in SGPRs
    const int j = G >= 64 ? __builtin_amdgcn_readfirstlane(tid / G) : tid / G;
    const int slot = tid / SUB;
    const bool writer = (tid % SUB) == SUB - 1;
    const int64_t lb = xcd_block();  // XCD-contiguous step runs
    const int64_t t = lb * SPW + j;
    uint32_t dhi = 0, khi = 0;  // CHECK: OR of the durations' and the keys' high words

    if (t < T) {  // uniform over the step group
        const int64_t* dt = d + t * (int64_t)S * R;
        for (int r0 = 0; r0 < R; r0 += RT) {
            // A slot past R takes the last rank pair again (in bounds, the
            // same cache line): a duplicate of a real key changes no maximum,
            // and neither does the overlap of a last pair at odd R.
            u64 q[K];
            bool ok[NLD];
            const int rb = r0 < R - VEC ? r0 : R - VEC;  // a tile of one rank starts one below it
            const int last = R - VEC - rb;
#pragma unroll
            for (int l = 0; l < NLD; ++l) {
                const int i = (l * G + gl) * VEC;
                ok[l] = i <= last;
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    q[l * VEC + e] = kRankMask - (u64)(rb + (ok[l] ? i : last) + e);
            }
            int64_t v[D][K];
            auto load_row = [&](int c, int s) {
                const int64_t* row = dt + (int64_t)s * R + rb;
#pragma unroll
                for (int l = 0; l < NLD; ++l) {
                    const uint32_t idx = (uint32_t)(ok[l] ? (l * G + gl) * VEC : last);
                    if (VEC == 2) {
                        const v2i64_a8 x = __builtin_nontemporal_load(reinterpret_cast<const v2i64_a8*>(row + idx));
                        v[c][2 * l] = x.x;
                        v[c][2 * l + 1] = x.y;
                    } else {
                        v[c][l] = __builtin_nontemporal_load(row + idx);
                    }
                }
            };
            u64 m;
            auto advance = [&](int c) {
                m = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    q[k] += (u64)v[c][k] << kRankBits;
                    m = umax64(m, q[k]);
                    if (CHECK) dhi |= (uint32_t)((u64)v[c][k] >> 32);
                }
                if (CHECK) khi |= (uint32_t)(m >> 32);
            };
            auto reduce = [&](int s) {
                m = group_max<SUB>(m);
                if (writer) {
                    // GTAB: the step's own out_increment row, read back by
                    // the same lane only until the decode below
                    u64* p = GTAB ? reinterpret_cast<u64*>(inc) + t * S + s : &tab[slot * S + s];
                    *p = (r0 == 0) ? m : umax64(*p, m);
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
                // row s + D is always there: no branch between the loads, so
                // each stage waits for its own row only
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
    if (CHECK) {
        const u64 bad = __ballot((dhi >> 15) != 0 || (khi >> 31) != 0);
        if (bad != 0 && (tid & 63) == __builtin_ctzll(bad)) atomicOr(status, (uint32_t)SF_ERANGE);
    }
    __syncthreads();

    const int64_t tb = lb * SPW;
    if constexpr (GTAB) {
        // the workgroup's steps are contiguous rows of out_increment holding
        // keys: decode them in place in chunks of WG entries, the last chunk
        // first.  A chunk reads its keys and the key before each (which lies
        // in the same chunk or the one below, not yet decoded), waits for
        // every thread's reads, then writes.
        const int64_t steps = T - tb < SPW ? T - tb : SPW;
        const int64_t n = steps * S;
        u64* g = reinterpret_cast<u64*>(inc) + tb * S;
        for (int64_t c = (n - 1) / WG; c >= 0; --c) {
            const int64_t i = c * WG + tid;
            const bool ok = i < n;
            u64 key = 0, kprev = 0;
            if (ok) {
                key = g[i];
                if (i % S != 0) kprev = g[i - 1];
            }
            __syncthreads();
            if (ok) {
                inc[tb * S + i] = (int64_t)(key >> kRankBits) - (int64_t)(kprev >> kRankBits);
                lead[tb * S + i] = (int32_t)(kRankMask - (key & kRankMask));
            }
        }
        return;
    }

    // decode F and the leader per (step, stage); rows of out are contiguous
    for (int i = tid; i < SPW * S; i += WG) {
        const int jj = i / S;
        const int s = i - jj * S;
        const int64_t tt = tb + jj;
        if (tt >= T) break;
        u64 key = 0, kprev = 0;
#pragma unroll
        for (int qd = 0; qd < SPS; ++qd) {
            key = umax64(key, tab[(jj * SPS + qd) * S + s]);
            if (s > 0) kprev = umax64(kprev, tab[(jj * SPS + qd) * S + s - 1]);
        }
        const int64_t F = (int64_t)(key >> kRankBits);
        const int64_t Fp = (int64_t)(kprev >> kRankBits);
        inc[tt * S + s] = F - Fp;
        lead[tt * S + s] = (int32_t)(kRankMask - (key & kRankMask));
    }
}

struct FrontierVariant {
    const void* fn;
    int K, G, WG;
    int per_cu;  // resident workgroups per CU to allow (0: no cap)
};

template <bool CHECK, int K, int G, int WG, bool GTAB = false, int D = 1, int VEC = 2>
FrontierVariant variant(int per_cu)
{
    return FrontierVariant{reinterpret_cast<const void*>(&k_frontier<VEC, K, G, WG, CHECK, GTAB, D>),
                           K, G, WG, per_cu};
}

// Launch shape by rank count, measured on MI355X over R = 8 .. 32768.
// Wide per-lane tiles (K = 32 ranks, about 250 VGPRs) and few resident
// workgroups per CU read HBM fastest where R fills them: fewer concurrent
// step streams, each with up to 32 KB of loads in flight per wave.  Lane slots
// past R cost no HBM traffic but hold a wave's issue slots, so ranks that
// leave half of such a tile empty take one closer to R (R = 700: 6.1 -> 7.0
// TB/s, 2049: 2.6 -> 7.0, 1030: 5.0 -> 5.8); near the full tile the wide ones
// stay ahead once the rows of all steps reach 32 MB (R = 1024: 7.07 against
// 6.80 TB/s; below, at 16 MB, 6.2 against 6.3, at 4 MB 3.0 against 4.8).
// Shapes with several rows in flight (D > 1) want stages to keep them there:
// from 1025 to 1792 ranks eight (1500 x 3000 steps, 4 stages 26 : 33 us, 6 36 :
// 41, 8 47 : 46), from 4097 to 5120 four (5120 x 3000, 2 stages 54 : 63, 6 129 :
// 124).
template <bool CHECK>
FrontierVariant pick_frontier(int R, int S, int64_t row_bytes)
{
    const bool many = row_bytes >= 32 << 20;
    if (R == 1) return variant<CHECK, 2, 4, 64, false, 1, 1>(0);
    if (R <= 8) return variant<CHECK, 2, 4, 64>(0);
    if (R <= 16) return variant<CHECK, 2, 8, 128>(0);
    if (R <= 32) return variant<CHECK, 4, 8, 128>(0);
    if (R <= 64) return variant<CHECK, 4, 16, 256>(6);
    if (R <= 128) return variant<CHECK, 8, 32, 256>(6);
    if (R <= 256) return variant<CHECK, 16, 32, 256>(4);
    if (R <= 512) return variant<CHECK, 4, 256, 256>(0);
    if (R <= 1024) return R > 896 && many ? variant<CHECK, 32, 64, 256>(6) : variant<CHECK, 4, 256, 256>(0);
    if (R <= 1792 && S >= 8) return variant<CHECK, 4, 512, 512, false, 4>(0);
    if (R <= 2048) return variant<CHECK, 8, 512, 512>(0);
    if (R <= 4096) return R > 3840 && many ? variant<CHECK, 32, 256, 256>(0) : variant<CHECK, 8, 512, 512>(0);
    if (R <= 5120 && S >= 4) return variant<CHECK, 8, 1024, 1024, false, 2>(0);
    return variant<CHECK, 32, 64, 64>(3);
}

// The deep shapes: the step over as many lanes as a workgroup takes, one
// tile up to 16384 ranks.
template <bool CHECK>
FrontierVariant pick_frontier_deep(int R)
{
    if (R <= 8) return variant<CHECK, 2, 4, 64, false, 8>(0);
    if (R <= 16) return variant<CHECK, 2, 8, 64, false, 8>(0);
    if (R <= 32) return variant<CHECK, 2, 16, 64, false, 8>(0);
    if (R <= 64) return variant<CHECK, 2, 32, 64, false, 8>(0);
    if (R <= 128) return variant<CHECK, 2, 64, 64, false, 8>(0);
    if (R <= 256) return variant<CHECK, 2, 128, 128, false, 8>(0);
    if (R <= 512) return variant<CHECK, 2, 256, 256, false, 8>(0);
    if (R <= 1024) return variant<CHECK, 2, 512, 512, false, 8>(0);
    if (R <= 2048) return variant<CHECK, 4, 512, 512, false, 4>(0);
    if (R <= 4096) return variant<CHECK, 4, 1024, 1024, false, 4>(0);
    if (R <= 8192) return variant<CHECK, 8, 1024, 1024, false, 2>(0);
    return variant<CHECK, 16, 1024, 1024>(0);
}

// Where the deep shapes are the faster ones (measured on MI355X).  Past 4096
// ranks the wide shape gives a step one wave, so below about 400 steps the
// chip idles (16384 ranks x 12 stages: 64 steps 87 -> 31 us, 256 steps 99 ->
// 63, 512 steps 115 -> 119).  Up to 4096 ranks the rows in flight are worth
// their registers while the stage rows of all steps are within 4 MB and there
// are enough stages to keep them in flight (130 x 100 stages: 1024 steps 66 ->
// 28 us, 4096 steps 88 -> 80); at few ranks that takes more of them, since a
// wave holds several steps' rows without it (2 ranks x 100000 steps: 9 stages
// 8.4 -> 11.5 us, 24 26.5 -> 28.3, 48 71.7 -> 58.8; 8 x 8192: 16 4.6 -> 5.1, 24
// 8.6 -> 7.1; 16 x 2048: 12 3.8 -> 4.3, 24 6.4 -> 6.0; 33 x 8192: 9 6.9 -> 7.8, 16
// 11.2 -> 10.1; 1024 x 8: 4.3 against 5.1); at 129 to 256 ranks they also win
// at few stages up to 2 MB (250 x 8: 256 steps 5.7 -> 4.7 us, 4096 steps 11.5 ->
// 14.5).
static bool deep_steps(int64_t T, int R, int S)
{
    const int64_t row = T * R * 8;
    if (R == 1) return false;
    if (R > 4096) return T < 400;
    if (R > 128 && R <= 256 && row <= 2 << 20) return true;
    const int few = R <= 8 ? 24 : R <= 16 ? 16 : R <= 32 ? 8 : R <= 64 ? 12 : R <= 128 ? 9 : R <= 256 ? 8 : R <= 512 ? 12 : 16;
    return S > few && row <= 4 << 20;
}

// Stage counts whose LDS table would exceed what a workgroup may hold: the
// shapes with one group of at most 64 lanes per step, with the table in the
// out_increment rows.
template <bool CHECK>
FrontierVariant pick_frontier_gtab(int R)
{
    if (R == 1) return variant<CHECK, 2, 4, 64, true, 1, 1>(0);
    if (R <= 8) return variant<CHECK, 2, 4, 64, true>(0);
    if (R <= 16) return variant<CHECK, 2, 8, 128, true>(0);
    if (R <= 32) return variant<CHECK, 4, 8, 128, true>(0);
    if (R <= 64) return variant<CHECK, 4, 16, 256, true>(6);
    if (R <= 128) return variant<CHECK, 8, 32, 256, true>(6);
    if (R <= 256) return variant<CHECK, 16, 32, 256, true>(4);
    return variant<CHECK, 32, 64, 64, true>(3);
}

// Largest S whose LDS table of partial maxima (16 slots of S keys in the
// widest-slot shapes) fits the 64 KB a workgroup is given.
constexpr int kFrontierLdsS = 512;

static int frontier_launch(const int64_t* durations, int64_t T, int32_t R, int32_t S,
                           int64_t* out_increment, int32_t* out_leader, uint32_t* status,
                           sf_stream_t stream)
{
    if (T < 0 || R < 1 || R > SF_MAX_R || S < 1) return SF_EINVAL;
    if (!fits(T, S, R, 8)) return SF_EINVAL;
    if (T == 0) return SF_OK;
    if (!durations || !out_increment || !out_leader) return SF_EINVAL;
    if (!aligned(durations, 8) || !aligned(out_increment, 8) || !aligned(out_leader, 4))
        return SF_EINVAL;
    const int64_t nd = T * S * (int64_t)R * 8, ni = T * S * 8, nl = T * S * 4;
    if (!disjoint(durations, nd, out_increment, ni) || !disjoint(durations, nd, out_leader, nl) ||
        !disjoint(out_increment, ni, out_leader, nl))
        return SF_EINVAL;
    if (status && (!aligned(status, 4) || !disjoint(status, 4, durations, nd) ||
                   !disjoint(status, 4, out_increment, ni) || !disjoint(status, 4, out_leader, nl)))
        return SF_EINVAL;

    const bool gtab = S > kFrontierLdsS;
    const bool deep = !gtab && deep_steps(T, R, S);
    const int64_t row = T * R * 8;
    const FrontierVariant v =
        gtab   ? (status ? pick_frontier_gtab<true>(R) : pick_frontier_gtab<false>(R))
        : deep ? (status ? pick_frontier_deep<true>(R) : pick_frontier_deep<false>(R))
               : (status ? pick_frontier<true>(R, S, row) : pick_frontier<false>(R, S, row));
    const int spw = v.WG / v.G;
    const int sub = v.G < 64 ? v.G : 64;
    const int64_t blocks = (T + spw - 1) / spw;
    if (blocks > INT32_MAX) return SF_EINVAL;
    const size_t lds = lds_request(gtab ? 0 : (size_t)(v.WG / sub) * S * sizeof(u64), v.per_cu);
    int Ri = R, Si = S;
    void* args[] = {(void*)&durations,     (void*)&T,          (void*)&Ri,    (void*)&Si,
                    (void*)&out_increment, (void*)&out_leader, (void*)&status};
    return launch(v.fn, dim3((unsigned)blocks), dim3(v.WG), args, lds, stream);
}

}  // namespace sfk

using namespace sfk;

SF_API int sf_frontier(const int64_t* durations, int64_t T, int32_t R, int32_t S,
                       int64_t* out_increment, int32_t* out_leader, sf_stream_t stream)
{
    return frontier_launch(durations, T, R, S, out_increment, out_leader, nullptr, stream);
}

SF_API int sf_frontier_checked(const int64_t* durations, int64_t T, int32_t R, int32_t S,
                               int64_t* out_increment, int32_t* out_leader, uint32_t* status,
                               sf_stream_t stream)
{
    if (!status) return SF_EINVAL;
    return frontier_launch(durations, T, R, S, out_increment, out_leader, status, stream);
}
