// gain.hip -- direct-exposure gain, Eq. (4).  Replacing stage s of every rank by
// b = min(d, btilde) changes the last frontier F[t,S] = max_r P[t,r,S] only
// through the rank totals: F^(s<-b)[t,S] = max_r (P[t,r,S] - delta[r,s]) with
// delta = max(0, d - btilde).  Step group layout as in k_frontier; each lane
// keeps its ranks' totals and the deltas of all stages in registers (the
// stage loop is unrolled to SMAX, rows past S re-read row 0 and are
// ignored), then every stage's candidate max and the plain max go through
// the idempotent DPP max, so lane slots past R (which re-read rank r0) need
// no masking.  When a step spans several rank tiles (and up to 16 stages)
// a lane keeps its running maxima over the tiles in registers and the group
// reduces once per step; otherwise the group reduces every tile.  Partial
// maxima of several groups meet in LDS.
//
// Long steps (use_near) take k_exposure_gain_near, which reads the durations
// once into rank totals and the baseline for the few ranks near the frontier
// only; a handful of ranks, or more stages than registers hold, take the
// two-pass k_exposure_gain_wide.

#include "sf_device.h"
#include "sf_host.h"
#include "sf_select.h"

#include <type_traits>

namespace sfk {

template <int K, int G, int WG, int SMAX, bool RUN>
__global__ __launch_bounds__(WG) void k_exposure_gain(
    const int64_t* __restrict__ d, const int64_t* __restrict__ btilde, int64_t T, int R, int S,
    int64_t window, int64_t* __restrict__ gain, int64_t* __restrict__ makespan)
{
    static_assert((K == 1 || K % 2 == 0) && (WG % G == 0 || G == WG), "shape");
    constexpr int VEC = K == 1 ? 1 : 2;
    constexpr int SUB = G < 64 ? G : 64;
    constexpr int SPW = WG / G;
    constexpr int SPS = G / SUB;
    constexpr int NLD = K / VEC;
    constexpr int RT = G * K;
    constexpr int NCOL = SMAX + 1;  // SMAX replaced-stage maxima, then F
    static_assert(!RUN || SMAX <= 16, "running maxima of up to 16 stages");

    __shared__ u64 tab[(WG / SUB) * NCOL];

    const int tid = threadIdx.x;
    const int gl = tid % G;
    const int slot = tid / SUB;
    const bool writer = (tid % SUB) == SUB - 1;
    const int64_t tb = xcd_block() * SPW;
    const int64_t t = tb + tid / G;

    if (t < T) {
        const int64_t* dt = d + t * (int64_t)S * R;
        const int64_t* bw = btilde + (t / window) * (int64_t)S * R;
        u64 run[RUN ? NCOL : 1];  // RUN: this lane's maxima so far ([SMAX] is F)
#pragma unroll
        for (int c = 0; c < (RUN ? NCOL : 1); ++c) run[c] = 0;
        for (int r0 = 0; r0 < R; r0 += RT) {
            int idx[NLD];
#pragma unroll
            for (int l = 0; l < NLD; ++l) {
                // R >= 2: with odd R the last pair overlaps the one before;
                // a pair past R re-reads the tile's first ranks (the last
                // pair instead ran 20% slower at 64 ranks)
                const int r = r0 + (l * G + gl) * VEC;
                idx[l] = min(r < R ? r : r0, R - VEC);
            }
            int64_t tot[K];
            int64_t dl[K][SMAX];
#pragma unroll
            for (int k = 0; k < K; ++k) tot[k] = 0;
            // the tile's loads all in flight before any is used: left to the
            // compiler, it waits for the first ones in between to save
            // registers (64 ranks x 6 stages: 237 us against 187 per 0.8 GB).
            // With running maxima (a step's tiles in series) the durations
            // come first, then the baseline: both at once took 108 us against
            // 88 for 32768 ranks x 6 x 100 and 237 against 208 for 45000 x 12 x
            // 100
            constexpr bool TWO = RUN && SMAX >= 6;
            typedef typename std::conditional<VEC == 2, v2i64_a8, int64_t>::type L;
            L x[SMAX][NLD], y[SMAX][NLD];
            auto at = [](const L& v, int e) {
                if constexpr (VEC == 2) return v[e];
                else return v;
            };
#pragma unroll
            for (int s = 0; s < SMAX; ++s) {
                const int sr = s < S ? s : 0;
#pragma unroll
                for (int l = 0; l < NLD; ++l) {
                    x[s][l] = __builtin_nontemporal_load(reinterpret_cast<const L*>(dt + (int64_t)sr * R + idx[l]));
                    if (!TWO) y[s][l] = *reinterpret_cast<const L*>(bw + (int64_t)sr * R + idx[l]);
                }
            }
            if (SMAX <= 8 && !RUN) __builtin_amdgcn_sched_barrier(0);
            if (TWO) {
#pragma unroll
                for (int l = 0; l < NLD; ++l)
#pragma unroll
                    for (int s = 0; s < SMAX; ++s)
#pragma unroll
                        for (int e = 0; e < VEC; ++e)
                            if (s < S) tot[l * VEC + e] += at(x[s][l], e);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < SMAX; ++s) {
                    const int sr = s < S ? s : 0;
#pragma unroll
                    for (int l = 0; l < NLD; ++l) y[s][l] = *reinterpret_cast<const L*>(bw + (int64_t)sr * R + idx[l]);
                }
            }
#pragma unroll
            for (int s = 0; s < SMAX; ++s) {
#pragma unroll
                for (int l = 0; l < NLD; ++l) {
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        const int64_t red = at(x[s][l], e) - at(y[s][l], e);
                        dl[l * VEC + e][s] = red > 0 ? red : 0;
                        if (!TWO && s < S) tot[l * VEC + e] += at(x[s][l], e);
                    }
                }
            }
            u64 fmax = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) fmax = umax64(fmax, (u64)tot[k]);
            if constexpr (RUN) {
                run[SMAX] = umax64(run[SMAX], fmax);
            } else {
                fmax = group_max<SUB>(fmax);
                if (writer) {
                    u64* p = &tab[slot * NCOL + SMAX];
                    *p = (r0 == 0) ? fmax : umax64(*p, fmax);
                }
            }
#pragma unroll
            for (int s = 0; s < SMAX; ++s) {
                if (s < S) {
                    u64 m = 0;
#pragma unroll
                    for (int k = 0; k < K; ++k) m = umax64(m, (u64)(tot[k] - dl[k][s]));
                    if constexpr (RUN) {
                        run[s] = umax64(run[s], m);
                    } else {
                        m = group_max<SUB>(m);
                        if (writer) {
                            u64* p = &tab[slot * NCOL + s];
                            *p = (r0 == 0) ? m : umax64(*p, m);
                        }
                    }
                }
            }
        }
        if constexpr (RUN) {
            // one reduction per step over the group
#pragma unroll
            for (int c = 0; c < (RUN ? NCOL : 1); ++c) {
                if (c < S || c == SMAX) {
                    const u64 m = group_max<SUB>(run[c]);
                    if (writer) tab[slot * NCOL + c] = m;
                }
            }
        }
    }
    __syncthreads();

    for (int i = tid; i < SPW * S; i += WG) {
        const int jj = i / S;
        const int s = i - jj * S;
        const int64_t tt = tb + jj;
        if (tt >= T) break;
        u64 F = 0, Fr = 0;
#pragma unroll
        for (int qd = 0; qd < SPS; ++qd) {
            F = umax64(F, tab[(jj * SPS + qd) * NCOL + SMAX]);
            Fr = umax64(Fr, tab[(jj * SPS + qd) * NCOL + s]);
        }
        gain[tt * S + s] = (int64_t)F - (int64_t)Fr;
        if (s == 0) makespan[tt] = (int64_t)F;
    }
}

// Few ranks and many stages, or more of either than the other kernels take:
// G lanes own a step (two ranks per lane and tile), and for each rank tile
// the group makes two passes over the stages, the rank totals first and then
// every stage's candidate max; the second pass finds a small step's rows in
// the caches.  The group's last lane keeps the maxima over tiles in the
// step's own out_gain row (the replaced-stage maxima) and out_makespan entry
// (F), and after a barrier the workgroup turns the rows into gains.  Rank
// pairs past R re-read the last pair, which cannot change a max.
template <int VEC, int G, int WG>
__global__ __launch_bounds__(WG) void k_exposure_gain_wide(
    const int64_t* __restrict__ d, const int64_t* __restrict__ btilde, int64_t T, int R, int S,
    int64_t window, int64_t* __restrict__ gain, int64_t* __restrict__ makespan)
{
    static_assert(G <= 64 && WG % G == 0, "one writer lane per step");
    constexpr int SPW = WG / G;
    constexpr int RT = G * VEC;
    constexpr int U = 8;  // stage rows in flight
    const int tid = threadIdx.x;
    const int gl = tid % G;
    const bool writer = gl == G - 1;
    const int64_t tb = xcd_block() * SPW;
    const int64_t t = tb + tid / G;
    if (t < T) {
        const int64_t* dt = d + t * (int64_t)S * R;
        const int64_t* bw = btilde + (t / window) * (int64_t)S * R;
        u64* fr = reinterpret_cast<u64*>(gain) + t * S;  // replaced-stage maxima so far
        u64* fm = reinterpret_cast<u64*>(makespan) + t;  // F so far
        for (int r0 = 0; r0 < R; r0 += RT) {
            const int r = min(r0 + gl * VEC, R - VEC);  // VEC <= R
            auto load = [&](const int64_t* row, int64_t* x) {
                if (VEC == 2) {
                    const v2i64_a8 a = *reinterpret_cast<const v2i64_a8*>(row + r);
                    x[0] = a.x;
                    x[VEC - 1] = a.y;
                } else {
                    x[0] = row[r];
                }
            };
            int64_t tot[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) tot[e] = 0;
#pragma unroll U
            for (int s = 0; s < S; ++s) {
                int64_t x[VEC];
                load(dt + (int64_t)s * R, x);
#pragma unroll
                for (int e = 0; e < VEC; ++e) tot[e] += x[e];
            }
            u64 f = 0;
#pragma unroll
            for (int e = 0; e < VEC; ++e) f = umax64(f, (u64)tot[e]);
            f = group_max<G>(f);
            if (writer) *fm = r0 == 0 ? f : umax64(*fm, f);
            for (int s0 = 0; s0 < S; s0 += U) {
                int64_t x[U][VEC], y[U][VEC];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int s = min(s0 + u, S - 1);
                    load(dt + (int64_t)s * R, x[u]);
                    load(bw + (int64_t)s * R, y[u]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    u64 m = 0;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        const int64_t red = x[u][e] - y[u][e];
                        m = umax64(m, (u64)(tot[e] - (red > 0 ? red : 0)));
                    }
                    m = group_max<G>(m);
                    if (writer && s0 + u < S) fr[s0 + u] = r0 == 0 ? m : umax64(fr[s0 + u], m);
                }
            }
        }
    }
    __syncthreads();  // the writer lanes' maxima are visible to the workgroup
    for (int i = tid; i < SPW * S; i += WG) {
        const int jj = i / S;
        const int64_t tt = tb + jj;
        if (tt >= T) break;
        const int64_t idx = tt * S + (i - jj * S);
        gain[idx] = makespan[tt] - gain[idx];
    }
}

// The ranks near the frontier only.  Replacing stage s lowers a rank's total
// by delta >= 0, so a rank r can raise the stage's maximum above a value
// already found only if its total P_r exceeds that value.  One workgroup per
// step adds the durations into rank totals in registers (one pass over the
// step, KP rank pairs per lane; with NS > 1 the workgroup's slices take
// different stages and add up through LDS), then
//  1. takes F and a rank that attains it, and reads that rank's durations and
//     baseline: F - delta is a first candidate maximum of every stage, L the
//     smallest of them;
//  2. reads durations and baseline of the ranks with P_r > L (a handful as a
//     rule), for the stages whose candidate they can still raise, adjacent
//     lanes on adjacent ranks of a stage.
// When half of the ranks or more than kNearCap lie above L (some stage's
// replacement drops the top rank far, or a collective has made the totals
// equal), the waves' own top ranks and the first kNearFirst of the list are
// tried first: that raises L where it was the top rank alone, and among equal
// totals a few ranks settle nearly every stage, where reading all of them cost
// more than the kernel saves (512 ranks x 8 x 4000 steps synchronised before
// the last stages 39 -> 31 us, 29 without the kernel; 1024 x 24 x 1000 with equal
// totals 59 -> 34, 52).  Then the stage of the smallest candidate is resolved
// over all ranks from its two rows, which leaves L to the others, up to
// kNearRows times; then all stages are.  The result is the same maximum in
// each case.  Pairs past R read 0 (they lie past the stage row's buffer
// resource), and a total of 0 never exceeds L >= 0; with odd R the last pair
// overlaps the one before.
//
// Bound: HBM, the totals pass.  Measured on MI355X: 1024 ranks x 132 stages x
// 1000 steps 1264 -> 183 us, 4096 x 12 x 5000 315 -> 295 us against the
// kernels that took these shapes before; 12000 x 12 x 2777 535 -> 489 us and
// 16384 x 12 x 2034 492 -> 483 us against a radix search over the totals for
// a bound with at least 32 ranks above it (which also needed a barrier per
// stage row to run well).  The shape past 16384 ranks holds 32 totals per lane
// and spills 56 VGPRs around the list's construction (two loads in flight
// instead of four spill the same and run 5-10% slower).
constexpr int kNearCap = 512;
constexpr int kNearFirst = 32;  // at most kNearCap: entries of the list
constexpr int kNearMaxR = 32768;
constexpr int64_t kNearFewSteps = 512;
constexpr int kNearMaxS = 4096;  // stages whose candidates fit in LDS (32 KB)
constexpr int kNearSBits = 12;   // a candidate (below 2^47) and its stage in one key
constexpr int kNearRows = 3;
constexpr u64 kNearDone = 1ull << 63;  // a candidate that is final

template <int WG, int KP, int NS>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(4))) void k_exposure_gain_near(
    const int64_t* __restrict__ d, const int64_t* __restrict__ btilde, int64_t T, int R, int S,
    int64_t window, int64_t* __restrict__ gain, int64_t* __restrict__ makespan)
{
    constexpr int NW = WG / 64;
    constexpr int GW = WG / NS;  // threads per slice (whole waves)
    constexpr int LC = KP < 8 ? KP : (WG == 1024 ? 4 : 8);  // loads of a stage in flight at once
    constexpr int U = KP < 8 ? 8 / KP : 1;                  // stages in flight at once
    static_assert(GW % 64 == 0 && KP % LC == 0, "shape");
    extern __shared__ u64 cand[];  // [S] candidate maxima
    __shared__ u64 part[NS > 1 ? GW * KP * 2 : 1];
    __shared__ u64 w_tot[NW], red[NW];
    __shared__ int w_rank[NW];
    __shared__ int q_rank[kNearCap];
    __shared__ u64 q_tot[kNearCap];
    __shared__ uint32_t q_n;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slice = NS > 1 ? __builtin_amdgcn_readfirstlane(tid / GW) : 0;
    const int tl = NS > 1 ? tid % GW : tid;
    const int64_t t = xcd_block();
    if (t >= T) return;  // uniform (the grid is T)
    const int64_t* dt = d + t * (int64_t)S * R;
    const int64_t* bw = btilde + (t / window) * (int64_t)S * R;
    auto rank0 = [&](int l) {  // first rank of the lane's pair l (R >= 2)
        const int r = (l * GW + tl) * 2;
        return r == R - 1 ? r - 1 : r;
    };

    for (int s = tid; s < S; s += WG) cand[s] = 0;
    if (NS > 1) {
        for (int i = tid; i < GW * KP * 2; i += WG) part[i] = 0;
    }
    if (tid == 0) q_n = 0;
    u64 tot[KP][2];
#pragma unroll
    for (int l = 0; l < KP; ++l) tot[l][0] = tot[l][1] = 0;
    for (int s0 = slice * U; s0 < S; s0 += NS * U) {
#pragma unroll
        for (int l0 = 0; l0 < KP; l0 += LC) {
            v2i64 x[U][LC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // a stage past S reads zeros
                const auto rs = buffer_rsrc(dt + (int64_t)(s0 + u) * R, s0 + u < S ? (uint32_t)R * 8u : 0u);
#pragma unroll
                for (int l = 0; l < LC; ++l) x[u][l] = buffer_load16_nt(rs, (uint32_t)rank0(l0 + l) * 8u, 0u);
            }
            __builtin_amdgcn_sched_barrier(0);  // the loads all in flight first
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int l = 0; l < LC; ++l) {
                    tot[l0 + l][0] += (u64)x[u][l].x;
                    tot[l0 + l][1] += (u64)x[u][l].y;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (NS > 1) {
        __syncthreads();
#pragma unroll
        for (int l = 0; l < KP; ++l) {
            atomicAdd(&part[(l * GW + tl) * 2], tot[l][0]);
            atomicAdd(&part[(l * GW + tl) * 2 + 1], tot[l][1]);
        }
        __syncthreads();
#pragma unroll
        for (int l = 0; l < KP; ++l) {
            tot[l][0] = slice == 0 ? part[(l * GW + tl) * 2] : 0;
            tot[l][1] = slice == 0 ? part[(l * GW + tl) * 2 + 1] : 0;
        }
    }
    // every wave's largest total and a rank that has it
    {
        u64 m = 0;
#pragma unroll
        for (int l = 0; l < KP; ++l) m = umax64(m, umax64(tot[l][0], tot[l][1]));
        const u64 wm = lane_value(group_max<64>(m), 63);
        int rk = -1;
#pragma unroll
        for (int l = 0; l < KP; ++l) {
            if (tot[l][0] == wm) rk = rank0(l);
            if (tot[l][1] == wm) rk = rank0(l) + 1;
        }
        const u64 has = __ballot(rk >= 0);
        const int src = __builtin_amdgcn_readlane(rk, (int)__builtin_ctzll(has));
        if (lane == 0) {
            w_tot[wave] = wm;
            w_rank[wave] = wm != 0 ? src : -1;  // only a rank below R has a total above 0
        }
    }
    __syncthreads();
    u64 F = 0;
    int top = -1;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        if (w_tot[i] > F) {
            F = w_tot[i];
            top = w_rank[i];
        }
    }
    if (F == 0) {  // uniform: every duration is 0
        for (int s = tid; s < S; s += WG) gain[t * S + s] = 0;
        if (tid == 0) makespan[t] = 0;
        return;
    }
    // candidates of rank `top`, and the smallest of them
    auto low_key = [](u64 c, int s) { return (c & kNearDone) ? ~0ull : (c << kNearSBits) | (u64)s; };
    u64 low = ~0ull;
    for (int s = tid; s < S; s += WG) {
        const int64_t e = dt[(int64_t)s * R + top] - bw[(int64_t)s * R + top];
        const u64 c = F - (u64)(e > 0 ? e : 0);  // 0 <= b: max(e, 0) <= d <= F
        cand[s] = c;
        low = umin64(low, low_key(c, s));
    }
    // fold the (rank, stage) pairs of a list of ranks: four per thread in flight
    auto fold = [&](const int* ranks, const u64* tots, uint32_t n) {
        const uint32_t np = n * (uint32_t)S;
        for (uint32_t i0 = tid; i0 < np; i0 += 4 * WG) {
            int64_t x[4], y[4];
            u64 tq[4];
            int sj[4];
            bool need[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t i = i0 + (uint32_t)(j * WG);
                const uint32_t ii = i < np ? i : 0u;
                const uint32_t sq = ii / n, q = ii - sq * n;
                const int s = (int)sq;
                tq[j] = tots[q];
                sj[j] = s;
                need[j] = i < np && tq[j] > cand[s];  // cand only grows: a stale read is safe
                x[j] = 0;
                y[j] = 0;
                if (need[j]) {
                    const int r = ranks[q];  // a total above a candidate: a rank below R
                    x[j] = dt[(int64_t)s * R + r];
                    y[j] = bw[(int64_t)s * R + r];
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (need[j]) {
                    const int64_t e = x[j] - y[j];
                    atomicMax(&cand[sj[j]], tq[j] - (u64)(e > 0 ? e : 0));
                }
            }
        }
    };
    // stage s over all ranks, by the waves that hold totals
    auto row = [&](int s) {
        const auto rd = buffer_rsrc(dt + (int64_t)s * R, (uint32_t)R * 8u);
        const auto rb = buffer_rsrc(bw + (int64_t)s * R, (uint32_t)R * 8u);
        u64 m = 0;
        constexpr int RC = KP < 4 ? KP : (KP == 16 ? 2 : 4);  // loads of each row in flight
#pragma unroll
        for (int l0 = 0; l0 < KP; l0 += RC) {
            v2i64 x[RC], y[RC];
#pragma unroll
            for (int l = 0; l < RC; ++l) {
                x[l] = buffer_load16_nt(rd, (uint32_t)rank0(l0 + l) * 8u, 0u);
                y[l] = buffer_load16_nt(rb, (uint32_t)rank0(l0 + l) * 8u, 0u);
            }
#pragma unroll
            for (int l = 0; l < RC; ++l) {
                const u64* p = NS > 1 ? &part[((l0 + l) * GW + tl) * 2] : tot[l0 + l];
                const int64_t e0 = x[l].x - y[l].x, e1 = x[l].y - y[l].y;
                m = umax64(m, p[0] - (u64)(e0 > 0 ? e0 : 0));
                m = umax64(m, p[1] - (u64)(e1 > 0 ? e1 : 0));
            }
        }
        m = group_max<64>(m);
        if (lane == 63) atomicMax(&cand[s], m);
    };
    for (int round = 0;; ++round) {
        // L, the smallest candidate that is not final, and its stage
        low = ~lane_value(group_max<64>(~low), 63);
        if (lane == 0) red[wave] = low;
        __syncthreads();
        u64 key = ~0ull;
#pragma unroll
        for (int i = 0; i < NW; ++i) key = umin64(key, red[i]);
        const u64 L = key >> kNearSBits;
        // Q, the ranks above L (rank `top` is done): a wave scan of the
        // per-lane counts, one atomic per wave
        uint32_t cm = 0;
#pragma unroll
        for (int l = 0; l < KP; ++l) {
#pragma unroll
            for (int e = 0; e < 2; ++e)
                cm |= (tot[l][e] > L && rank0(l) + e != top) ? 1u << (2 * l + e) : 0u;
        }
        if (__ballot(cm != 0) != 0) {
            const uint32_t nc = (uint32_t)__popc(cm);
            const uint32_t incl = wave_scan_incl(nc);
            uint32_t wb = 0;
            if (lane == 63) wb = atomicAdd(&q_n, incl);
            uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)wb, 63) + incl - nc;
#pragma unroll
            for (int k = 0; k < 2 * KP; ++k) {
                if ((cm >> k) & 1u) {
                    if (pos < (uint32_t)kNearCap) {
                        q_rank[pos] = rank0(k / 2) + (k & 1);
                        q_tot[pos] = tot[k / 2][k & 1];
                    }
                    ++pos;
                }
            }
        }
        __syncthreads();
        const uint32_t nq = q_n;
        // (a workgroup of 1024 for so few ranks has few steps, and a round
        // costs it more than the reads)
        const int at_once = round == 0 && WG < 1024 && R < 2 * kNearCap ? max(kNearFirst, R / 2) : kNearCap;
        if (nq <= (uint32_t)at_once) {
            fold(q_rank, q_tot, nq);
            break;
        }
        const int s_low = __builtin_amdgcn_readfirstlane((int)(key & ((1u << kNearSBits) - 1u)));
        if (round == 0) {
            fold(w_rank, w_tot, NW);
            fold(q_rank, q_tot, kNearFirst);
        } else if (round <= kNearRows) {
            if (slice == 0) row(s_low);
        } else {
            for (int s = slice; s < S; s += NS) {
                if (!(cand[s] & kNearDone)) row(s);  // uniform over the wave
            }
            break;
        }
        __syncthreads();  // every thread has read q_n, every candidate is in
        if (tid == 0) {
            q_n = 0;
            if (round > 0) cand[s_low] |= kNearDone;
        }
        __syncthreads();
        low = ~0ull;
        for (int s = tid; s < S; s += WG) low = umin64(low, low_key(cand[s], s));
    }
    __syncthreads();
    for (int s = tid; s < S; s += WG) gain[t * S + s] = (int64_t)(F - (cand[s] & ~kNearDone));
    if (tid == 0) makespan[t] = (int64_t)F;
}

struct GainVariant {
    const void* fn;
    int G, WG;
};

template <int K, int G, int WG, int SMAX, bool RUN = false>
GainVariant gain_variant()
{
    return GainVariant{reinterpret_cast<const void*>(&k_exposure_gain<K, G, WG, SMAX, RUN>), G, WG};
}

// Two ranks per lane keep the deltas in registers; G covers R in one tile up
// to 512 ranks, larger R loops over tiles.  Chosen by measurement on MI355X
// (wider K held more registers and ran up to 2x slower).
template <int SMAX>
GainVariant pick_gain_g(int R)
{
    if (R <= 32) return gain_variant<2, 16, 64, SMAX>();
    if constexpr (SMAX <= 16) {
        if (R <= 128) return gain_variant<2, 64, 256, SMAX>();
        // four or more tiles per step: running maxima (measured: 1-2% faster
        // at 4096 and 16384 ranks; at one or two tiles they only cost registers)
        if (R > 3 * 512) return gain_variant<2, 256, 256, SMAX, true>();
    }
    return gain_variant<2, 256, 256, SMAX>();
}

// SMAX close above S: every unrolled stage past S still issues its two loads
// and holds its deltas, so 12 stages under SMAX = 16 ran 14-18% slower than
// under SMAX = 12 (and 6 under 8, 9% slower) on MI355X.
constexpr int kGainRegS = 24;  // stages whose deltas k_exposure_gain keeps in registers
constexpr int kGainMaxS = 64;  // the same where k_exposure_gain_near does not reach

GainVariant pick_gain(int R, int S)
{
    if (S <= 4) return pick_gain_g<4>(R);
    if (S <= 6) return pick_gain_g<6>(R);
    if (S <= 8) return pick_gain_g<8>(R);
    if (S <= 12) return pick_gain_g<12>(R);
    if (S <= 16) return pick_gain_g<16>(R);
    if (S <= 24) return pick_gain_g<24>(R);
    if (S <= 32) return gain_variant<2, 256, 256, 32>();
    return gain_variant<1, 256, 256, 64>();  // S <= kGainMaxS
}

template <int WG, int KP, int NS = 1>
GainVariant near_variant()
{
    return GainVariant{reinterpret_cast<const void*>(&k_exposure_gain_near<WG, KP, NS>), WG, WG};
}

template <int VEC, int G>
GainVariant wide_variant()
{
    return GainVariant{reinterpret_cast<const void*>(&k_exposure_gain_wide<VEC, G, 256>), G, 256};
}

GainVariant pick_wide(int R)
{
    if (R == 1) return wide_variant<1, 4>();
    if (R <= 8) return wide_variant<2, 4>();
    if (R <= 16) return wide_variant<2, 8>();
    if (R <= 32) return wide_variant<2, 16>();
    if (R <= 64) return wide_variant<2, 32>();
    return wide_variant<2, 64>();
}

// 8 loads in flight per lane: KP pairs of 8 / KP stages (two chunks of four
// in the 1024-thread shapes).  From 4097 to 8192 ranks 512 threads x 8 pairs
// beat 1024 x 4 by 5-40%.  With few steps the
// stages of one are split over the waves of a wide workgroup, since there are
// not enough workgroups to fill the chip: up to 1024 ranks while every step has
// a CU to itself (384 ranks x 8: 256 steps 10.4 us, 300 12.0 against 9.1).
GainVariant pick_near(int64_t T, int R)
{
    if (T <= (R <= 1024 ? 256 : kNearFewSteps)) {
        if (R <= 256) return near_variant<1024, 1, 8>();
        if (R <= 512) return near_variant<1024, 1, 4>();
        if (R <= 1024) return near_variant<1024, 1, 2>();
        if (R <= 2048) return near_variant<1024, 1>();
        if (R <= 4096) return near_variant<1024, 2>();
    }
    if (R <= 256) return near_variant<256, 1, 2>();
    if (R <= 512) return near_variant<256, 1>();
    if (R <= 1024) return near_variant<256, 2>();
    if (R <= 2048) return near_variant<256, 4>();
    if (R <= 4096) return near_variant<256, 8>();
    if (R <= 8192) return near_variant<512, 8>();
    if (R <= 16384) return near_variant<1024, 8>();
    return near_variant<1024, 16>();  // R <= kNearMaxR
}

// Where the near-frontier pass wins (measured on MI355X over 0.8 GB, us, near
// against the best other kernel).  It wants steps long enough to cover its
// few dependent reads, and many stages: with 6 or fewer, one stage is a large
// part of the step and its replacement often takes the row passes (16384
// ranks: 175 against 145; with 12 stages 130 against 149).
//   9 stages and more: past 128 ranks (12 stages: 200 ranks 141 : 237, 1024
//     130 : 147, 4096 127 : 136; 128 ranks 191 : 130); past 16384 ranks, one
//     workgroup per CU, 13 stages, or 9 up to 256 steps (24576 x 12: 100 steps
//     66 : 121, 600 272 : 280, synchronised 347 : 280);
//   7 and 8: from 129 to 2048 ranks, to 4096 up to 512 steps (8 stages: 200
//     ranks 183 : 237, 2048 x 4000 90 : 91, 4096 x 1000 53 : 50, synchronised 61 : 50);
//   17 and more: wherever a step holds 1600 samples (20 stages x 96 ranks
//     190 : 229, 32 x 64 211 : 245, 32 x 48 259 : 245, 132 x 1024 153 : 640);
//   few steps past 4096 ranks, where the other kernels give a step 256 threads:
//     up to 256 steps with 5 stages, or past 8192 ranks (16384 x 5: one step 15 :
//     36, 100 33 : 48, 400 72 : 70; 8192 x 4 x 64 19 : 21); past 16384 ranks up to 8
//     steps, or 64 with 7 stages (32768 x 8: 8 steps 53 : 102, 64 58 : 107, 150 82 :
//     112, synchronised 105 : 112; x 5: 8 56 : 74, 64 67 : 82, synchronised 150 steps
//     83 : 85).
bool use_near(int64_t T, int R, int S)
{
    if (R > kNearMaxR || S > kNearMaxS || T > INT32_MAX) return false;
    if (S >= 17 && R >= 48 && R * S >= 1600) return true;
    if (R > 16384) return S >= 13 || T <= (S >= 9 ? 256 : S >= 7 ? 64 : 8);
    if (R > 4096 && T <= 256 && (S >= 5 || R > 8192 || T <= 8)) return true;
    return R > 128 && (S >= 9 || (S >= 7 && R <= (T <= kNearFewSteps ? 4096 : 2048)));
}

// Where the two-pass kernel beats the one with the deltas in registers: a
// handful of ranks (8 ranks x 6 stages 66 : 88, x 12 157 : 166, x 24 322 :
// 442), 13 and more stages from 33 to 64 ranks (48 x 16 227 : 287), more
// stages than the registers hold, and 17 to 24 of them where its lanes would
// idle (16 ranks x 20 302 : 324, 48 x 24 236 : 382; 32 x 20 261 : 200).  Past
// kNearMaxR ranks the registers hold up to 64 stages (45000 ranks x 100 steps: 25
// stages 700 us against 5000, 64 x 32 3200 against 12000).
bool use_wide(int R, int S)
{
    if (R <= 8 || S > (R > kNearMaxR ? kGainMaxS : kGainRegS)) return true;
    if (R > kNearMaxR) return false;
    if (S >= 17) return R <= 16 || (R > 32 && R <= 128);
    return S >= 13 && R > 32 && R <= 64;
}

}  // namespace sfk

using namespace sfk;

SF_API int sf_exposure_gain(const int64_t* durations, const int64_t* baseline, int64_t T,
                            int32_t R, int32_t S, int64_t window, int64_t* out_gain,
                            int64_t* out_makespan, int64_t* out_window_gain,
                            int64_t* out_window_makespan, sf_stream_t stream)
{
    if (T < 0 || R < 1 || R > SF_MAX_R || S < 1 || window < 1) return SF_EINVAL;
    if (!fits(T, S, R, 8)) return SF_EINVAL;
    if (T == 0) return SF_OK;
    const int64_t W = sf_num_windows(T, window);
    if (!fits(W, S, R, 8)) return SF_EINVAL;
    const void* bufs[6] = {durations, baseline, out_gain, out_makespan, out_window_gain,
                           out_window_makespan};
    const int64_t sizes[6] = {T * S * (int64_t)R * 8, W * S * (int64_t)R * 8, T * S * 8, T * 8,
                              W * S * 8, W * 8};
    for (int a = 0; a < 6; ++a)
        if (!bufs[a] || !aligned(bufs[a], 8)) return SF_EINVAL;
    for (int a = 0; a < 6; ++a)
        for (int b = (a < 2 ? 2 : a + 1); b < 6; ++b)
            if (!disjoint(bufs[a], sizes[a], bufs[b], sizes[b])) return SF_EINVAL;

    int Ri = R, Si = S;
    void* args[] = {(void*)&durations, (void*)&baseline, (void*)&T, (void*)&Ri, (void*)&Si,
                    (void*)&window, (void*)&out_gain, (void*)&out_makespan};
    GainVariant v;
    size_t lds = 0;
    if (use_near(T, R, S)) {
        v = pick_near(T, R);
        lds = (size_t)S * sizeof(u64);
    } else if (use_wide(R, S)) {
        v = pick_wide(R);
    } else {
        v = pick_gain(R, S);
    }
    const int spw = v.WG / v.G;
    const int64_t blocks = (T + spw - 1) / spw;
    if (blocks > INT32_MAX) return SF_EINVAL;
    const int rc = launch(v.fn, dim3((unsigned)blocks), dim3(v.WG), args, lds, stream);
    if (rc != SF_OK) return rc;
    return launch_window_sum(out_gain, T, S, window, W, out_window_gain, out_makespan,
                             out_window_makespan, stream);
}
