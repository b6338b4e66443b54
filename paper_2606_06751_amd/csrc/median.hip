// median.hip -- per-rank window median, a candidate baseline btilde of Eq. (4)
// (Sec. 4): med[w][s][r] = the lower median over the n steps t of window w of
// d[t][s][r] (the value of rank floor((n-1)/2) in ascending order).
//
// The layout [T][S][R] is [T][C] with C = S * R columns, and a window's
// medians are column medians: stages and ranks play no part.  A tile is
// (window, COLS adjacent columns).  Persistent workgroups read the next
// tile's row pieces into registers (16-byte loads, through a buffer resource
// that ends at the window's last row) while they resolve the current one,
// which lies in LDS as 32-bit words, row by row.
//
// PARTS adjacent lanes share a column and hold 32 W of its values each.  The
// select works on bit planes: 32 values' 16 bits from the tile's top set bit
// down become 16 words, one bit of every value each (bit_planes16), and one
// bit is resolved at a time from the top: of the candidates (a bit mask per
// 32 values) those with a 0 there are counted with one popcount per lane and
// summed over the column's lanes by DPP, and the half that holds the target
// stays.  A bit of 32 values costs about 12 VALU instructions instead of 2
// per value.  Once every column of the wave has one candidate left its value
// is read back from LDS; else the next 16 bits follow.  No guess and no
// histogram: the time does not depend on the values' distribution, apart
// from the second round.  Bound: the loads (without the select the kernel
// takes 94-97% of its time up to 512 steps).  Measured on MI355X, 4096 ranks
// x 12 stages x 5000 steps: windows of 250 steps 535 -> 350 us, of 100 steps
// 1073 -> 340 us against the former per-column radix select with LDS
// histograms; 256 x 6 x 40000, windows of 2000: 2540 -> 110 us (the former
// kernel streamed each column there).
//
// A tile with a value of 2^32 or above is resolved twice: by the high halves,
// while the values are still in registers, then by the low halves of the
// candidates left.  Nothing overlaps its first select, but the time still does
// not depend on how many columns are such ones: with one stage of 6 s, 4096 x 12
// x 1000, windows of 250 79 us (73 without; 228 for the former kernel, 450 where
// a saturated column was streamed from global memory by its wave), 58 x 6 x 2000,
// windows of 50 10 (11, 45).
//
// Windows longer than the tile rows, and a single column, are streamed from
// global memory column by column (wave_select_stream).

#include "sf_device.h"
#include "sf_host.h"
#include "sf_select.h"

#include <type_traits>

namespace sfk {

// orders this wave's LDS accesses before the ones that follow (a wave's LDS
// operations complete in issue order; this keeps the compiler from moving
// them across)
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// OR over the 64 lanes, in every lane
__device__ __forceinline__ uint32_t wave_or32(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, true);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

__device__ __forceinline__ u64 wave_or64(u64 v)
{
    return ((u64)wave_or32((uint32_t)(v >> 32)) << 32) | wave_or32((uint32_t)v);
}

template <typename V>
__device__ __forceinline__ bool sel_match_t(V u, int hi, V prefix)
{
    return hi >= (int)(8 * sizeof(V)) || (u >> hi) == prefix;
}

template <typename V>
__device__ __forceinline__ int sel_first_lo_t(V range)
{
    const int nbits = (int)(8 * sizeof(V)) - (sizeof(V) == 8 ? __builtin_clzll((u64)range)
                                                              : __builtin_clz((uint32_t)range));
    return nbits > 8 ? nbits - 8 : 0;
}

// Exact lower median of the n 64-bit values get(0..n-1), read pass by pass
// (any n): the OR, then one histogram pass per digit, then a search for the
// one value left.  h: the wave's histogram (zero on entry and on return).
template <typename Get>
__device__ u64 wave_select_stream(Get get, int64_t n, uint32_t* h, int lane)
{
    u64 vor = 0;
    for (int64_t i = lane; i < n; i += 64) vor |= get(i);
    vor = wave_or64(vor);
    if (vor == 0) return 0;
    int lo = sel_first_lo_t(vor), hi = lo + 8;
    u64 prefix = 0;
    uint32_t kk = (uint32_t)((n - 1) / 2);
    for (;;) {
        for (int64_t i = lane; i < n; i += 64) {
            const u64 x = get(i);
            if (sel_match_t(x, hi, prefix)) atomicAdd(&h[(uint32_t)((x >> lo) & ((1u << (hi - lo)) - 1u))], 1u);
        }
        wave_lds_fence();
        uint32_t digit, count;
        sel_scan_wave(h, lane, kk, digit, count);
        sel_clear_lane_bins(h, lane);
        wave_lds_fence();
        prefix = (prefix << (hi - lo)) | (u64)digit;
        hi = lo;
        if (hi == 0) return prefix;
        lo = lo > 8 ? lo - 8 : 0;
        if (count == 1) {
            u64 x = 0;
            bool has = false;
            for (int64_t i = lane; i < n; i += 64) {
                const u64 y = get(i);
                if (sel_match_t(y, hi, prefix)) {
                    x = y;
                    has = true;
                }
            }
            const u64 hm = __ballot(has);
            return lane_value(x, hm ? __builtin_ctzll(hm) : 0);
        }
    }
}

constexpr int kMedWG = 512;
constexpr int64_t kMedTileRows = 4096;  // longest window of the tiled kernel

// Sum over aligned groups of N lanes (a power of two), in every lane of the
// group.  Past 16 lanes gfx950's row swaps: with both operands the same
// value, the two results hold a lane's own and its partner row's value in
// some order.
template <int N>
__device__ __forceinline__ uint32_t group_sum_all32(uint32_t v)
{
    if (N >= 2) v += dpp0<0xB1>(v);   // quad_perm [1,0,3,2]
    if (N >= 4) v += dpp0<0x4E>(v);   // quad_perm [2,3,0,1]
    if (N >= 8) v += dpp0<0x141>(v);  // row_half_mirror
    if (N >= 16) v += dpp0<0x140>(v); // row_mirror
    if (N >= 32) {
        const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = p[0] + p[1];
    }
    if (N >= 64) {
        const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = p[0] + p[1];
    }
    return v;
}

template <int N>
__device__ __forceinline__ uint32_t group_max_all32(uint32_t v)
{
    if (N >= 2) v = max(v, dpp0<0xB1>(v));
    if (N >= 4) v = max(v, dpp0<0x4E>(v));
    if (N >= 8) v = max(v, dpp0<0x141>(v));
    if (N >= 16) v = max(v, dpp0<0x140>(v));
    if (N >= 32) {
        const auto p = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = max(p[0], p[1]);
    }
    if (N >= 64) {
        const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = max(p[0], p[1]);
    }
    return v;
}

// Bits [0, 16) of 32 values as bit planes: bit k of x[b] is bit b of value
// k.  On entry x[i] holds value i in its low half and value i + 16 in its
// high half.  112 VALU instructions: byte permutes for the 8-bit exchange,
// shift and bit-field insert for the others.
__device__ __forceinline__ void bit_planes16(uint32_t (&x)[16])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint32_t a = x[i], b = x[i + 8];
        x[i] = __builtin_amdgcn_perm(b, a, 0x06020400u);
        x[i + 8] = __builtin_amdgcn_perm(b, a, 0x07030501u);
    }
    auto step = [&](int i, int h, uint32_t m) {
        const uint32_t a = x[i], b = x[i + h];
        x[i] = (a & m) | ((b << h) & ~m);
        x[i + h] = ((a >> h) & m) | (b & ~m);
    };
#pragma unroll
    for (int g = 0; g < 16; g += 8) {
#pragma unroll
        for (int i = g; i < g + 4; ++i) step(i, 4, 0x0F0F0F0Fu);
    }
#pragma unroll
    for (int g = 0; g < 16; g += 4) {
#pragma unroll
        for (int i = g; i < g + 2; ++i) step(i, 2, 0x33333333u);
    }
#pragma unroll
    for (int g = 0; g < 16; g += 2) step(g, 1, 0x55555555u);
}

template <int N>
using Int = std::integral_constant<int, N>;

// A workgroup holds 512 / PARTS columns of up to 32 * W * PARTS steps: two
// workgroups per CU (W = 1, 80 KB of LDS, at most 128 VGPRs), whose loads and
// selects cover each other, or one (W = 2, 152 KB) that relies on its own
// prefetch.
template <int PARTS, int W>
__global__ __launch_bounds__(kMedWG) __attribute__((amdgpu_waves_per_eu(W == 1 ? 4 : 2))) void k_window_median(
    const int64_t* __restrict__ d, int64_t T, int64_t C, int64_t window, int64_t nchunk,
    int64_t tiles, int64_t* __restrict__ med)
{
    constexpr int COLS = kMedWG / PARTS;
    constexpr int ROWS = 32 * W * PARTS;
    constexpr int STRIDE = COLS + COLS / 8;  // words per tile row: a wave's column reads hit distinct banks
    constexpr int TPR = COLS / 2;            // threads per tile row, two columns each
    constexpr int RPS = kMedWG / TPR;        // rows per load sweep
    constexpr int NSW = ROWS / RPS;          // load sweeps (16 W)
    constexpr int CPW = 64 / PARTS;          // columns per wave
    static_assert(PARTS >= 2 && PARTS <= 64 && NSW == 16 * W, "shape");
    __shared__ __attribute__((aligned(16))) uint32_t tile[ROWS * STRIDE];
    __shared__ uint32_t wide_sh;  // some value of the tile has a high word

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = tid / TPR;        // this thread's first tile row
    const int c = (tid % TPR) * 2;   // its column pair within a tile row
    const int part = lane % PARTS;
    const int col = wave * CPW + lane / PARTS;  // the column it selects in
    if (tid == 0) wide_sh = 0;

    // the workgroups in flight take adjacent tiles, an XCD's side by side, so
    // that neighbouring pieces of a row are read together (measured against a
    // contiguous run of tiles per XCD: level up to 512 steps, 1-7% faster
    // above 512, 10-15% above 2048)
    const int64_t nslot = gridDim.x;
    auto rows_of = [&](int64_t w) {  // 1 <= n <= ROWS
        const int64_t t0 = w * window;
        return (int)((t0 + window < T ? t0 + window : T) - t0);
    };
    // the next tile in flight.  A pair past the last column is moved back to
    // the last two (C >= 2), of which it takes the second.
    const int wrow = __builtin_amdgcn_readfirstlane(i0);  // the wave's first row
    v2i64 x[NSW];
    auto load = [&](int64_t w, int64_t c0) {
        const int n = rows_of(w);
        const int64_t cc = c0 + c < C - 2 ? c0 + c : C - 2;
        // the wave's rows of a sweep through a buffer resource that ends
        // after row n - 1: slots past the window read 0 without a branch or
        // memory traffic.  A wave of one row or less has it start at the
        // tile's first column, which bounds its offsets at any C; the others
        // are 3-6% slower so (4096 ranks x 12 x 5000, windows of 250 348 : 361 us)
        const int64_t cb = PARTS <= 4 ? c0 : 0;
        const char* q = reinterpret_cast<const char*>(d + (w * window + wrow) * C + cb);
        const uint32_t off = (uint32_t)(((i0 - wrow) * C + cc - cb) * 8);  // below 2^32: the host checks
        const int64_t step = (int64_t)RPS * C * 8;
        int64_t left = ((n - wrow) * C - cb) * 8;
#pragma unroll
        for (int j = 0; j < NSW; ++j) {
            const int over = (int)(left >> 32);  // compared by halves: the scalar unit has no 64-bit order
            const uint32_t bytes = over < 0 ? 0u : (over > 0 ? 0xFFFFFFFFu : (uint32_t)left);
            x[j] = buffer_load16_nt(buffer_rsrc(q, bytes), off, 0);
            q += step;
            left -= step;
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    int64_t id = xcd_block();  // the grid is at most `tiles`
    const int64_t dw = nslot / nchunk, dk = nslot % nchunk;
    int64_t w = id / nchunk, k0 = id % nchunk;  // the tile's window and column chunk
    load(w, min(k0 * COLS, C - 2));
    for (;;) {
        const int n = rows_of(w);
        const int64_t c0 = min(k0 * COLS, C - 2);
        __syncthreads();  // every wave has taken the previous tile's columns
        uint32_t* const at = tile + i0 * STRIDE + (int)(min(c0 + c, C - 2) - c0);
        auto put = [&](bool high) {  // the tile's words: the values' low or high halves
            if (STRIDE % 2 == 0 && (C & 1) == 0) {
                // pairs at even words: one 8-byte store each
#pragma unroll
                for (int j = 0; j < NSW; ++j)
                    *reinterpret_cast<uint2*>(__builtin_assume_aligned(at + j * RPS * STRIDE, 8)) =
                        high ? make_uint2((uint32_t)((u64)x[j].x >> 32), (uint32_t)((u64)x[j].y >> 32))
                             : make_uint2((uint32_t)x[j].x, (uint32_t)x[j].y);
            } else {
#pragma unroll
                for (int j = 0; j < NSW; ++j) {
                    at[j * RPS * STRIDE] = high ? (uint32_t)((u64)x[j].x >> 32) : (uint32_t)x[j].x;
                    at[j * RPS * STRIDE + 1] = high ? (uint32_t)((u64)x[j].y >> 32) : (uint32_t)x[j].y;
                }
            }
        };
        put(false);
        uint32_t hiw = 0;
#pragma unroll
        for (int j = 0; j < NSW; ++j) hiw |= (uint32_t)((u64)x[j].x >> 32) | (uint32_t)((u64)x[j].y >> 32);
        if (__ballot(hiw != 0) != 0 && lane == 0) wide_sh = 1;
        __syncthreads();
        const bool wide = wide_sh != 0;  // uniform over the workgroup
        const int64_t wc = w;
        id += nslot;
        const bool more = id < tiles;
        const uint32_t* base = tile + part * STRIDE + col;
        const bool live = c0 + col < C;
        // the lane's 32 W values (slots part, part + PARTS, ...): the mask m
        // of those that are candidates, at first those within the window, of
        // which the median has rank kk
        uint32_t m[W];
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const int nv = (n - part + PARTS - 1) / PARTS - q * 32;  // slots of this word below n
            m[q] = nv >= 32 ? 0xFFFFFFFFu : (nv <= 0 ? 0u : (1u << nv) - 1u);
        }
        uint32_t kk = (uint32_t)((n - 1) / 2);
        // the candidates' median in the tile's words; fewer are left in m
        auto select = [&]() {
        // the bits below the top one of the columns' OR
        int nbits;
        {
            uint32_t vor = 0;
#pragma unroll
            for (int q = 0; q < W; ++q) {
#pragma unroll
                for (int k = 0; k < 32; ++k) vor |= base[(q * 32 + k) * PARTS * STRIDE];
            }
            vor = wave_or32(vor);
            nbits = vor ? 32 - __builtin_clz(vor) : 0;
        }
        int sh = nbits > 16 ? nbits - 16 : 0;
        for (;;) {
            // bits [sh, sh + 16) of the values as planes; in a second round
            // the candidates agree in those above the first round's sh
            uint32_t v[W][16];
#pragma unroll
            for (int q = 0; q < W; ++q) {
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    v[q][k] = __builtin_amdgcn_perm(base[(q * 32 + k + 16) * PARTS * STRIDE] >> sh,
                                                    base[(q * 32 + k) * PARTS * STRIDE] >> sh, 0x05040100u);
                bit_planes16(v[q]);
                // all planes in registers here: left alone, the compiler
                // moves parts of the transpose into the loop below and spills
#pragma unroll
                for (int k = 0; k < 16; ++k) asm volatile("" : "+v"(v[q][k]));
            }
            // one bit at a time from the top: the candidates with a 0 there
            // are counted over the column's lanes
            auto levels = [&](auto hi, auto lo) {
#pragma unroll
                for (int b = decltype(hi)::value; b >= decltype(lo)::value; --b) {
                    uint32_t one[W], zero[W], cnt = 0;
#pragma unroll
                    for (int q = 0; q < W; ++q) {
                        one[q] = m[q] & v[q][b];
                        zero[q] = m[q] ^ one[q];
                        cnt += (uint32_t)__popc(zero[q]);
                    }
                    cnt = group_sum_all32<PARTS>(cnt);
                    const bool up = kk >= cnt;
#pragma unroll
                    for (int q = 0; q < W; ++q) m[q] = up ? one[q] : zero[q];
                    kk = min(kk, kk - cnt);
                }
                // whether every column of the wave has one candidate left
                uint32_t left = 0;
#pragma unroll
                for (int q = 0; q < W; ++q) left += (uint32_t)__popc(m[q]);
                return __ballot(live && group_sum_all32<PARTS>(left) != 1) == 0;
            };
            bool one_left = levels(Int<15>(), Int<7>());
            if (!one_left) one_left = levels(Int<6>(), Int<4>());
            if (!one_left) one_left = levels(Int<3>(), Int<0>());
            if (one_left || sh == 0) break;
            sh = sh > 16 ? sh - 16 : 0;
        }
        // the candidates left are equal (or one): any lane that has one
        // gives the column's median
        uint32_t res = 0;
#pragma unroll
        for (int q = 0; q < W; ++q)
            if (m[q]) res = base[(q * 32 + __builtin_ctz(m[q])) * PARTS * STRIDE];
        return group_max_all32<PARTS>(res);
        };
        uint32_t high = 0;
        if (wide) {
            // the high halves first (the values are still in x), then the low
            // ones of the candidates that are left
            __syncthreads();  // every wave has read wide_sh
            put(true);
            if (tid == 0) wide_sh = 0;
            __syncthreads();
            high = select();
            __syncthreads();
            put(false);
            __syncthreads();
        }
        if (more) {
            w += dw;
            k0 += dk;
            if (k0 >= nchunk) {
                k0 -= nchunk;
                ++w;
            }
            load(w, min(k0 * COLS, C - 2));  // flies while this tile is resolved
        }
        const uint32_t res = select();
        if (part == 0 && live) med[wc * C + c0 + col] = (int64_t)(((u64)high << 32) | res);
        if (!more) break;
    }
}

// Windows longer than the tile rows (or a single column): one wave per
// (window, stage, rank), the 64-bit streaming select over the column in global memory.
constexpr int kMedLongWG = 256;

__global__ __launch_bounds__(kMedLongWG) void k_window_median_long(const int64_t* __restrict__ d,
                                                                    int64_t T, int R, int S,
                                                                    int64_t window, int64_t W,
                                                                    int64_t* __restrict__ med)
{
    __shared__ __attribute__((aligned(16))) uint32_t hist[kMedLongWG / 64][kSelWords];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    uint32_t* h = hist[wave];
    for (int i = lane; i < kSelWords; i += 64) h[i] = 0;
    wave_lds_fence();
    const int64_t total = W * S * (int64_t)R;
    const int64_t waves = (int64_t)gridDim.x * (kMedLongWG / 64);
    for (int64_t id = (int64_t)blockIdx.x * (kMedLongWG / 64) + wave; id < total; id += waves) {
        const int64_t ws = id / R;
        const int r = (int)(id - ws * R);
        const int64_t w = ws / S;
        const int s = (int)(ws - w * S);
        const int64_t t0 = w * window;
        const int64_t n = (t0 + window < T ? t0 + window : T) - t0;
        const int64_t* col = d + (t0 * S + s) * (int64_t)R + r;
        const int64_t cs = (int64_t)S * R;
        const u64 m = wave_select_stream([&](int64_t i) { return (u64)col[i * cs]; }, n, h, lane);
        if (lane == 0) med[id] = (int64_t)m;
    }
}

struct MedianVariant {
    const void* fn;
    int cols;  // columns per tile
    int64_t most;  // columns C whose rows of one wave lie within 32-bit offsets
};

template <int PARTS, int W>
MedianVariant median_variant()
{
    // a wave's load takes PARTS / 4 rows, or a part of one
    return MedianVariant{reinterpret_cast<const void*>(&k_window_median<PARTS, W>), kMedWG / PARTS,
                         PARTS <= 4 ? INT64_MAX : (int64_t)(UINT32_MAX / 8 / (PARTS / 4))};
}

// By the longest window's steps.  Past 512 steps W = 2: twice the columns per
// tile row beat the second workgroup per CU (measured at 4096 ranks: windows
// of 1000 steps 4.3 -> 5.0 TB/s with 256- instead of 128-byte row pieces, of
// 2000 steps 2.5 -> 3.6 with 128 instead of 64).
MedianVariant pick_median(int64_t n)
{
    if (n <= 64) return median_variant<2, 1>();
    if (n <= 128) return median_variant<4, 1>();
    if (n <= 256) return median_variant<8, 1>();
    if (n <= 512) return median_variant<16, 1>();
    if (n <= 1024) return median_variant<16, 2>();
    if (n <= 2048) return median_variant<32, 2>();
    return median_variant<64, 2>();  // n <= kMedTileRows
}

}  // namespace sfk

using namespace sfk;

SF_API int sf_window_median(const int64_t* durations, int64_t T, int32_t R, int32_t S,
                            int64_t window, int64_t* out_median, sf_stream_t stream)
{
    if (T < 0 || R < 1 || R > SF_MAX_R || S < 1 || window < 1) return SF_EINVAL;
    if (!fits(T, S, R, 8)) return SF_EINVAL;
    if (T == 0) return SF_OK;
    const int64_t n_max = window < T ? window : T;
    const int64_t W = sf_num_windows(T, window);
    if (!fits(W, S, R, 8)) return SF_EINVAL;
    if (!durations || !out_median) return SF_EINVAL;
    if (!aligned(durations, 8) || !aligned(out_median, 8)) return SF_EINVAL;
    if (!disjoint(durations, T * S * (int64_t)R * 8, out_median, W * S * (int64_t)R * 8))
        return SF_EINVAL;
    int cus = 0;
    if (device_cus(stream, &cus) != SF_OK) return SF_EHIP;
    if (cus < 1) cus = 1;
    const int64_t C = (int64_t)S * R;
    const MedianVariant v = pick_median(n_max);
    if (n_max > kMedTileRows || C < 2 || C > v.most) {
        const int64_t total = W * C;
        const int64_t want = (total + kMedLongWG / 64 - 1) / (kMedLongWG / 64);
        const int64_t grid = want < (int64_t)cus * 8 ? want : (int64_t)cus * 8;
        int Ri = R, Si = S;
        int64_t Wl = W;
        void* args[] = {(void*)&durations, (void*)&T, (void*)&Ri, (void*)&Si,
                        (void*)&window, (void*)&Wl, (void*)&out_median};
        return launch(reinterpret_cast<const void*>(&k_window_median_long), dim3((unsigned)grid),
                      dim3(kMedLongWG), args, 0, stream);
    }
    int64_t nchunk = (C + v.cols - 1) / v.cols;
    int64_t tiles = W * nchunk;
    const int64_t most = (int64_t)cus * (n_max <= 512 ? 2 : 1);
    const int64_t grid = tiles < most ? tiles : most;
    void* args[] = {(void*)&durations, (void*)&T,     (void*)&C,         (void*)&window,
                    (void*)&nchunk,    (void*)&tiles, (void*)&out_median};
    return launch(v.fn, dim3((unsigned)grid), dim3(kMedWG), args, 0, stream);
}
