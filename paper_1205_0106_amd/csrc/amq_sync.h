// amq_sync.h — device-wide waits and fixed-order reductions shared by the
// persistent sweep and the estimator kernels (gfx950).
#pragma once

#include "amq_internal.h"

namespace amq {

// threadIdx.x through an empty asm: a value the compiler cannot share across
// calls.  The helpers below run once per date inside the sweeps' date loops;
// with their per-lane indexes and addresses derived from it, those are
// recomputed at each call (a few instructions) instead of being hoisted out
// of the loop and held in registers, or spilled to scratch memory and
// reloaded on the date's critical path, in kernels whose registers hold
// path data.
__device__ __forceinline__ uint32_t tid_x()
{
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

__device__ __forceinline__ uint32_t ld_agent(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A wave-uniform binary64 value moved to scalar registers.
__device__ __forceinline__ double uniform_f64(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Lane l's binary64 value in every lane.
__device__ __forceinline__ double readlane_f64(double x, int l)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), l);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ void raise_error(uint32_t *err)
{
    __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// x + (the value DPP control `CTRL` moves into this lane), binary64 through
// two 32-bit DPP moves.  Lanes outside ROW_MASK, or without a source lane,
// get an unspecified value: only lane 63 of the final sum is used, and it
// depends on none of them.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, ROW_MASK, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xF, false);
    return x + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Sum of x over the 64 lanes of a wave, valid in lane 63 (other lanes hold
// unspecified values), in a fixed order on the vector unit (DPP, no LDS
// round trips): neighbour swaps within quads, the half-row and row mirrors
// (every lane of a 16-lane row then holds the row sum), then row 2 into row 3
// (row_bcast:15) and row 1 into row 3 (row_bcast:31).
__device__ __forceinline__ double wave_sum(double x)
{
    x = dpp_add<0xB1, 0xF>(x);    // quad_perm [1,0,3,2]
    x = dpp_add<0x4E, 0xF>(x);    // quad_perm [2,3,0,1]
    x = dpp_add<0x141, 0xF>(x);   // row_half_mirror
    x = dpp_add<0x140, 0xF>(x);   // row_mirror
    x = dpp_add<0x142, 0xA>(x);   // row_bcast:15 into rows 1 and 3
    x = dpp_add<0x143, 0xC>(x);   // row_bcast:31 into rows 2 and 3
    return x;
}

// x(row 2i) + x(row 2i+1) in every lane of both rows (16-lane rows), and
// x(lane l mod 32) + x(lane l mod 32 + 32): gfx950's row-swapping permutes
// (v_permlane16_swap / v_permlane32_swap), lower operand first in every lane.
__device__ __forceinline__ double add_rows16(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)b, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
    return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}

__device__ __forceinline__ double add_halves32(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)b, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
    return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
           __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}

// Sum NV doubles over a workgroup of WG threads in a fixed order (wave_sum
// in each wave, then the waves in order).  The last NU components are
// wave-uniform (a wave's total already, e.g. a ballot count): summed over the
// waves only.  s_red: LDS [WG / 64][32].  Returns, in the first wave, the
// total of the lane's component `comp` (0 for comp >= NV): one lane per
// component adds the waves' partials, where one thread adding every
// component's would read NV WG / 64 words in turn.
template <int NV, int NU = 0, int WG = kWG>
__device__ __forceinline__ double group_sum(double (&v)[NV], double (*s_red)[32], uint32_t comp)
{
    const uint32_t tx = tid_x();
    const int lane = tx & 63, wave = tx >> 6;
#pragma unroll
    for (int q = 0; q < NV - NU; ++q) v[q] = wave_sum(v[q]);
    if (lane == 63) {
#pragma unroll
        for (int q = 0; q < NV; ++q) s_red[wave][q] = v[q];
    }
    __syncthreads();
    double t = 0.0;
    if (tx < 64 && comp < (uint32_t)NV) {
        t = s_red[0][comp];
#pragma unroll
        for (int w = 1; w < WG / 64; ++w) t += s_red[w][comp];
    }
    return t;
}

// The same sum through LDS for groups with two waves per SIMD: every thread
// stores its NV - NU components ([8][WG] doubles at s_x), then component q's
// WG/8 threads each add 8 of them (stride WG/8, ascending) and reduce their
// partials on the vector unit (a 64-lane wave_sum, or the 32-lane half of it
// for WG = 256); the wave-uniform components go through s_red as in
// group_sum.  Fewer vector instructions than a DPP tree per component when
// NV - NU is large.  Result as group_sum's.
template <int NV, int NU, int WG>
__device__ __forceinline__ double group_sum_lds(double (&v)[NV], double *s_x, double (*s_red)[32], uint32_t comp)
{
    const uint32_t tx = tid_x();
    constexpr int NC = NV - NU, TPC = WG / 8;
    static_assert(NC <= 8 && NV <= 32 && (TPC == 32 || TPC == 64), "component slots");
    const int tid = tx, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int q = 0; q < NC; ++q) s_x[q * WG + tid] = v[q];
    if (lane == 63) {
#pragma unroll
        for (int u = 0; u < NU; ++u) s_red[wave][NC + u] = v[NC + u];
    }
    __syncthreads();
    const int q = tid / TPC, l = tid % TPC;
    double acc = 0.0;
    if (q < NC) {
        double x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = s_x[q * WG + l + i * TPC];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += x[i];
    }
    if (TPC == 64) {
        acc = wave_sum(acc);
        if (lane == 63 && q < NC) s_red[0][q] = acc;
    } else {
        acc = dpp_add<0xB1, 0xF>(acc);
        acc = dpp_add<0x4E, 0xF>(acc);
        acc = dpp_add<0x141, 0xF>(acc);
        acc = dpp_add<0x140, 0xF>(acc);
        acc = dpp_add<0x142, 0xA>(acc);   // lanes 31 and 63: their half-wave's sum
        if ((lane & 31) == 31 && q < NC) s_red[0][q] = acc;
    }
    __syncthreads();
    double t = 0.0;
    if (tx < 64 && comp < (uint32_t)NV) {
        t = s_red[0][comp];
        if (NU > 0 && comp >= (uint32_t)NC) {
#pragma unroll
            for (int w = 1; w < WG / 64; ++w) t += s_red[w][comp];
        }
    }
    return t;
}

// The same sum in three steps, so that the first wave is free between them:
// the threads' components into LDS (one barrier, inside), their reduction by
// waves 1 .. NC (component q by wave q + 1; bitwise group_sum_lds' sums), and,
// after a barrier of the caller's, each lane's component.
template <int NV, int NU, int WG>
__device__ __forceinline__ void split_sum_store(const double (&v)[NV], double *s_x, double (*s_red)[32])
{
    const uint32_t tx = tid_x();
    constexpr int NC = NV - NU;
    static_assert(WG == 512 && NC <= 7, "one wave per component, beside the first");
#pragma unroll
    for (int q = 0; q < NC; ++q) s_x[q * WG + tx] = v[q];
    if ((tx & 63u) == 63u) {
#pragma unroll
        for (int u = 0; u < NU; ++u) s_red[tx >> 6][NC + u] = v[NC + u];
    }
    __syncthreads();
}

template <int NV, int NU, int WG>
__device__ __forceinline__ void split_sum_reduce(const double *s_x, double (*s_red)[32])
{
    const uint32_t tx = tid_x();
    constexpr int NC = NV - NU, TPC = WG / 8;
    const int wave = __builtin_amdgcn_readfirstlane((int)(tx >> 6)), l = tx & 63;
    if (wave >= 1 && wave <= NC) {
        const int q = wave - 1;
        double x[8], acc = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = s_x[q * WG + l + i * TPC];
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += x[i];
        acc = wave_sum(acc);
        if (l == 63) s_red[0][q] = acc;
    }
}

template <int NV, int NU, int WG>
__device__ __forceinline__ double split_sum_fetch(double (*s_red)[32], uint32_t comp)
{
    constexpr int NC = NV - NU;
    double t = 0.0;
    if (tid_x() < 64 && comp < (uint32_t)NV) {
        t = s_red[0][comp];
        if (NU > 0 && comp >= (uint32_t)NC) {
#pragma unroll
            for (int w = 1; w < WG / 64; ++w) t += s_red[w][comp];
        }
    }
    return t;
}

// Fixed-order sum of G partial slots (kPartStride doubles apart) into
// tot[0..NV-1] (LDS), by the whole workgroup.  Thread t owns component t % 32
// of groups t/32, t/32 + 8, ...; its loads are issued in batches of 4 before
// any is consumed, then added in group order.
template <int NV>
__device__ void reduce_partials(const double *part, uint32_t G, double *tot, double (*s_red8)[32])
{
    const uint32_t tx = tid_x();
    const int c = tx & 31, sgrp = tx >> 5;   // 8 groups of 32
    double v = 0.0;
    if (c < NV) {
        for (uint32_t g0 = sgrp; g0 < G; g0 += 8 * 4) {
            double buf[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t g = g0 + 8u * u;
                buf[u] = g < G ? part[(size_t)g * kPartStride + c] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) v += buf[u];
        }
    }
    s_red8[sgrp][c] = v;
    __syncthreads();
    if (tx < NV) {
        double t = 0.0;
#pragma unroll
        for (int s = 0; s < 8; ++s) t += s_red8[s][tx];
        tot[tx] = t;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Device-wide fixed-order sum of NV doubles, every workgroup receiving the
// total (an all-gather of per-group partials; no group waits on another's
// release).
//
// Each group owns one row of RW 8-byte words in the parity-(epoch & 1) half
// of `rows` ([2][G][RW]).  Lanes of the first wave store the group's NV partials there with
// single-copy-atomic 8-byte stores, the two lowest mantissa bits of each word
// replaced by epoch & 3 (a change of at most 3 units in the last place, the
// same in every run).  A reader reads rows until every word carries this
// epoch's tag (no store needs to drain before another), then adds them in a
// fixed order.  Forms by group count and tile:
//  - few groups (spins_on_rows): the first wave of every group reads all rows;
//  - up to kFlatMaxGroups, in tiles with work to do behind the exchange
//    (register-resident): flat.  Thread 0 bumps its team's arrival
//    counter with the row; behind the overlapped work the whole group reads
//    every row at once, and only on a miss waits for the counters;
//  - up to kFlatMaxGroups, in other tiles: relayed.  Group g belongs to
//    team g mod kXcds, on one XCD where workgroups are dealt to XCDs in turn;
//    the first member (group t of team t) adds its team's rows, up to 32 and
//    from its own L2, and publishes a team row; every group reads the kXcds
//    team rows.  One round trip inside an XCD and one through memory, where the
//    flat form takes two through memory and 8 MB of reads a date (245 groups x
//    60 dates 1103 us per call flat, 995 relayed; 2^24 x 252 15.28 and 14.9 ms;
//    but register-resident, 256 groups x 100 dates, 778 flat and 814 relayed:
//    the first round trip is hidden there, the relay's turn is not);
//  - above: teams of consecutive groups; a team's last arriver (its arrival
//    counter's return value) sums the team's rows, every group then polls and
//    sums the team rows.
// Every group computes bitwise the same total.
//
// Two parities suffice: a group writes the parity of epoch e + 2 only after
// epoch e + 1 is complete, and every group finished reading epoch e before
// publishing its e + 1 row.  A stale word left from epoch e - 2 carries a
// different tag.  The generation kernel zeroes the rows (tag 0) before each
// sweep, so words of an earlier sweep never match epochs 1..3, and epoch 4
// reads words rewritten at epoch 2.
//
// Waits are bounded by `limit` polls; on running out, or on seeing the error
// word raised by another group, returns false (the caller exits).
// v: lane c of the first wave holds component c.  tot: LDS [>= NV], valid in every thread on return.
// s_flag: LDS [2 + WG / 64]; s_red: LDS [WG / 64][32].
// ---------------------------------------------------------------------------
// Fixed-order sum of rows [0, count) of `slots` (RW words each, tagged):
// lane c of each RW-lane slice reads word c, KB rows per thread in flight;
// every word must carry `tag`, else on_miss(attempt) is called by every
// thread (a collective wait that returns false to give up) and the rows are
// read again, at most `limit` times.  Each thread adds its rows in ascending
// order, then the group's lanes and waves in a fixed tree.  tot: LDS
// [>= NV], valid in every thread on true.
template <int NV, int RW, int WG, typename OnMiss>
__device__ inline bool sum_rows(const uint64_t *slots, uint32_t count, uint64_t tag, uint32_t *err,
                                uint32_t limit, double *tot, double (*s_red)[32], int *s_flag, OnMiss on_miss)
{
    const uint32_t tx = tid_x();
    static_assert(RW == 16 || RW == 32, "row width");
    constexpr int NW = WG / 64;
    constexpr uint32_t RP = WG / RW;    // rows per pass
    // passes per batch (loads in flight per thread; 512-thread groups hold
    // their cashflows and slab values in registers meanwhile).  The order in
    // which a thread adds its rows does not depend on it.
    constexpr int KB = WG >= 512 ? 8 : 16;
    const uint32_t c = tx % RW, rs = tx / RW;
    const int lane = tx & 63, wave = tx >> 6;
    uint32_t it = 0;
    for (;;) {
        double acc = 0.0;
        bool bad = false;
        for (uint32_t r0 = 0; r0 < count; r0 += KB * RP) {
            uint64_t w[KB];
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                const uint32_t r = r0 + rs + (uint32_t)k * RP;
                w[k] = (r < count && c < (uint32_t)NV)
                           ? __hip_atomic_load(slots + (size_t)r * RW + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                           : tag;
            }
#pragma unroll
            for (int k = 0; k < KB; ++k) {
                bad |= (w[k] & 3u) != tag;
                acc += __longlong_as_double((long long)(w[k] & ~3ull));
            }
        }
        // lanes c, c + RW, ... of a wave hold the same component
        if (RW == 16) acc = add_rows16(acc);
        acc = add_halves32(acc);
        const bool wbad = __builtin_amdgcn_ballot_w64(bad) != 0;
        if (lane < RW) s_red[wave][lane] = acc;
        if (lane == 0) s_flag[1 + wave] = wbad ? 1 : 0;
        __syncthreads();
        bool anybad = false;
#pragma unroll
        for (int q = 0; q < NW; ++q) anybad |= s_flag[1 + q] != 0;
        if (!anybad) {
            if (tx < NV) {
                double t = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) t += s_red[q][tx];
                tot[tx] = t;
            }
            __syncthreads();
            return true;
        }
        if (++it > limit) {
            if (tx == 0) raise_error(err);
            return false;
        }
        if (!on_miss(it)) return false;
    }
}

// The default wait between reads of rows: a short sleep; false once another
// group has raised the error word.  Collective.
__device__ inline bool rows_backoff(uint32_t *err, int *s_flag)
{
    const uint32_t tx = tid_x();
    if (tx == 0) s_flag[0] = ld_agent(err) != 0u ? 1 : 0;
    __builtin_amdgcn_s_sleep(1);
    __syncthreads();
    return s_flag[0] == 0;
}

// Lanes 0..NV-1 of the first wave: store the lane's value v as word `lane` of
// a tagged row (single-copy-atomic words, one store instruction).  local:
// every reader shares this group's L2 (xcd_local), so the store stops there;
// else it is written through for the other XCDs.
template <int NV>
__device__ __forceinline__ void put_row(uint64_t *row, double v, uint64_t tag, bool local = false)
{
    const uint32_t tx = tid_x();
    if (tx < (uint32_t)NV) {
        const uint64_t b = ((uint64_t)__double_as_longlong(v) & ~3ull) | tag;
        if (local) __hip_atomic_store(row + tx, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else __hip_atomic_store(row + tx, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Words of all rows (G x RW) up to which one wave reads every row in one go
// and spins on the tags themselves (spin_rows): eight loads per lane.  With
// arrival counters, waiting on a counter and reading the rows
// after it was one memory round trip more per date, which is most of a date
// with few groups: 15 groups x 365 dates (30011 paths, binary32) 1554 -> 1340
// us per call, 16 groups x 50 dates 217 -> 194 us, a book of 12 options 3861
// -> 3037 us.
constexpr uint32_t kSpinWords = 512;
constexpr uint32_t kXcds = 8;
constexpr uint32_t kFlatMaxGroups = 32 * kXcds;
template <int RW> __host__ __device__ __forceinline__ bool spins_on_rows(uint32_t G) { return G * (uint32_t)RW <= kSpinWords; }

// Which forms of the sum a kernel holds.  The single-option sweeps of
// register-resident tiles are compiled apart for few groups and for counters:
// with both in one kernel each date took 0.15 to 0.25 us longer (binary32,
// degree 2, 49 groups x 50 dates 214 us per call, apart 203; 10^5 paths x 10
// dates 51.8 and 49.4).
enum : int {
    kAnyForm,       // few groups, flat and teams
    kRelayForm,     // few groups, relayed and teams
    kFewForm,       // few groups
    kCounterForm,   // flat and teams
};

// Whether the first wave gathers the totals alone: rows spun on, or relayed.
template <int FORM, int RW>
__device__ __forceinline__ bool first_wave_gathers(uint32_t G)
{
    if constexpr (FORM == kFewForm) return true;
    else if constexpr (FORM == kCounterForm) return false;
    else return spins_on_rows<RW>(G) || (FORM == kRelayForm && G <= kFlatMaxGroups);
}

// Publishing half of the sum: the first wave's lanes store the group's row
// (lane c: word c); where counters are kept (flat, and above kFlatMaxGroups)
// thread 0 bumps its team's, and above kFlatMaxGroups the team's last arriver
// also sums its team's rows into the team row.
// The caller may do independent work before the gathering half with the same
// epoch.  Uses s_flag[1 + WG / 64] (the team-last flag), so that the
// gathering half's flags never overlap it.  local: see put_row.
template <int NV, int RW, int WG, int FORM>
__device__ inline bool allreduce_publish(double v, uint32_t gid, uint32_t G, uint64_t *rows,
                                         uint32_t *words, uint32_t *err, uint32_t epoch, uint32_t limit,
                                         double *tot, double (*s_red)[32], int *s_flag, bool local = false)
{
    const uint32_t tx = tid_x();
    static_assert(NV <= RW && RW <= 32 && (RW & (RW - 1)) == 0, "row width");
    const uint64_t tag = epoch & 3u;
    if (FORM != kCounterForm && G == 1) {
        // alone: the group's sums are the totals (rounded as a row's words are)
        if (tx < (uint32_t)NV)
            tot[tx] = __longlong_as_double((long long)((uint64_t)__double_as_longlong(v) & ~3ull));
        return true;
    }
    uint64_t *slots = rows + (size_t)(epoch & 1u) * G * RW;
    put_row<NV>(slots + (size_t)gid * RW, v, tag, local);
    if (first_wave_gathers<FORM, RW>(G)) return true;
    uint64_t *tslots = rows + (size_t)2 * G * RW + (size_t)(epoch & 1u) * kMaxTeams * RW;
    const uint32_t TS = team_size(G);
    const uint32_t tau = gid / TS;
    if (G <= kFlatMaxGroups) {
        // the counter's old value is not used: nothing waits for the round trip
        if (tx == 0)
            (void)__hip_atomic_fetch_add(words + kSyncLine * (1 + tau), 1u, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    // team level: the team's last arriver sums its team's rows in member
    // order and publishes the team row (tagged like the group rows)
    if (tx == 0) {
        const uint32_t old = __hip_atomic_fetch_add(words + kSyncLine * (1 + tau), 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
        s_flag[1 + WG / 64] = old + 1u == epoch * min(TS, G - tau * TS) ? 1 : 0;
    }
    __syncthreads();
    if (s_flag[1 + WG / 64]) {
        const uint32_t first = tau * TS;
        if (!sum_rows<NV, RW, WG>(slots + (size_t)first * RW, min(TS, G - first), tag, err, limit, tot, s_red,
                                  s_flag, [&](uint32_t) { return rows_backoff(err, s_flag); }))
            return false;
        put_row<NV>(tslots + (size_t)tau * RW, tx < (uint32_t)NV ? tot[tx] : 0.0, tag);
    }
    return true;
}

// Reads `count` rows, `stride` words apart, until each word carries the
// epoch's tag, by the first wave alone, then adds them in exactly sum_rows'
// order (thread rs + 64 / RW wave of the group there is lane rs of step
// `wave` here), so the totals are bitwise the same.  NL: loads per lane
// (count RW <= 64 NL).  t: the total of component `lane` in lanes 0..NV-1.
// Returns false (in every lane) when the wait runs out or another group
// raised the error word.
template <int NV, int RW, int WG, int NL>
__device__ __forceinline__ bool spin_rows(const uint64_t *slots, uint32_t stride, uint32_t count, uint64_t tag,
                                          uint32_t *err, uint32_t limit, double &t)
{
    constexpr int NW = WG / 64;
    constexpr uint32_t RL = 64 / RW;    // rows per step
    const uint32_t lane = tid_x() & 63u, sub = lane / RW;
    const uint32_t c = min(lane % RW, (uint32_t)NV - 1u);
    uint64_t w[NL];
    uint32_t it = 0;
    for (;;) {
        // rows past the last read the last again (its tag is waited for anyway)
#pragma unroll
        for (int j = 0; j < NL; ++j)
            w[j] = __hip_atomic_load(slots + (size_t)min((uint32_t)j * RL + sub, count - 1u) * stride + c,
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t raised = ld_agent(err);
        bool bad = false;
#pragma unroll
        for (int j = 0; j < NL; ++j) bad |= (w[j] & 3u) != tag;
        if (__builtin_amdgcn_ballot_w64(bad) == 0) break;
        if (raised != 0u) return false;
        if (++it / 4 > limit) {   // (a quarter of a counter poll's length each)
            if (lane == 0) raise_error(err);
            return false;
        }
    }
    t = 0.0;
#pragma unroll
    for (int q = 0; q < NW && q < NL; ++q) {
        double acc = 0.0;
#pragma unroll
        for (int j = q; j < NL; j += NW)
            acc += (uint32_t)j * RL + sub < count ? __longlong_as_double((long long)(w[j] & ~3ull)) : 0.0;
        if (RW == 16) acc = add_rows16(acc);
        t += add_halves32(acc);
    }
    return true;
}

// The totals of `epoch` where rows are spun on or relayed, by the first wave
// alone.  tot: LDS [>= NV], written by lanes 0..NV-1.
template <int NV, int RW, int WG, int FORM>
__device__ __forceinline__ bool first_wave_totals(uint64_t *rows, uint32_t gid, uint32_t G, uint32_t *err,
                                                  uint32_t epoch, uint32_t limit, double *tot)
{
    if (G == 1) return true;   // (published straight into tot)
    const uint64_t tag = epoch & 3u;
    const uint64_t *slots = rows + (size_t)(epoch & 1u) * G * RW;
    const uint32_t lane = tid_x() & 63u;
    double t = 0.0;
    if (FORM == kFewForm || spins_on_rows<RW>(G)) {
        const bool ok = G * (uint32_t)RW <= kSpinWords / 2
                            ? spin_rows<NV, RW, WG, 4>(slots, RW, G, tag, err, limit, t)
                            : spin_rows<NV, RW, WG, 8>(slots, RW, G, tag, err, limit, t);
        if (!ok) return false;
    } else if constexpr (FORM == kRelayForm) {
        uint64_t *tslots = rows + (size_t)2 * G * RW + (size_t)(epoch & 1u) * kMaxTeams * RW;
        if (gid < kXcds) {
            if (!spin_rows<NV, RW, WG, RW / 2>(slots + (size_t)gid * RW, kXcds * RW, (G - gid + kXcds - 1) / kXcds, tag,
                                               err, limit, t))
                return false;
            put_row<NV>(tslots + (size_t)gid * RW, t, tag);
        }
        if (!spin_rows<NV, RW, WG, (int)kXcds * RW / 64>(tslots, RW, kXcds, tag, err, limit, t)) return false;
    }
    if (lane < (uint32_t)NV) tot[lane] = t;
    return true;
}

// Which stores may stop in an L2.  The device deals a launch's workgroups out
// to its XCDs in turn.  With few groups, kXcds times as many are launched and
// every kXcds-th, all on one XCD, is kept; with more, a relayed team is one
// XCD's.  That placement is not relied on: groups announce the XCD they run on
// (hardware register XCC_ID; past the team rows, zeroed with them, device
// scope), and a group's rows stay in its L2 only where all readers are there
// too: every group (spins_on_rows; all give the same answer), or its team's
// first (relayed).  Readers use device-scope loads either way.  Between groups
// on different XCDs a published row takes a round trip through memory: 1.07 us
// per exchange of 16 groups, 0.44 on one XCD (measured alone).
__device__ __forceinline__ uint64_t own_xcd()
{
    return 1ull + (uint64_t)(__builtin_amdgcn_s_getreg((31 << 11) | 20) & 0xFFu);   // XCC_ID, whole register
}

template <int RW>
__device__ __forceinline__ uint64_t *xcd_words(uint64_t *rows, uint32_t G)
{
    return rows + (size_t)2 * G * RW + (size_t)kXcds * RW;
}

template <int RW>
__device__ __forceinline__ void xcd_announce(uint64_t *rows, uint32_t gid, uint32_t G)
{
    if (tid_x() == 0 && gid < (spins_on_rows<RW>(G) ? G : kXcds))
        __hip_atomic_store(xcd_words<RW>(rows, G) + gid, own_xcd(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Call with every lane of the first wave.
template <int RW>
__device__ __forceinline__ bool xcd_local(uint64_t *rows, uint32_t gid, uint32_t G, uint32_t *err, uint32_t limit)
{
    const uint32_t lane = tid_x() & 63u;
    const uint64_t *w = xcd_words<RW>(rows, G) + (spins_on_rows<RW>(G) ? min(lane, G - 1u) : gid % kXcds);
    uint64_t x = 0;
    for (uint32_t it = 0;;) {
        x = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t raised = ld_agent(err);
        if (__builtin_amdgcn_ballot_w64(x == 0) == 0) break;
        if (raised != 0u) return false;
        if (++it / 4 > limit) {
            if (lane == 0) raise_error(err);
            return false;
        }
    }
    return __builtin_amdgcn_ballot_w64(x != own_xcd()) == 0;
}

// Wave-level ordering of LDS writes before LDS reads by other lanes.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Gathering half: wait until every group (or team) of `epoch` has published,
// then sum the rows in the fixed order into tot (LDS, every thread).  Flat:
// wave 0 waits on the team counters, then the rows are read (re-read until
// every word carries the tag).  With rows_first (a caller that did other
// work since publishing, so the rows usually all carry the tag already) the
// rows are read once before the counters, which saves their round trip.
// Teams: wave 0 waits on the team rows' tags, then the team rows are summed.
template <int NV, int RW, int WG>
__device__ inline bool allreduce_gather(uint32_t G, uint64_t *rows, uint32_t *words, uint32_t *err,
                                        uint32_t epoch, uint32_t limit, double *tot, double (*s_red)[32],
                                        int *s_flag, bool rows_first)
{
    const uint32_t tx = tid_x();
    const uint64_t tag = epoch & 3u;
    uint64_t *slots = rows + (size_t)(epoch & 1u) * G * RW;
    uint64_t *tslots = rows + (size_t)2 * G * RW + (size_t)(epoch & 1u) * kMaxTeams * RW;
    const uint32_t TS = team_size(G), NT = (G + TS - 1) / TS;
    const bool flat = G <= kFlatMaxGroups;
    auto poll = [&]() -> bool {
        if (tx < 64) {
            // flat: lane t < NT watches team t's counter; teams: lane t
            // watches team t's row (word 0 carries the epoch tag).
            // Wave-uniform exit.
            const uint32_t lane = tx;
            const uint32_t want = lane < NT ? min(TS, G - lane * TS) * epoch : 0u;
            uint32_t it = 0;
            bool ok = true;
            for (;;) {
                bool pending;
                if (flat) {
                    const uint32_t seen = lane < NT ? ld_agent(words + kSyncLine * (1 + lane)) : 0u;
                    pending = seen < want;
                } else {
                    const uint64_t w0 = lane < NT ? __hip_atomic_load(tslots + (size_t)lane * RW, __ATOMIC_RELAXED,
                                                                      __HIP_MEMORY_SCOPE_AGENT)
                                                  : tag;
                    pending = (w0 & 3u) != tag;
                }
                if (__builtin_amdgcn_ballot_w64(pending) == 0) break;
                if (ld_agent(err) != 0u) { ok = false; break; }
                if (++it > limit) { if (lane == 0) raise_error(err); ok = false; break; }
                __builtin_amdgcn_s_sleep(1);
            }
            if (lane == 0) s_flag[0] = ok ? 1 : 0;
        }
        __syncthreads();
        return s_flag[0] != 0;
    };
    const bool early = flat && rows_first;
    if (!early && !poll()) return false;
    return sum_rows<NV, RW, WG>(flat ? slots : tslots, flat ? G : NT, tag, err, limit, tot, s_red, s_flag,
                                [&](uint32_t attempt) {
                                    return (early && attempt == 1) ? poll() : rows_backoff(err, s_flag);
                                });
}

// Gathering half with the follow-up work `solve` (the first wave only, on the
// totals in LDS): one group barrier between the totals and the group's use of
// what `solve` left in LDS.  s_flag[0] carries the outcome.  meanwhile():
// work that needs no total and in which the first wave has no part.  Where rows
// are spun on or relayed the other waves do it while the first waits; else it
// comes before the rows are first read, which then more often finds them there
// (400000 paths x 100 dates, Laguerre, binary64 514 us per call, behind the
// first reads 523; binary32, degree 2, 10^5 x 50 203 and 208; 2^20 x 100 the same
// either way).
struct Nothing { __device__ __forceinline__ void operator()() const {} };
template <int NV, int RW, int WG, int FORM, typename Solve, typename Work = Nothing>
__device__ inline bool gather_and_solve(uint32_t gid, uint32_t G, uint64_t *rows, uint32_t *words, uint32_t *err,
                                        uint32_t epoch, uint32_t limit, double *tot, double (*s_red)[32], int *s_flag,
                                        bool rows_first, Solve solve, Work meanwhile = Work())
{
    const uint32_t tx = tid_x();
    const bool one = first_wave_gathers<FORM, RW>(G);
    if (!one) {
        meanwhile();
        if (!allreduce_gather<NV, RW, WG>(G, rows, words, err, epoch, limit, tot, s_red, s_flag, rows_first)) return false;
    }
    if (tx < 64) {
        const bool ok = !one || first_wave_totals<NV, RW, WG, FORM>(rows, gid, G, err, epoch, limit, tot);
        if (ok) {
            wave_lds_fence();
            solve();
        }
        if (one && tx == 0) s_flag[0] = ok ? 1 : 0;
    } else if (one) {
        meanwhile();
    }
    __syncthreads();
    return !one || s_flag[0] != 0;
}

}  // namespace amq
