// amq_internal.h — types shared by the HIP kernels and the host engine.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace amq {

constexpr int kWG = 256;          // threads per workgroup (4 wave64)
constexpr int kWaves = kWG / 64;
constexpr int kMaxSlots = 13;     // bridge register window (tree depth + 2 and the anchor; depth <= 10 for 640 dates)
constexpr int kAnchorSlot = kMaxSlots - 1;   // read by the first bridge node only
constexpr int kMaxDates = 640;    // on-chip Sobol lane tables (<= 64 KiB of LDS) bound this
constexpr int kRec = 40;          // doubles per date record
constexpr int kRecTime = 32;      // record slots 32..37: device clock stamps of the date's phases
constexpr int kPartStride = 32;   // doubles per workgroup partial slot (estimator kernel)
constexpr int kMaxGroups = 2048;  // workgroups of one sweep or estimator launch, at most
constexpr int kMaxReps = 64;      // randomised QMC replicates per call

// Barrier block of one sweep (uint32 words, one 64-byte line per counter):
//   line 0: [2] error word (a wait ran out: every workgroup exits),
//           [4] ticket (paper kernel);
//   lines 1 .. kMaxTeams: team arrival counters (monotone; team t has
//   received all arrivals of epoch e at e * (its member count)).
// Groups form at most kMaxTeams teams of team_size(G) consecutive groups.
constexpr int kMaxTeams = 32;
constexpr int kSyncLine = 16;
constexpr int kSyncWords = kSyncLine * (1 + kMaxTeams);
__host__ __device__ inline uint32_t team_size(uint32_t G) { return (G + kMaxTeams - 1) / kMaxTeams; }

// Partial-sum rows of one sweep: [2 epoch parities][G][row_words] 8-byte
// words, then the team rows [2][kMaxTeams][row_words]; each word holds an FP64 partial whose two lowest mantissa bits carry
// epoch & 3 (see allreduce in amq_sync.h).  Zeroed by the generation kernel.
__host__ __device__ constexpr int row_words(int degree) { return 3 * degree + 3 <= 16 ? 16 : 32; }
constexpr int kMaxRowWords = 32;
// group rows [2][G][row_words] then team rows [2][kMaxTeams][row_words]
__host__ __device__ inline int64_t rows_words(int64_t G, int degree) { return 2 * (G + kMaxTeams) * row_words(degree); }
// row padding: a multiple of every sweep tile up to 32768 paths; the
// 65536-path tile is used only where it divides the padded row
constexpr int64_t kLdAlign = 32768;

// One node of the Brownian bridge, in depth-first construction order.  The
// value of W at date m (in units of sqrt(dt)) is
//   W[dst] = wl * W[sl] + wr * W[sr] + sd * z(dim)
// where slots hold the values of the current node's ancestors (slot 0 is the
// constant W(0) = 0).  The first node (date M) reads the anchor slot
// kAnchorSlot with weight 1, which holds 0 for W; no node writes that slot.
// Because wl + wr = 1 below the root, the same schedule carries any process
// a + b t + c W(t): the generation kernels run it on the log-price
// log S0 + (r - sigma^2/2) t + sigma W(t), with slot 0 = log S0, the anchor
// = log S0 + (r - sigma^2/2) T and sigma sqrt(dt) z in place of z.
struct BridgeNode {
    int32_t m;      // date index 1..M
    int32_t dim;    // Sobol dimension, 0-based
    int32_t sl, sr, dst;
    double wl, wr, sd;
};

// The node as the generation kernels read it (scalar loads, half a line).
struct alignas(32) GenNode {
    uint32_t md;     // m | dim << 16
    uint32_t slots;  // 2 sl | 2 sr << 8 | 2 dst << 16: register offsets of the slots
    double wl, wr, sd;
};
static_assert(sizeof(GenNode) == 32, "packed bridge node");
static_assert(kMaxDates < 65536 && 2 * kMaxSlots <= 256, "bridge node packing");

// A schedule of M dates in Q = 2^v segments of `len` nodes each, one after
// another: segment s holds the ancestors of the s-th interval of tree level
// v (recomputed by every segment below them, to bitwise the same values) and
// then that interval's nodes in depth-first order; shorter segments repeat
// their last node, which changes nothing.  A segment's nodes need no others,
// so segments of one path block run in different waves.
constexpr int kSegVariants = 4;    // Q = 1, 2, 4, 8

// Nodes whose tail normals are evaluated together (binary64 paths): a
// 64-point Sobol block puts 10 to 13 of its 64 points of each dimension in
// the tails (|u - 1/2| >= 0.42; 10.24 on average, nearly always 10 or 11), so
// the tails of 6 nodes fill one wave and seldom more (2^24 x 252: 15.64 ms per
// call with 5 nodes, 15.49 with 6).
constexpr int kTailChunk = 6;
// Tail points staged per wave and chunk.  An aligned block of 64 Sobol points
// has exactly one point in each interval [k/64, (k+1)/64) of every dimension
// (the generator matrix's leading 6 x 6 block is triangular with unit
// diagonal; a digital shift permutes the intervals), and the tails meet 12
// such intervals; a wave's lanes hold 63 points of one aligned block and the
// first of the next, so a node has at most 13 tail points.  The staging holds every lane of every node all the same, so no point
// set could write outside it; a point's word becomes its normal in place.
constexpr int kTailCap = kTailChunk * 64;

// Dynamic LDS of a generation workgroup (bytes): the exponential's table [64]
// f64 and the logarithm's [64] {1/F, log F} at fixed offsets (their addresses
// are then immediates), the per-wave tail staging ([kTailCap] points, then
// normals, and 64 spare words), then per schedule node the lane tables [16]
// u32, every wave's block words [2] u32 and the node's dimension.
constexpr size_t kLdsLog = 64 * 8, kLdsTz = kLdsLog + 64 * 16, kLdsSpare = kLdsTz + (size_t)kWaves * kTailCap * 8,
                 kLdsNodes = kLdsSpare + (size_t)kWaves * 64 * 4, kLdsPerNode = 64 + kWaves * 8 + 4;
inline size_t gen_lds_bytes(int len) { return kLdsNodes + (size_t)len * kLdsPerNode; }
constexpr size_t kLdsCu = 160 * 1024;

// Per-date constants written by the generation kernel, read by the sweep.
//   disc = exp(-r t_k); standardised abscissa xs = S * xa + xb with
//   xa = 1/(K sd_k), xb = -mean_k/sd_k (mean/sd of S_k/K in the money under
//   the model).
struct DateConst {
    double disc, xa, xb, pad;
};

struct GenArgs {
    void *S;                  // [M][ld] T (what = 0) or debug output
    const uint32_t *V;        // [dims][32] direction numbers
    const GenNode *sched;     // [segs][seg_len]
    DateConst *datec;         // [M+1]
    uint32_t *sync;           // barrier words, zeroed here
    int64_t N, ld;
    int64_t nblocks;          // 64-path blocks to write: ld / 64 (padding included)
    int32_t segs, seg_len;    // schedule segments and their nodes
    int32_t M, R;             // dates, 64-path blocks per wave
    int32_t what;             // 0 paths, 1 sobol ints, 2 normals (debug)
    int32_t pad;
    const uint32_t *shift;    // [M] digital shift (randomised QMC) or nullptr
    double S0, K, r, sigma, T;
    double mu, vol;           // (r - sigma^2/2) dt, sigma sqrt(dt)
    int32_t is_call, pad2;    // payoff side (standardisation of the in-the-money region)
    uint64_t *rows;           // partial-sum rows to zero (with the barrier words)
    int64_t rows_n;           // their count in 8-byte words
};

struct SweepArgs {
    const void *S;            // [M][ld] T
    void *pv_out;             // [ld] T
    uint64_t *rows;           // partial-sum rows [2][G][row_words(degree)]
    double *rec;              // [M+1][kRec]
    double *result;           // [8]
    uint32_t *sync;           // barrier block [kSyncWords]
    uint32_t *err;            // error word: a wait ran out (every group exits)
    const DateConst *datec;   // [M+1]
    int64_t N, ld;
    int32_t M, G;
    int32_t is_call, allow_exercise, laguerre, degree;
    double S0, K;
    uint32_t spin_limit;
    int32_t xcd_stride;       // > 1: every xcd_stride-th workgroup is a group; > 0: groups announce their XCD
                              // (set by launch_sweep; above 1 on entry: a test's stride)
    double *rep_out;          // randomised QMC: replicate prices [n_rep] or nullptr
    int32_t rep, n_rep;
    double *host_out;         // pinned host copy of the result (put_host_result), or nullptr
};

// Result words in pinned host memory: result[0..5], then 1.0 once written.
// A call that waits for its price reads it there after the stream is done;
// copying 128 bytes back was a kernel of its own on the stream (3.7 us and
// its launch).
constexpr int kHostResultFlag = 8, kHostResultWords = 16;
__device__ inline void put_host_result(double *host, const double *result)
{
    if (!host) return;
    for (int q = 0; q < 6; ++q) host[q] = result[q];
    host[kHostResultFlag] = 1.0;
}

struct PaperArgs {
    const void *S;            // [m][ld] T, dates t_i = i dt
    double *part;             // [kMaxGroups][kPartStride]
    uint32_t *ticket;         // zeroed by the generation kernel
    double *result;           // [8]
    int64_t N, ld;
    int32_t m, is_call;
    double K, r, sigma, dt, S0;
    double *host_out;         // as SweepArgs'
};

// One option of a batch, as the kernels see it (all pointers into the
// caller's workspace or the library's schedule cache).
struct alignas(64) BatchOpt {
    void *S;                  // [M][ld] T
    void *pv;                 // [ld] T
    const GenNode *sched;     // [segments][seg_len]
    DateConst *datec;         // [M+1]
    double *rec;              // [M+1][kRec]
    double *result;           // [8]
    uint32_t *sync;           // barrier block [kSyncWords] of this option
    uint64_t *rows;           // partial-sum rows [2][G][row_words(degree)] of this option
    int64_t rows_n;           // their count in 8-byte words (zeroed by generation)
    int64_t N, ld;
    int32_t M, G;             // dates, tiles
    int32_t tile_base;        // first partial slot / global tile index
    int32_t is_call, allow_exercise;
    int32_t seg_len;          // nodes of one schedule segment
    double S0, K, r, sigma, T, mu, vol;
    const uint32_t *shift;    // [M] digital shift per dimension (randomised QMC), or null
};

struct GenUnit {              // one generation workgroup: blocks [b0, b1) of option opt, schedule segment seg
    int32_t opt, seg;
    int64_t b0, b1;
};

// Claim queues of a batch sweep: a workgroup claims from queue blockIdx mod
// kClaimQueues (the device deals workgroups out to its XCDs in turn, so an
// option's tiles run on one XCD and exchange within its L2).  Only where every
// group has a compute unit of its own; else there is one queue.
constexpr int kClaimQueues = 8;

struct BatchGlobal {
    uint32_t *claim;          // claim counters [queues] (zeroed by generation)
    int32_t queues;           // kClaimQueues or 1
    int32_t q_off[kClaimQueues + 1];   // queue q: tiles q_off[q] .. q_off[q + 1] - 1 of the list
    uint32_t *err;            // error word (zeroed by generation), of every option of the launch
    int32_t total_tiles, laguerre;
    uint32_t spin_limit, pad;
    // a launch over both storage types (kMixed): the binary64 part's options, else null
    const BatchOpt *opts64;
};

// `fp64` of the batch sweep's launcher and capacity for both storage types
// in one launch (monomials; ppt then names the binary32 tile, 64).
constexpr int kMixed = 2;

// Whether a path's log-price can leave the range in which the generator's
// exponential builds the exponent by adding (|x| < 700).  |X| <= |log S0| +
// |mu| M + 6.4 (the largest normal) x vol sqrt(M) x (1 + 1/2 + 1/2^1.5 + ...,
// the bridge levels' deviations: below 2.8).
inline bool wide_exponent(double S0, double mu, double vol, int M)
{
    const double bound = fabs(log(S0)) + fabs(mu) * M + 18.0 * vol * sqrt((double)M);
    return !(bound < 700.0);
}
constexpr int kGenWide = 4;    // beside the storage type of launch_generate_batch: some option is wide

// Launchers (defined with the kernels).
hipError_t launch_generate(const GenArgs &a, int fp64, hipStream_t s);
// Load the single-option generation kernels on the current device.
hipError_t preload_generate();
// Single-option sweep with wg (256 or 512) threads per group.  Returns
// hipErrorInvalidValue if no kernel exists for (fp64, a.laguerre, wg, ppt,
// a.degree).
hipError_t launch_sweep(const SweepArgs &a, int fp64, int wg, int ppt, hipStream_t s);
// Workgroups of the sweep kernel that fit on one CU (0: no such kernel).
int sweep_blocks_per_cu(int fp64, int laguerre, int wg, int ppt, int degree);
hipError_t launch_paper(const PaperArgs &a, int fp64, hipStream_t s);
hipError_t launch_generate_batch(const BatchOpt *opts, const GenUnit *units, int n_units,
                                 const uint32_t *V, uint32_t *gsync, int max_seg_len, int fp64,
                                 bool shifted, hipStream_t s);
// spread: at most one workgroup per CU (grid <= CUs, nothing else persistent beside it).
hipError_t launch_sweep_batch(const BatchOpt *opts, const int32_t *tile_opt, const BatchGlobal &g,
                              int grid, int fp64, int ppt, int degree, bool spread, hipStream_t s);
int sweep_batch_blocks_per_cu(int fp64, int laguerre, int ppt, int degree);
// Beside the storage type of sweep_batch_blocks_per_cu: how many of those
// groups find room whatever else has run on the CU.  With k - 1 groups anywhere
// in its LDS a hole for the k-th is left if (2k - 1) groups' LDS fit (one of the
// 66 KB tiles, though two fit side by side).
constexpr int kAnyPlacement = 8;
// Sweep kernel tables, one translation unit per (precision, basis kind); kinds
// as sweep_addr says.  Null where not built.
const void *sweep_table_f32_mono(int ppt, int degree, int kind);
const void *sweep_table_f32_lag(int ppt, int degree, int kind);
const void *sweep_table_f64_mono(int ppt, int degree, int kind);
const void *sweep_table_f64_lag(int ppt, int degree, int kind);
// Many options of both storage types, 64 binary32 or 32 binary64 paths per thread.
const void *sweep_table_mixed(int degree);

}  // namespace amq
