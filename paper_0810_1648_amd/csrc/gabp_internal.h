// Internal declarations shared by the host runtime and the HIP kernels of
// the GaBP SVM solver.  Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include <string>

#include "../../include/gabp_svm.h"

namespace gabp {

// Pairs {i, j}, i < j, are processed in TILE x TILE tiles of the upper
// triangle; every per-pair device array is a sequence of full tiles stored
// row-major (tile-local row r, column c at r * TILE + c).
constexpr int TILE = 256;
constexpr int TT = TILE * TILE;
constexpr int WG = 256;               // threads per workgroup (4 wave64)
constexpr int FB = 64;                // nodes per finalize workgroup

enum Prec : int { PREC_FP64 = 0, PREC_FP32 = 1, PREC_MIXED = 2 };
enum GramKind : int { GRAM_F32 = 0, GRAM_BF16 = 1, GRAM_BF16X3 = 2, GRAM_F64 = 3, GRAM_BF16X6 = 4 };
enum KSrc : int { KSRC_PLANE = 0, KSRC_RECOMPUTE = 1 };
enum Reason : int { R_NONE = 0, R_CONVERGED = 1, R_MAX_SWEEPS = 2, R_DIVERGED = 3, R_STAGNATED = 4 };

// Device-resident solve status, advanced by k_status once per sweep.  Every
// sweep kernel returns at once when `done` is set, so the state a solve
// stops in does not depend on how often the host polls.
struct DevStatus {
    int32_t t;           // completed sweeps
    int32_t done;
    int32_t reason;
    int32_t since_best;  // sweeps since the smallest change so far
    int32_t bad;         // set when a cavity precision <= 0 or a value is not finite
    int32_t g;           // served grouped schedule: the group the next step visits
    uint32_t ticket;     // finalize workgroups of the running sweep that have written their maxima
    double delta;        // ||alpha^t - alpha^(t-1)||_inf
    double amax;         // ||alpha^t||_inf
    double best_delta;
};

struct StopRule {
    double tol_abs, tol_rel, stag_rel;
    int32_t max_sweeps, stag_window;
};

// Features staged for the Gram: row-major NPAD x m_pad, zero padded.
struct Features {
    const float* f32;        // GRAM_F32: centred FP32
    const uint16_t* hi;      // GRAM_BF16/BF16X3: centred, rounded to BF16
    const uint16_t* lo;      // GRAM_BF16X3/X6: BF16 of the rounding remainder x - hi
    const uint16_t* lo2;     // GRAM_BF16X6: BF16 of the second remainder x - hi - lo
    const double* f64;       // GRAM_F64: uncentred FP64
    const float* nrm;        // squared norms of the staged rows (FP32)
    int32_t m_pad;
    int32_t kind;            // GramKind
    // BF16 kinds with m + 2 <= m_pad, K' recomputed: the training rows
    // augmented as (x, |x|^2, 1) (aug0) and (c x, -c/2, -c/2 |x|^2) (aug1,
    // c = 2 gamma log2(e)), in the kind's split planes `aug_plane` apart, so
    // that their Gram is the exponent -gamma log2(e) |x_i - x_j|^2 itself
    // (null: K' from the plain Gram and the norms)
    const uint16_t* aug0;
    const uint16_t* aug1;
    int64_t aug_plane;
};

struct KernelParams {
    int64_t N;
    int32_t NB;
    float neg_gamma_log2e;   // -gamma * log2(e): K = exp2(neg_gamma_log2e * d2)
    double gamma;
    double lam2;             // lambda^2 added to every RBF entry
};

// Validates a parameter struct (shared by the solver and the server).
gabp_status check_params(const gabp_svm_params* p, std::string& why);

inline int64_t n_tiles(int NB) { return (int64_t)NB * (NB + 1) / 2; }

// Workgroups (of WG threads) per launch.  A launch holds fewer than 2^32 threads
// and silently drops the rest: 2^24 workgroups, the tiles of 1.48 M points.
// in_launches calls f(first, count) for consecutive parts of n workgroups.
constexpr int64_t kMaxBlocks = (int64_t)1 << 23;
template <class F>
inline hipError_t in_launches(int64_t n, F&& f) {
    for (int64_t o = 0; o < n; o += kMaxBlocks) {
        const hipError_t e = f(o, std::min(kMaxBlocks, n - o));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Stateless plan from the contraction bound.  rr = 1.25 rho bounds
// |A_ij| / Q_ij, the factor with which a reverse message enters the next
// one, so unrolling `levels` levels truncates the recursion by about
// rr^levels.  Levels needed: the smallest count with rr^levels below the
// path's message precision, 2^-24 (FP32), 2^-30 (MIXED, FP32-stored
// messages), 2^-50 (FP64); 9 when no count up to 8 suffices.
inline int stateless_levels_needed(int prec, double rr) {
    const double eps = (prec == PREC_FP32) ? std::ldexp(1.0, -24)
                     : (prec == PREC_MIXED) ? std::ldexp(1.0, -30) : std::ldexp(1.0, -50);
    if (rr == 0.0) return 1;
    if (!(rr < 1.0)) return 9;
    return std::max(1, (int)std::ceil(std::log(eps) / std::log(rr)));
}
// Reciprocal form of a stateless plan: 0 exact reciprocals; 1 / 2 series
// around 1/P~ with a one- / two-term top level; 3 a one-term top level over
// lower levels that take G = 1/P~ (no series term).  |e| <= rr^2, so the
// one-term lower levels err by rr^4, entering the top level scaled by rr,
// and the top level errs by rr^4 (one term) or rr^6 (two terms).  Form 3
// drops the lower levels' e: G errs by rr^2, which reaches the top level's
// precision term scaled by rr^2 (rr^4) and its mean term through F scaled by
// rr (rr^3); it needs a middle level (levels >= 3).  Each error must stay
// below the precision of the message arithmetic (FP32 messages: FP32 and
// MIXED; FP64 messages: FP64).
inline int stateless_series_form(int prec, int levels, double rr) {
    const double eps = (prec == PREC_FP64) ? std::ldexp(1.0, -52) : std::ldexp(1.0, -24);
    if (levels < 1 || levels > 6 || !(rr < 0.25) || std::pow(rr, 5) > eps) return 0;
    if (std::pow(rr, 4) <= eps) return (levels >= 3 && std::pow(rr, 3) <= eps) ? 3 : 1;
    if (std::pow(rr, 6) <= eps) return 2;
    return 0;
}
// The kernels of a synchronous series sweep: the form, plus kSerLevels where the
// plan would sum over powers of K' (two levels of form 1, three of form 3) but
// those powers leave the range of its arithmetic, and the sweep runs level by
// level instead.  The recursion forms K'^2 only; the sums K'^3 and K'^4, beside
// 1/P~^2.  amax bounds |K'_ij|, pmin (the contraction bound's m*) every P~ from
// below.  FP32: K' up to 2^30 keeps K'^4 at 2^120, so that its products, which
// are below K'^2 again, sum without overflow; P~ from 2^-16 on: what underflow
// takes from K'^4 (2^-126 each) is then at most 2^-126 2^64 of P~ for one
// pair, 2^-38 for 2^24 of them.  FP64 likewise with 2^240 and 2^-200.  (Entries
// of order one, as every RBF kernel has, run 1.05 to 1.5 times as fast by the
// sums; the parameter lambda_aug and a given matrix reach any scale.)
constexpr int kSerLevels = 4;
inline int series_kernels(int prec, int levels, int ser, double amax, double pmin) {
    if (!((levels == 2 && ser == 1) || (levels == 3 && ser == 3))) return ser;
    const bool fp64 = prec == PREC_FP64;
    const bool in_range = amax <= std::ldexp(1.0, fp64 ? 240 : 30) && pmin >= std::ldexp(1.0, fp64 ? -200 : -16);
    return in_range ? ser : ser | kSerLevels;
}
// Entries of the grouped schedule's visit lists: bit 31 = messages into the
// row block (BWD; clear: into the column block), bit 30 = both blocks lie in
// the visited group, low 30 bits = tile index.
constexpr uint32_t GE_BWD = 0x80000000u, GE_WITHIN = 0x40000000u, GE_TILE = 0x3FFFFFFFu;
// Synchronous stateless sweeps over an FP32 K' plane with FP32 partial sums
// (FP32 plan, or FP32 messages) run over 2 x 2 chunks of tiles where the
// chunk's sums fit beside the message recursion in the registers of four
// waves per SIMD: one level, two with series reciprocals, three with series
// form 3.
__host__ __device__ constexpr bool chunk_plan(bool fp32_partials, int levels, int ser) {
    return fp32_partials && (levels == 1 || (levels == 2 && ser > 0) || (levels == 3 && ser == 3));
}
// The choice for one solve (`mode`: the tile_chunk parameter): automatic
// (0) takes chunks only with at least four per workgroup slot of the GPU (256
// CUs x 4 workgroups), since fewer balance worse than single tiles; 1 never,
// 2 wherever the plan allows.
constexpr int64_t kChunkMin = 4096;
inline bool chunk_sweep(bool fp32_partials, int levels, int ser, int NB, int mode) {
    const int64_t nbc = (NB + 1) / 2;
    if (mode == 1 || !chunk_plan(fp32_partials, levels, ser)) return false;
    return mode == 2 || nbc * (nbc + 1) / 2 >= kChunkMin;
}
// Row parts per tile of a sweep over whole tiles (1, 2, 4 or 8 workgroups per
// tile, each with 256 / split of its rows), for a launch of `items` tiles or
// single-direction entries: the fewest that give two workgroups per CU.  A
// tile's 64 row steps are one serial chain per wave, so a launch of fewer
// tiles than that takes the chain's time whatever its size: N = 500 in FP64
// (3 tiles) 13.4 -> 3.8 ms per solve with eight parts, N = 3,001 in FP32 (78
// tiles) 4.5 -> 2.8 ms.  Beyond it the parts' prologues and column partials
// cost more than they fill: visits of 1,550 entries (N = 40,009, 16 groups) 11.4
// ms at 512, 12.1 at 2,048 and 15.6 at 8,192, 3,160 tiles (N = 20,000) 20.1,
// 20.2 and 21.8 ms, a burst of 48 served solves 54, 57 and 61 ms.
inline int tile_split(int64_t items) {
    for (int sp = 1; sp < 8; sp *= 2)
        if (items * sp >= 512) return sp;
    return 8;
}
// Partial-sum slots of node block K when every tile is split into `split` row
// parts (a tile's column sums then take one slot per part, its row sums one
// slot, each part storing its own rows): the column sums of part s of tile
// (I, K), I < K, in slot I split + s; the row sums of tile (K, J) in slot
// K split + J - K; the column sums of part s of the diagonal tile in slot
// K split + NB - K + s.  part_stride slots are set aside per block;
// part_slots(K) of them are in use.
__host__ __device__ inline int part_stride(int NB, int split) { return NB * split + 1; }
__host__ __device__ inline int part_slots(int K, int NB, int split) { return split * (K + 1) + NB - K; }
// Synchronous sweeps with stored pair records over a K' plane (single solves)
// write the records every third sweep and form the sweeps between again from
// the aggregates: 25.3 bytes per FP32 pair and sweep instead of 36, for one
// more message level per sweep on average.  N = 20,011 (2.0e8 pairs, 7.2 GB of
// planes) 116 -> 77 ms per solve of 76 sweeps, the same to the bit; a period
// of four would save 5% of the bytes more and take another level in registers.
// Planes that stay in the last-level cache take the period too: N = 2,000 in
// FP64 6.0 -> 4.4 ms, N = 4,000 in MIXED 7.3 -> 5.5 ms, N = 500 1.6 and 1.8 ms.
// A plan whose budget has no room for the two rings more writes every sweep.
constexpr int kStoredPeriod = 3;
// Storage index of tile (I, J), I <= J: row-major over the upper triangle.
__host__ __device__ inline int64_t tile_index(int I, int J, int NB) {
    return (int64_t)I * NB - (int64_t)I * (I - 1) / 2 + (J - I);
}

// ---- launchers (gabp_kernels.hip); all asynchronous on `s` ----
hipError_t launch_fill_tiles(uint32_t* tiles, int NB, hipStream_t s);
hipError_t launch_validate(const float* X, const float* y, int64_t N, int64_t m,
                           int32_t* flag, hipStream_t s);
hipError_t launch_colmean(const float* X, int64_t N, int64_t m, double* mean, hipStream_t s);
hipError_t launch_stage(const float* X, const double* mean, int64_t N, int64_t m,
                        int64_t NPAD, int m_pad, int kind, float* f32, uint16_t* hi,
                        uint16_t* lo, uint16_t* lo2, double* f64, float* nrm, hipStream_t s);
// FP32-stored K' (every Gram kind but FP64) together with the row/column
// sum and maximum partials of k_rowsum, in one pass.  `tiles` lists the
// upper tiles in any order (each is written at its tile_index position).
hipError_t launch_gram_sums(const Features& F, const KernelParams& kp, const uint32_t* tiles, int64_t ntiles,
                            void* Kp, int NB, double* psum, double* pmax, hipStream_t s);
hipError_t launch_gram(const Features& F, const KernelParams& kp, const uint32_t* tiles,
                       int64_t ntiles, void* Kp, hipStream_t s);
hipError_t launch_gather_dense(const double* K, const KernelParams& kp,
                               const uint32_t* tiles, int64_t ntiles, void* Kp, int prec,
                               double* kdiag, hipStream_t s);
hipError_t launch_fill_value(double* dst, int64_t n, double v, hipStream_t s);
hipError_t launch_rowsum(const void* Kp, int prec, int ksrc, const Features& F,
                         const KernelParams& kp, const uint32_t* tiles, int64_t ntiles, int NB,
                         double* psum, double* pmax, hipStream_t s);
hipError_t launch_diag(int64_t N, int NB, const double* psum, const double* pmax,
                       const double* kdiag, int mode, double C, double delta, double* Adiag,
                       double* rowmax, double* rsum, double* scratch_blk, double* scratch_one,
                       hipStream_t s);
// boxC > 0 (here and in the finalize launchers): belief means projected
// onto [0, boxC] (the box-projected variant); 0: no projection.
hipError_t launch_init(int prec, int64_t N, int64_t NPAD, int R, const double* Adiag, const float* y,
                       void* Pt, void* S, double* alpha, DevStatus* st, hipStream_t s, double boxC = 0.0);

// Arguments of one sweep launch.  HP/HS are rings of R aggregate vectors
// (NPAD entries each); slot_top holds the aggregates of the previous sweep,
// slot_top - k (mod R) those k sweeps earlier.
struct SweepArgs {
    const uint32_t* tiles;
    int64_t ntiles;
    int NB;
    const void* Kp;               // K' plane (KSRC_PLANE)
    void *Pf, *Pb, *Ef, *Eb;      // pair planes: P_ij, P_ji, E_ij, E_ji (i < j), stored state
    const void *HP, *HS;          // aggregate rings
    const void *HI, *HM;          // series: rings of 1/P~ and S/P~ (null: formed in the tile)
    int64_t NPAD;
    int R, slot_top, levels;      // ring depth, top slot, stateless levels in use
    int part32;                   // 1: partial sums stored in FP32 (FP32-message plans)
    void *partP, *partE;          // [NB][part_stride][TILE] partial sums (aggregate type, or FP32);
                                  // chunked sweeps: [NB][NBc+1][TILE], NBc = ceil(NB / chunk)
    const uint32_t* chunks;       // chunked synchronous sweep: Ic << 16 | Jc, Ic <= Jc < NBc (row-major)
    int64_t nchunks;
    int chunk;                    // tiles per chunk side (0 or 1: one tile per workgroup)
    int split;                    // row parts per tile (1 with chunks)
    int period, between;          // stored state: sweeps per write of the planes (0 or 1: every sweep), and how
                                  // many sweeps before this one they were last written
    DevStatus* st;
    Features F;                   // KSRC_RECOMPUTE
    KernelParams kp;
};
// Per-request state of the served form: sweep arguments plus what the
// finalize and stop-rule steps need.  Aggregates live in sw.HP / sw.HS (ring
// of sw.R slots: 1 for stored pair records, 8 for the stateless form; the
// slot of a sweep follows from the request's sweep count).
struct ReqDesc {
    SweepArgs sw;
    int64_t N;
    const double* Adiag;
    const float* y;
    double* alpha;
    double* blk_delta;
    double* blk_amax;
    double* trace;
    StopRule rule;
    int nblk;
    int G;               // groups of the grouped schedule (1: synchronous)
};
// One served step for the requests of one group (precision, level count:
// 0 = stored pair records, >= 1 stateless; series reciprocals): batched sweep
// over the (request, tile) items, batched finalize over the (request, node
// block) items, batched stop rule for the request slots listed in `slots`,
// whose statuses are copied to status_out[0..nslots).
// A served step, launched in this order on one stream: the batched sweep of
// every launch group (items (request, tile); grouped: (request, list entry)
// of each request's current group), the batched finalize of the (request,
// node block) items of each aggregate type (grouped: the current group's
// blocks), and the stop rule of every active request (grouped: after the
// visit of its last group; G = 1 is the synchronous schedule), whose
// statuses are copied to status_out[0..nslots).
hipError_t launch_served_sweep(int prec, int levels, int ser, bool grouped, const ReqDesc* reqs, const uint2* items,
                               int n, hipStream_t s);
hipError_t launch_served_finalize(bool agg_f32, const ReqDesc* reqs, const uint2* items, int n, hipStream_t s);
hipError_t launch_served_status(const ReqDesc* reqs, const int* slots, int nslots, DevStatus* status_out,
                                hipStream_t s);
hipError_t launch_served_sweep_f32(int levels, int ser, bool grouped, const ReqDesc* reqs, const uint2* items, int n,
                                   hipStream_t s);
hipError_t launch_served_sweep_mixed(int levels, int ser, bool grouped, const ReqDesc* reqs, const uint2* items,
                                     int n, hipStream_t s);
hipError_t launch_served_sweep_f64(int levels, int ser, bool grouped, const ReqDesc* reqs, const uint2* items, int n,
                                   hipStream_t s);
// depth 0 = stored edge state, 1..8 = stateless with up to `depth` levels.
// levels: 0 = stored edge state, >= 1 = stateless with that many levels in
// this launch; ser: stateless reciprocals by the series around 1/P~;
// e0 / e1 (optional): events that take the kernel's begin / end timestamps.
hipError_t launch_sweep(int prec, int ksrc, int gram, int levels, bool first, int ser, const SweepArgs& a,
                        hipStream_t s, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_sweep_f32(int ksrc, int gram, int levels, bool first, int ser, const SweepArgs& a,
                            hipStream_t s, hipEvent_t e0, hipEvent_t e1);
hipError_t launch_sweep_mixed(int ksrc, int gram, int levels, bool first, int ser, const SweepArgs& a,
                              hipStream_t s, hipEvent_t e0, hipEvent_t e1);
hipError_t launch_sweep_f64(int ksrc, int gram, int levels, bool first, int ser, const SweepArgs& a,
                            hipStream_t s, hipEvent_t e0, hipEvent_t e1);
// Arguments of one finalize launch: the new aggregates of the nodes
// [b0 FB, N) (b1 > 0: of the 256-node blocks [b0, b1)) from the partial sums.
// Inv / Mean (optional, with Pt / S): the new 1/P~ and S/P~ of the series
// sweeps, formed once per node here instead of in every tile.  part32: the
// partial sums are FP32 (SweepArgs::part32).  trace: the last workgroup to
// finish applies the stop rule to the sweep (null: no stop rule, as after the
// visits of all groups but the last).
struct FinalizeArgs {
    int64_t N;
    int stride, split, NB;        // slots set aside per block; part_slots(K, NB, split) in use (split = 1: all)
    const void *partP, *partE;
    const double* Adiag;
    const float* y;
    void *Pt, *S, *Inv, *Mean;
    double *alpha, *blk_delta, *blk_amax;
    DevStatus* st;
    double boxC;
    int part32;
    int64_t b0, b1;               // 256-node blocks (b1 = 0: all)
    double* trace;
    StopRule rule;
};
hipError_t launch_finalize(int prec, const FinalizeArgs& f, hipStream_t s);
// Inv / Mean of every ring slot from Pt / S (R slots of NPAD entries).
hipError_t launch_ring_recip(int prec, int64_t NPAD, int R, const void* Pt, const void* S, void* Inv, void* Mean,
                             hipStream_t s);
// Grouped schedule: one group visit.  `within` lists the stored-record tiles
// inside the group (both directions), `dir` the single-direction entries
// (tile index | GE_BWD | GE_WITHIN bits, see gabp_device.h); t = sweep index.
hipError_t launch_sweep_grouped(int prec, int ksrc, int gram, int levels, int ser, const SweepArgs& a,
                                const uint32_t* within, int nwithin, const uint32_t* dir, int ndir, int t,
                                hipStream_t s);
hipError_t launch_sweep_grouped_f32(int ksrc, int gram, int levels, int ser, const SweepArgs& a,
                                    const uint32_t* within, int nwithin, const uint32_t* dir, int ndir, int t,
                                    hipStream_t s);
hipError_t launch_sweep_grouped_mixed(int ksrc, int gram, int levels, int ser, const SweepArgs& a,
                                      const uint32_t* within, int nwithin, const uint32_t* dir, int ndir, int t,
                                      hipStream_t s);
hipError_t launch_sweep_grouped_f64(int ksrc, int gram, int levels, int ser, const SweepArgs& a,
                                    const uint32_t* within, int nwithin, const uint32_t* dir, int ndir, int t,
                                    hipStream_t s);
// Sparsified kernel (gabp_sparse.hip): build passes, sorts and scans (the
// temporary storage size comes back in *bytes when tmp is NULL), and the
// sweep by row quads with the join of the rows that leave a workgroup's range.
// count: kept pairs of tiles[0], tiles[stride], ... (ntiles launched);
// fill: every listed tile's kept pairs appended at *cursor (slots >= cap
// counted, not written), keys i << sh | j.
// FA, FB: the augmented A and B rows (launch_sp_augment), whose Gram is
// -d^2 / 2.
hipError_t launch_sp_count(const Features& FA, const Features& FB, const uint32_t* tiles, int64_t ntiles,
                           int64_t stride, int64_t N, float cut, int64_t* counts, hipStream_t s);
hipError_t launch_sp_fill(const Features& FA, const Features& FB, const uint32_t* tiles, int64_t ntiles, int64_t N,
                          float cut, float neg_gamma_log2e, float lam2, int64_t cap, unsigned long long* cursor, int sh,
                          uint64_t* keys, float* kv, hipStream_t s);
// Columns m, m + 1 (< m_pad) of the staged rows: A planes (n_i, 1), B planes
// the first m columns of A and (-1/2, -n_i/2); NPAD rows.
hipError_t launch_sp_augment(int64_t NPAD, int64_t m, int m_pad, int kind, const float* nrm, float* f32a,
                             uint16_t* hia, uint16_t* loa, uint16_t* lo2a, float* f32b, uint16_t* hib,
                             uint16_t* lob, uint16_t* lo2b, hipStream_t s);
// Exclusive sums of n 64-bit values (64 bits on both sides: the scan adds in
// its input's type, and the sums of all rows pass 2^31 from 2^30 kept pairs on).
hipError_t sp_scan(void* tmp, size_t* bytes, const int64_t* in, int64_t* out, int64_t n, hipStream_t s);
// The tile list in super-blocked order (S x S tiles per super-block, NB
// blocks per side), through the key buffers k0, k1 (nt entries each).
hipError_t sp_tile_order(void* tmp, size_t* bytes, uint32_t* tiles, int64_t nt, int S, int NB, uint64_t* k0,
                         uint64_t* k1, hipStream_t s);
// Locality order: nearest of the K landmark points lm[] for every point
// (key = landmark << 32 | point, ids = point), rows permuted into that order,
// block centroids / radii and the tiles that may hold kept pairs, and
// compaction of the tile list.
hipError_t launch_sp_order(const float* X, int64_t N, int64_t m, const int32_t* lm, int K, uint64_t* key,
                           int32_t* ids, hipStream_t s);
hipError_t launch_sp_permute(const float* X, const float* y, int64_t N, int64_t m, const int32_t* order, float* Xp,
                             float* yp, hipStream_t s);
hipError_t launch_sp_prune(const float* Xp, int64_t N, int64_t m, int NB, const uint32_t* tiles, int64_t nt,
                           double cut, double* cent, double* rad, uint8_t* keep, hipStream_t s);
hipError_t sp_select(void* tmp, size_t* bytes, const uint32_t* in, const uint8_t* flags, uint32_t* out,
                     int64_t* nsel, int64_t n, hipStream_t s);
hipError_t sp_sort_keys(void* tmp, size_t* bytes, const uint64_t* kin, uint64_t* kout, const float* vin,
                        float* vout, int64_t n, int bits, hipStream_t s);
hipError_t sp_sort_ids(void* tmp, size_t* bytes, const uint64_t* kin, uint64_t* kout, const int32_t* vin,
                       int32_t* vout, int64_t n, hipStream_t s);
hipError_t launch_sp_unpack(const uint64_t* keys, int64_t E, int sh, int32_t* ei, int32_t* ej, uint64_t* keys_t,
                            hipStream_t s);
// First position of every node in sorted keys (node = key >> sh; N + 1 values).
hipError_t launch_sp_offsets(const uint64_t* keys, int64_t E, int sh, int64_t N, int64_t* off, hipStream_t s);
// Row lengths (N + 1 values, the last 0) in whole quads, at least one, and
// the rows of all nodes (neighbour, K') from row[k] (the exclusive sums of the
// lengths), a node's i-end edges first; at most 2 E + 4 N entries.  qrow: the
// node of every quad.
hipError_t launch_sp_rowlen(int64_t N, const int64_t* off_i, const int64_t* off_j, int64_t* len, hipStream_t s);
hipError_t launch_sp_rows(int64_t E, int64_t N, int sh, const int32_t* ei, const int32_t* ej, const float* kv,
                          const uint64_t* keys_t, const float* kv_t, const int64_t* off_i, const int64_t* off_j,
                          const int64_t* row, int32_t* col, float* rkv, int32_t* qrow, hipStream_t s);
hipError_t launch_sp_rowsum(int64_t N, const int64_t* row, const float* kv, double* psum, double* pmax, hipStream_t s);
// (P~, S) pairs from the separate aggregates.
hipError_t launch_sp_pack(int prec, int64_t N, const void* Pt, const void* S, void* PS, hipStream_t s);
// Sweep t = 1, 2, ... over the rows with its stop rule: rec[t & 1] holds the
// packed (P, E) messages into every node of sweep t - 2 and takes sweep t's,
// PS[t & 1] the packed aggregates likewise; PS[(t - 1) & 1] those of sweep
// t - 1.  dmax / amax: 256 doubles each, zero before the first sweep; edge:
// four aggregates per 256 quads.
struct SparseSweep {
    int64_t nq;                  // quads of all rows
    const int64_t* row;
    const int32_t *qrow, *col;
    void* edge;
    const float* kv;
    void* rec[2];
    void* PS[2];
    const double* Adiag;
    const float* y;
    double *alpha, *dmax, *amax, *trace;
    DevStatus* st;
    double boxC;
    StopRule rule;
};
hipError_t launch_sp_sweep(int prec, const SparseSweep& a, int t, hipStream_t s);
// A-priori contraction bound: one[0] = -m* (minus the aggregate lower
// bound), one[1] = rho (+inf when no bound exists), one[2] = max |K'_ij|.
// blk: two doubles per 256 nodes.
hipError_t launch_rho_bound(int64_t N, const double* Adiag, const double* rowmax, const double* rsum,
                            double* blk, double* one, hipStream_t s);
// Residual certificate of a finished dense solve: out[0] = ||1 - A alpha||_inf,
// out[1] = min_i (A_ii - sum_{j != i} |A_ij|), out[2] = out[0] / out[1]
// (Varah's bound on ||alpha - A^-1 1||_inf; +inf unless out[1] > 0).  K'
// from the plane or recomputed; w (NPAD), part (partial-sum layout), blk1,
// blk2 (grid1(N)) are work buffers.
hipError_t launch_residual(const void* Kp, int prec, int ksrc, const Features& F, const KernelParams& kp,
                           const uint32_t* tiles, int64_t ntiles, int NB, int64_t N, int64_t NPAD,
                           const double* alpha, const float* y, const double* Adiag, const double* rsum,
                           double* w, double* part, double* blk1, double* blk2, double* out, hipStream_t s);
hipError_t launch_kernel_entries(const void* Kp, int prec, int NB, const int64_t* rows,
                                 const int64_t* cols, int64_t n, double* out, hipStream_t s);
// Decision function (gabp_predict.hip).  Queries are padded to
// predict_query_pad(nq) rows; the MFMA form splits the training rows into
// nchunk chunks of bpc 32-row blocks (predict_chunks) and writes
// part[nchunk][NQPAD]; the direct FP64 form writes part[nq].
int64_t predict_query_pad(int64_t nq);
// Bytes of the per-device scratch array of the allocation-free decision
// function (gabp_svm_predict_noalloc), and its device address on the current
// device (looked up once per device, then cached).
constexpr size_t PREDICT_SCRATCH_BYTES = size_t(64) << 20;
hipError_t predict_scratch(void** ptr);
void predict_chunks(int64_t NPAD, int64_t NQPAD, int* nchunk, int* bpc);
// w and its sums over blocks of WG rows (ceil(NPAD / WG) of them).
hipError_t launch_predict_weights(const double* alpha, const float* y, int64_t N, int64_t NPAD, bool box,
                                  double C, double* w, double* blk, hipStream_t s);
hipError_t launch_predict_direct(const float* Xtr, const double* w, int64_t N, int64_t m, const float* Xq,
                                 int64_t nq, double gamma, double* part, hipStream_t s);
hipError_t launch_predict_mfma(const Features& Ft, const Features& Fq, const double* w, int64_t NPAD,
                               int64_t NQPAD, float neg_gamma_log2e, int nchunk, int bpc, double* part,
                               hipStream_t s);
// Augmented form (BF16 split kinds, m + 2 <= mp, mp = 32 or 64): rows staged
// by launch_stage_aug (side 0 queries (x, n, 1); side 1 training rows
// c (x, -1/2, -n/2), c = 2 gamma log2(e); `out` holds np planes of NPAD x mp
// BF16); queries padded to predict_query_pad_aug, part[nchunk][NQPAD].
int64_t predict_query_pad_aug(int64_t nq);
void predict_chunks_aug(int64_t NPAD, int64_t NQPAD, int* nchunk, int* bpc);
hipError_t launch_stage_aug(const float* X, const double* mean, int64_t n, int64_t m, int64_t NPAD, int mp, int kind,
                            int side, float c, uint16_t* out, hipStream_t s);
// e0 / e1 (optional): events that take the kernel's begin / end timestamps.
hipError_t launch_predict_aug(int kind, int mp, const uint16_t* Bt, int64_t NPAD, const uint16_t* Aq, int64_t NQPAD,
                              const double* w, int nchunk, int bpc, double* part, hipStream_t s,
                              hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// Few queries (augmented rows): queries read and augmented by the kernel
// itself, weights formed from alpha and y; part[nchunk][NQPAD], wpart[nchunk].
int64_t predict_query_pad_small(int64_t nq);
void predict_chunks_small(int64_t NPAD, int64_t NQPAD, int* nchunk, int* bpc);
hipError_t launch_predict_small(int kind, int mp, const uint16_t* Bt, int64_t NPAD, const float* Xq, const double* mean,
                                int64_t nq, int64_t m, const double* alpha, const float* y, int64_t N, bool box,
                                double C, int64_t NQPAD, int nchunk, int bpc, double* part, double* wpart,
                                hipStream_t s, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
hipError_t launch_predict_reduce(const double* part, int nchunk, int64_t stride, int64_t nq, const double* wpart, int nw,
                                 double lam2, double* f, hipStream_t s);
// Results of a solve packed for one download: alpha, P~ (read with `stride`
// aggregates from one node to the next), A_ii as N doubles each, then the
// labels as N floats; order (optional): node r of the inputs goes to order[r].
hipError_t launch_pack_out(int prec, int64_t N, const double* alpha, const void* Pt, int stride, const double* Adiag,
                           const float* y, const int32_t* order, double* out, hipStream_t s);

}  // namespace gabp
