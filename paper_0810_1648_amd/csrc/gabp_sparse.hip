// Sparsified kernel (the closing discussion's route to millions of points):
// the message graph keeps the pairs with exp(-gamma d^2) >= tau, i.e.
// d^2 <= cut = -ln(tau) / gamma, with K'_ij = exp(-gamma d^2) + lambda^2 on
// them and no message on the others.  GaBP itself is unchanged (Algorithm 2
// with N(i) the kept neighbours); the pair records live in edge order.
//
// Build (every pair of the unpruned tiles is examined on MFMA, over rows
// augmented so that the Gram is -d^2 / 2):
//   k_sp_augment the A and B rows of the build;
//   k_sp_count  kept pairs i < j of every 32nd tile: an estimate that sizes
//               the fill's output;
//   k_sp_fill   per tile: keys (i << sh | j) and K' appended at a global
//               cursor (arbitrary order); a second pass runs only if the
//               estimate fell short;
//   radix sort of the keys: edges in (i, j) order, so every node's edges
//   with the node as i-end are contiguous; a second sort by (j, i) lists
//   each node's edges as j-end; k_sp_rows puts both ends of every node
//   together as its row (neighbour, K'), j-ends after i-ends.
// Sweep (Algorithm 2, synchronous, information form), by rows: a row's
// records are the messages INTO its node, so everything a node needs lies in
// its row except its neighbours' aggregates (k_sp_sweep).
#include "gabp_device.h"

#include <hipcub/hipcub.hpp>

namespace gabp {

namespace {

// Thresholded distances of the listed tiles tiles[p0, p1) on MFMA.  The rows
// are augmented (k_sp_augment): A row a_i = (x_i, n_i, 1), B row
// b_j = (x_j, -1/2, -n_j/2) with n = ||x||^2, so the Gram a_i . b_j is
// -d_ij^2 / 2 and the keep test d^2 <= cut is a single compare of the MFMA
// output with -cut / 2.  Wave w computes the 32-row bands w and w + 4 of a
// tile together (their A fragments in registers, reloaded only when the row
// block changes, each B fragment loaded once for both) and walks the
// tiles' 32-column blocks in order, the next block's B fragment (across
// tile boundaries too) in flight during the current MFMAs.  For every
// block, `visit(g0, g1, i0r, jcol, hc)` receives the Gram values of both
// bands, where the pair of register r of a lane is kept iff its value is
// >= hc = -cut / 2 (its ballot is the block's mask for that register).
// Blocks off the diagonal tile and before the last column hold only pairs
// i < j < N; in the others the pairs outside i < j < N get -inf first, so
// that the test stays one compare everywhere.
template <int KIND, int MP, class Visit>
__device__ inline void sp_tiles(const Features& FA, const Features& FB, const uint32_t* __restrict__ tiles,
                                int64_t p0, int64_t p1, int64_t N, float cut, Visit&& visit) {
    if (p0 >= p1) return;
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6, h = l >> 5, l32 = l & 31;
    const float hc = -0.5f * cut;
    auto coord = [&](int64_t p) {
        const uint32_t ij = tiles[p];
        return TileCoord{(int)(ij >> 16), (int)(ij & 0xFFFFu)};
    };
    // first column block with a pair i < j for the wave's lower band
    auto first_cb = [&](const TileCoord& t) {
        int c = 0;
        while (c < TILE / 32 && (int64_t)t.J * TILE + c * 32 + 31 < (int64_t)t.I * TILE + w * 32) ++c;
        return c;
    };
    int64_t p = p0;
    TileCoord tc = coord(p);
    int cb = first_cb(tc);
    RowFrag<KIND, MP> fa0, fa1, fb;
    fa0.load(FA, (int64_t)tc.I * TILE + w * 32 + l32);
    fa1.load(FA, (int64_t)tc.I * TILE + (w + 4) * 32 + l32);
    if constexpr (MP > 0) fb.load(FB, (int64_t)tc.J * TILE + cb * 32 + l32);
    while (true) {
        // the next (tile, block) of the walk
        int64_t pn = p;
        TileCoord tn = tc;
        int cbn = cb + 1;
        if (cbn == TILE / 32) {
            pn = p + 1;
            if (pn < p1) {
                tn = coord(pn);
                cbn = first_cb(tn);
            }
        }
        const bool more = pn < p1;
        const int64_t i0 = (int64_t)tc.I * TILE, j0 = (int64_t)tc.J * TILE;
        const int64_t rowA0 = i0 + w * 32 + l32, rowA1 = i0 + (w + 4) * 32 + l32;
        const int64_t j = j0 + cb * 32 + l32;
        f32x16 g0 = {}, g1 = {};
        if constexpr (MP > 0) {
            RowFrag<KIND, MP> fn;
            fn.load(FB, more ? (int64_t)tn.J * TILE + cbn * 32 + l32 : j);
            frag_mma(fa0, fb, g0, FA.m_pad);
            frag_mma(fa1, fb, g1, FA.m_pad);
            fb = fn;
        } else {
            RowFrag<KIND, MP>::gram2(fa0, fa1, FA, rowA0, rowA1, FB, j, g0, g1);
        }
        if (!((tc.I < tc.J) && (j0 + cb * 32 + 31 < N))) {
            // register r of lane l holds row 8 (r / 4) + 4 (l / 32) + r % 4 of its band
            const int64_t dj = j - (i0 + w * 32 + 4 * h);
            const bool jn = j < N;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int ro = 8 * (r >> 2) + (r & 3);
                if (!(jn && dj > ro)) g0[r] = -INFINITY;
                if (!(jn && dj > ro + 128)) g1[r] = -INFINITY;
            }
        }
        visit(g0, g1, i0 + w * 32, j, hc);
        if (!more) break;
        if (tn.I != tc.I) {
            fa0.load(FA, (int64_t)tn.I * TILE + w * 32 + l32);
            fa1.load(FA, (int64_t)tn.I * TILE + (w + 4) * 32 + l32);
        }
        p = pn;
        tc = tn;
        cb = cbn;
    }
}

// Kept pairs of every stride-th listed tile (stride 1: all of them), one
// count per launched tile; the host sums a strided sample to size the fill.
template <int KIND, int MP>
__global__ __launch_bounds__(WG) void k_sp_count(Features FA, Features FB, const uint32_t* __restrict__ tiles, int64_t stride,
                                                 int64_t N, float cut, int64_t* __restrict__ counts) {
    __shared__ int wsum[4];
    int c = 0;   // wave-uniform
    sp_tiles<KIND, MP>(FA, FB, tiles + (int64_t)blockIdx.x * stride, 0, 1, N, cut, [&](const f32x16& g0, const f32x16& g1, int64_t, int64_t, float hc) {
#pragma unroll
        for (int r = 0; r < 16; ++r) c += __popcll(__ballot(g0[r] >= hc)) + __popcll(__ballot(g1[r] >= hc));
    });
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

constexpr int SP_TPW = 16;   // listed tiles per workgroup of the fill

// Kept pairs appended at a global cursor.  A wave collects its kept pairs
// (key and K' value) in an LDS buffer, register by register in lane order;
// a full buffer is drained to slots reserved by one atomic, and at the end
// of its tiles one atomic reserves the slots of all four waves' remainders.
// The order across waves and tiles is arbitrary: the (i, j) sort that
// follows fixes it, and every pair's key and K' value do not depend on it.
// Slots at or beyond cap are not written but still counted, so the cursor
// ends at the exact number of kept pairs and the host repeats the pass with
// room for all of them.
template <int KIND, int MP>
__global__ __launch_bounds__(WG) void k_sp_fill(Features FA, Features FB, const uint32_t* __restrict__ tiles,
                                                int64_t ntiles, int64_t N,
                                                float cut, float neg_gamma_log2e, float lam2, int64_t cap,
                                                unsigned long long* __restrict__ cursor, int sh,
                                                uint64_t* __restrict__ keys, float* __restrict__ kv) {
    constexpr int BW = 512;   // entries buffered per wave
    __shared__ uint64_t bkey[4][BW];
    __shared__ float bval[4][BW];
    __shared__ unsigned long long wbase[4];
    __shared__ int wcnt[4];
    // SP_TPW consecutive listed tiles per workgroup (mostly one row block of a
    // super-block: the A fragments stay in registers)
    const int64_t p0 = xcd_contiguous(blockIdx.x, gridDim.x) * SP_TPW;
    const int64_t p1 = (p0 + SP_TPW < ntiles) ? p0 + SP_TPW : ntiles;
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6, h = l >> 5;
    const uint64_t below = (1ull << l) - 1ull;
    int n = 0;   // wave-uniform: entries in the wave's buffer
    // the wave's n buffered entries to slots base, base + 1, ...
    auto drain = [&](unsigned long long base) {
        for (int k = l; k < n; k += 64) {
            const int64_t slot = (int64_t)base + k;
            if (slot < cap) {
                keys[slot] = bkey[w][k];
                kv[slot] = bval[w][k];
            }
        }
    };
    sp_tiles<KIND, MP>(FA, FB, tiles, p0, p1, N, cut, [&](const f32x16& g0, const f32x16& g1, int64_t ib, int64_t j,
                                                          float hc) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float gv = half ? g1[r] : g0[r];
                const uint64_t mask = __ballot(gv >= hc);
                if (mask == 0) continue;
                if (n + 64 > BW) {
                    wave_lds_sync();
                    unsigned long long first = 0;
                    if (l == 0) first = atomicAdd(cursor, (unsigned long long)n);
                    drain(__shfl(first, 0));
                    n = 0;
                    wave_lds_sync();
                }
                if ((mask >> l) & 1ull) {
                    const int k = n + __popcll(mask & below);
                    const int64_t i = ib + 128 * half + 8 * (r >> 2) + 4 * h + (r & 3);
                    bkey[w][k] = ((uint64_t)i << sh) | (uint64_t)j;
                    bval[w][k] = __builtin_amdgcn_exp2f(neg_gamma_log2e * fmaxf(-2.0f * gv, 0.0f)) + lam2;
                }
                n += __popcll(mask);
            }
        }
    });
    if (l == 0) wcnt[w] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long c0 = wcnt[0], c1 = wcnt[1], c2 = wcnt[2], c3 = wcnt[3];
        const unsigned long long tot = c0 + c1 + c2 + c3;
        const unsigned long long b = tot ? atomicAdd(cursor, tot) : 0ull;
        wbase[0] = b;
        wbase[1] = b + c0;
        wbase[2] = b + c0 + c1;
        wbase[3] = b + c0 + c1 + c2;
    }
    __syncthreads();
    drain(wbase[w]);
}

// Ends of every edge in (i, j) order, and the keys of the (j, i) order.
__global__ void k_sp_unpack(const uint64_t* __restrict__ keys, int64_t E, int sh, int32_t* __restrict__ ei,
                            int32_t* __restrict__ ej, uint64_t* __restrict__ keys_t) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= E) return;
    const uint64_t k = keys[e];
    const int32_t i = (int32_t)(k >> sh), j = (int32_t)(k & ((1ull << sh) - 1ull));
    ei[e] = i;
    ej[e] = j;
    keys_t[e] = ((uint64_t)j << sh) | (uint64_t)i;
}

// off[k] = first position whose key's node (key >> sh) is >= k, k = 0 .. N, by
// bisection: a thread per position that fills the nodes up to its own leaves a
// run of points without edges to one lane (490,000 points, none with an edge:
// 24.5 of the 26.4 ms of their build).
__global__ void k_sp_offsets(const uint64_t* __restrict__ keys, int64_t E, int sh, int64_t N, int64_t* __restrict__ off) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k > N) return;
    int64_t lo = 0, hi = E;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if ((int64_t)(keys[mid] >> sh) < k) lo = mid + 1;
        else hi = mid;
    }
    off[k] = lo;
}

// Row lengths: a node's edges of both ends in whole quads, at least one.
__global__ void k_sp_rowlen(int64_t N, const int64_t* __restrict__ off_i, const int64_t* __restrict__ off_j,
                            int64_t* __restrict__ len) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k > N) return;
    const int64_t d = (k < N) ? (off_i[k + 1] - off_i[k]) + (off_j[k + 1] - off_j[k]) : 0;
    len[k] = (k < N) ? (d > 0 ? (d + 3) / 4 * 4 : 4) : 0;
}

// Rows (neighbour, K'): node k's row begins at row[k] with its i-end edges,
// then its j-end edges; its last quad is filled up with the node itself and
// K' = 0, whose messages are zero.  qrow names the node of every quad.
// Thread e places edge e of both orders; thread k < N fills row k's end and
// names its quads.
__global__ void k_sp_rows(int64_t E, int64_t N, int sh, const int32_t* __restrict__ ei, const int32_t* __restrict__ ej,
                          const float* __restrict__ kv, const uint64_t* __restrict__ keys_t,
                          const float* __restrict__ kv_t, const int64_t* __restrict__ off_i,
                          const int64_t* __restrict__ off_j, const int64_t* __restrict__ row, int32_t* __restrict__ col,
                          float* __restrict__ rkv, int32_t* __restrict__ qrow) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < E) {
        const int64_t i = ei[e], a = row[i] + (e - off_i[i]);
        col[a] = ej[e];
        rkv[a] = kv[e];
        const uint64_t k = keys_t[e];
        const int64_t j = (int64_t)(k >> sh), b = row[j] + (off_i[j + 1] - off_i[j]) + (e - off_j[j]);
        col[b] = (int32_t)(k & ((1ull << sh) - 1ull));
        rkv[b] = kv_t[e];
    }
    if (e < N) {
        for (int64_t a = row[e] / 4; a < row[e + 1] / 4; ++a) qrow[a] = (int32_t)e;
        for (int64_t a = row[e] + (off_i[e + 1] - off_i[e]) + (off_j[e + 1] - off_j[e]); a < row[e + 1]; ++a) {
            col[a] = (int32_t)e;
            rkv[a] = 0.0f;
        }
    }
}

// Row sums and maxima of K' over each node's row (the sparse r_i), written
// as one partial per node (the dense layout with a single slot); sixteen
// lanes per node as in k_sp_sweep.
__global__ __launch_bounds__(WG) void k_sp_rowsum(int64_t N, const int64_t* __restrict__ row,
                                                  const float* __restrict__ kv, double* __restrict__ psum,
                                                  double* __restrict__ pmax) {
    const int64_t k = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 4;
    const int q = threadIdx.x & 15;
    double s = 0.0, m = 0.0;
    if (k < N)
        for (int64_t e = row[k] + q, r1 = row[k + 1]; e < r1; e += 16) {
            s += (double)kv[e];
            m = fmax(m, (double)kv[e]);
        }
    s = sum16(s);
    m = fmax(m, dpp<0xB1>(m));
    m = fmax(m, dpp<0x4E>(m));
    m = fmax(m, dpp<0x141>(m));
    m = fmax(m, dpp<0x140>(m));
    if (k < N && q == 0) { psum[k] = s; pmax[k] = m; }
}

// Aggregates of every node packed as (P~, S) pairs, so that the sweep's
// reads of a random neighbour fetch one 8- or 16-byte item (the start of the
// solve; the sweeps write them packed).
template <class AT>
__global__ void k_sp_pack(int64_t N, const AT* __restrict__ Pt, const AT* __restrict__ S, AT* __restrict__ PS) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < N) { PS[2 * k] = Pt[k]; PS[2 * k + 1] = S[k]; }
}
constexpr int SP_MAXS = 256;   // slots of the sweep's change / magnitude maxima

// New aggregates and alpha of node k from the sums of its messages; d and am
// take its change and magnitude.  Returns false when the node diverged.
template <class AT>
__device__ inline bool sp_node(int64_t k, AT sp, AT se, const SparseSweep& a, AT* __restrict__ PS, double& d, double& am) {
    const double yk = (double)a.y[k];
    const AT p = (AT)a.Adiag[k] + sp;
    AT s = (AT)a.y[k] + se;
    double an = (double)(s / p) * yk;
    const bool ok = p > (AT)0 && isfinite((double)p) && isfinite((double)s);
    if (a.boxC > 0.0) {
        an = fmin(fmax(an, 0.0), a.boxC);
        s = p * (AT)(an * yk);
    }
    PS[2 * k] = p;
    PS[2 * k + 1] = s;
    d = fmax(d, fabs(an - a.alpha[k]));
    am = fmax(am, fabs(an));
    a.alpha[k] = an;
    return ok;
}

// Change and magnitude maxima of a workgroup into the sweep's slots by
// integer maximum (non-negative doubles order as their bits), which no order
// of arrival changes.
__device__ inline void sp_maxima(double d, double am, const SparseSweep& a) {
    __shared__ double sh4[4];
    d = block_max(d, sh4);
    am = block_max(am, sh4);
    if (threadIdx.x == 0) {
        atomicMax(reinterpret_cast<unsigned long long*>(a.dmax) + blockIdx.x % SP_MAXS,
                  (unsigned long long)__double_as_longlong(d));
        atomicMax(reinterpret_cast<unsigned long long*>(a.amax) + blockIdx.x % SP_MAXS,
                  (unsigned long long)__double_as_longlong(am));
    }
}

// Sweep t (1, 2, ...): workgroup w takes the quads [256 w, 256 w + 256) of
// the rows, one per thread, whatever rows they belong to (degrees spread over
// three decades, and sixteen lanes per row left most of them waiting for the
// longest row: 2.3 ms per sweep at 90.8 M edges).
//
// The message j -> k of sweep t needs the reverse message k -> j of sweep
// t - 1, which lies in the row of j; but k -> j of sweep t - 1 follows from
// node k's own aggregates of sweep t - 2 and the message j -> k of sweep
// t - 2, which lies here.  So each row keeps the messages into its node by
// the parity of the sweep (rec: those of sweep t - 2, overwritten with sweep
// t's), and nothing is scattered or gathered but the neighbours' packed
// aggregates: 25 bytes per directed edge in row order and one 16-byte read
// that the locality order keeps in L2.  With q = P~_k - P_jk of the older
// pair (checked as the reverse message's own cavity one sweep earlier) and
// h = a / q, the reverse message is P_kj = -a h, E_kj = -h (S_k - E_jk), and
//   P_jk = -a^2 / Q,  E_jk = -a (S_j + h (S_k - E_jk)) / Q,  Q = P~_j + a h.
// (Both follow from the one reciprocal of Q q as well, but its products a^2 q
// and P~_j q leave the range of FP32 at entries of 1e12, a^2 only at 1e19;
// the second reciprocal costs nothing beside the neighbours' reads.)
// (Records per edge updated by one thread and gathered by node through a
// permutation moved 12.1 GB per sweep at 90.8 M edges, 2.63 ms with their five
// launches; this is 4.5 GB and 1.75 ms, 0.65 of them the neighbours' reads.
// At 3.65 M edges 101 -> 69 us.)
// FIRST: sweep 1, whose reverse messages are zero.  Sweep 2's older messages
// are those of sweep 0, zero too.
//
// The quads' sums meet in LDS: sixteen lanes add a row's quads in a fixed
// tree, one thread per row forms its node.  A row that leaves the workgroup's
// range puts its sum into the workgroup's head (begun earlier) or tail slot
// of `edge` for k_sp_join.
template <class ST, class MT, class AT, bool FIRST>
__global__ __launch_bounds__(WG) void k_sp_sweep(SparseSweep a, int t) {
    if (a.st->done) return;
    typedef ST Rec2 __attribute__((ext_vector_type(4)));          // two records
    typedef int32_t Int4 __attribute__((ext_vector_type(4)));
    typedef AT AggT __attribute__((ext_vector_type(2)));
    __shared__ AT qP[WG], qE[WG], rowP[WG], rowE[WG];
    const int par = t & 1, tid = threadIdx.x;
    const AggT* const A1 = static_cast<const AggT*>(a.PS[par ^ 1]);
    AT* const PS2 = static_cast<AT*>(a.PS[par]);
    const int64_t w = xcd_contiguous(blockIdx.x, gridDim.x), q0 = w * WG;
    const int nq = (int)(a.nq - q0 < WG ? a.nq - q0 : WG);
    const int ra = a.qrow[q0], rb = a.qrow[q0 + nq - 1];          // first and last row here
    bool bad = false;
    if (tid < nq) {
        const int64_t e = q0 + tid;
        const int k = a.qrow[e];
        const Int4 c = reinterpret_cast<const Int4*>(a.col)[e];
        const f32x4v kk = reinterpret_cast<const f32x4v*>(a.kv)[e];
        Rec2* const R = static_cast<Rec2*>(a.rec[par]) + 2 * e;
        Rec2 old[2] = {Rec2{0, 0, 0, 0}, Rec2{0, 0, 0, 0}}, m[2];
        MT Pk = 1, Sk = 0;
        if (!FIRST) {
            // the node's own aggregates of sweep t - 2
            const AggT own = *reinterpret_cast<const AggT*>(PS2 + 2 * (int64_t)k);
            Pk = (MT)own[0];
            Sk = (MT)own[1];
            if (t > 2) { old[0] = R[0]; old[1] = R[1]; }
        }
        AggT g[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) g[u] = A1[c[u]];
        AT sp = 0, se = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const MT av = (MT)kk[u], a2 = av * av;
            MT d = (MT)g[u][0], x = (MT)g[u][1];
            if (!FIRST) {
                const MT h = av * rcp_pos(Pk - (MT)old[u / 2][2 * (u & 1)]);
                d = fma(av, h, d);
                x = fma(h, Sk - (MT)old[u / 2][2 * (u & 1) + 1], x);
            }
            bad |= !(d > (MT)0);
            const MT r = rcp_pos(d);
            const ST mp = (ST)(-a2 * r), me = (ST)(-(av * x) * r);
            m[u / 2][2 * (u & 1)] = mp;
            m[u / 2][2 * (u & 1) + 1] = me;
            sp += (AT)mp;
            se += (AT)me;
        }
        R[0] = m[0];
        R[1] = m[1];
        qP[tid] = sp;
        qE[tid] = se;
    }
    __syncthreads();
    const int q = tid & 15;
    for (int r = ra + (tid >> 4); r <= rb; r += WG / 16) {
        const int64_t b = a.row[r] / 4 - q0, e = a.row[r + 1] / 4 - q0;
        const int lo = b > 0 ? (int)b : 0, hi = e < nq ? (int)e : nq;
        AT sp = 0, se = 0;
        for (int x = lo + q; x < hi; x += 16) { sp += qP[x]; se += qE[x]; }
        sp = sum16(sp);
        se = sum16(se);
        if (q == 0) { rowP[r - ra] = sp; rowE[r - ra] = se; }
    }
    __syncthreads();
    double d = 0.0, am = 0.0;
    if (tid <= rb - ra) {
        const int r = ra + tid;
        const bool head = a.row[r] / 4 < q0, tail = a.row[r + 1] / 4 > q0 + nq;
        if (head || tail) {
            AT* const o = static_cast<AT*>(a.edge) + 4 * w + (head ? 0 : 2);
            o[0] = rowP[tid];
            o[1] = rowE[tid];
        } else {
            bad |= !sp_node<AT>(r, rowP[tid], rowE[tid], a, PS2, d, am);
        }
    }
    if (__any(bad) && (tid & 63) == 0) a.st->bad = 1;
    sp_maxima(d, am, a);
}

// The rows that cross workgroup ranges of k_sp_sweep: thread w takes the row
// that begins in range w and leaves it, adding the tail of w and the heads of
// the ranges after it in order.  The workgroup that takes the last ticket
// applies the stop rule (as in k_finalize) and clears the maxima for the
// next sweep.
template <class AT>
__global__ __launch_bounds__(WG) void k_sp_join(SparseSweep a, int t) {
    if (a.st->done) return;
    __shared__ int last;
    const int64_t w = (int64_t)blockIdx.x * WG + threadIdx.x, nw = (a.nq + WG - 1) / WG;
    double d = 0.0, am = 0.0;
    bool bad = false;
    if (w + 1 < nw) {
        const int r = a.qrow[w * WG + WG - 1];
        const int64_t b = a.row[r] / 4, e = a.row[r + 1] / 4;
        if (b >= w * WG && e > (w + 1) * WG) {
            const AT* const x = static_cast<const AT*>(a.edge);
            AT sp = x[4 * w + 2], se = x[4 * w + 3];
            for (int64_t v = w + 1; v * WG < e; ++v) { sp += x[4 * v]; se += x[4 * v + 1]; }
            bad = !sp_node<AT>(r, sp, se, a, static_cast<AT*>(a.PS[t & 1]), d, am);
        }
    }
    if (__any(bad) && (threadIdx.x & 63) == 0) store_agent(&a.st->bad, 1);
    sp_maxima(d, am, a);
    wait_vm<0>();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&a.st->ticket, 1u) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    if (threadIdx.x == 0) a.st->ticket = 0;
    status_update(SP_MAXS, a.dmax, a.amax, a.st, a.trace, a.rule);
    a.dmax[threadIdx.x] = 0.0;
    a.amax[threadIdx.x] = 0.0;
}
static_assert(SP_MAXS == WG, "one slot per thread");

// ---- locality order and tile pruning
//
// Points are reordered so that each 256-point block is compact: every point
// goes to its nearest landmark (landmarks: K evenly spaced input points;
// ties to the smaller landmark index) and points are sorted by (landmark,
// input index).  Then a tile whose blocks are provably farther apart than
// the cut is skipped by the build (triangle inequality on block centroids
// and radii), and the neighbours of a node sit in few cache lines during the
// sweep.  GaBP is equivariant under the relabelling; results are returned in
// input order.

// Nearest landmark of every point by direct FP32 differences; landmarks are
// staged through LDS in chunks.  key = (landmark << 32) | point.
__global__ __launch_bounds__(WG) void k_sp_assign(const float* __restrict__ X, int64_t N, int64_t m,
                                                  const int32_t* __restrict__ lm, int K, uint64_t* __restrict__ key,
                                                  int32_t* __restrict__ ids) {
    extern __shared__ float sl[];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int chunk = (int)(8192 / m) > 0 ? (int)(8192 / m) : 1;
    float best = INFINITY;
    int arg = 0;
    for (int k0 = 0; k0 < K; k0 += chunk) {
        const int kc = (K - k0 < chunk) ? K - k0 : chunk;
        __syncthreads();
        for (int64_t t = threadIdx.x; t < (int64_t)kc * m; t += blockDim.x)
            sl[t] = X[(int64_t)lm[k0 + t / m] * m + t % m];
        __syncthreads();
        if (i < N) {
            for (int k = 0; k < kc; ++k) {
                float d2 = 0.0f;
                for (int64_t c = 0; c < m; ++c) {
                    const float d = X[i * m + c] - sl[(int64_t)k * m + c];
                    d2 = fmaf(d, d, d2);
                }
                if (d2 < best) { best = d2; arg = k0 + k; }
            }
        }
    }
    if (i < N) {
        key[i] = ((uint64_t)(uint32_t)arg << 32) | (uint64_t)i;
        ids[i] = (int32_t)i;
    }
}

// The same for rows of up to MR features: a thread keeps its point's row in
// registers (the general kernel reads it from memory once per landmark, lanes a
// row apart, and that bounds it) and takes four landmarks at a time, whose LDS
// reads are broadcasts.  Features beyond m are zero in both, so every
// distance has the general kernel's bits.  200,000 points of 20 features against
// 97 landmarks 1.08 -> 0.042 ms.
template <int MR>
__global__ __launch_bounds__(WG) void k_sp_assign_reg(const float* __restrict__ X, int64_t N, int m,
                                                      const int32_t* __restrict__ lm, int K,
                                                      uint64_t* __restrict__ key, int32_t* __restrict__ ids) {
    constexpr int CH = 8192 / MR, Q = MR / 4;
    __shared__ float4 sl[CH * Q];
    float* sf = reinterpret_cast<float*>(sl);
    const int64_t i = (int64_t)blockIdx.x * WG + threadIdx.x;
    float x[MR];
#pragma unroll
    for (int c = 0; c < MR; ++c) x[c] = (i < N && c < m) ? X[i * m + c] : 0.0f;
    float best = INFINITY;
    int arg = 0;
    for (int k0 = 0; k0 < K; k0 += CH) {
        const int kc = (K - k0 < CH) ? K - k0 : CH;
        __syncthreads();
        for (int t = threadIdx.x; t < kc * MR; t += WG) {
            const int c = t % MR;
            sf[t] = c < m ? X[(int64_t)lm[k0 + t / MR] * m + c] : 0.0f;
        }
        __syncthreads();
        auto dist = [&](int k, auto& d2) {
            constexpr int U = sizeof(d2) / sizeof(float);
#pragma unroll
            for (int c = 0; c < Q; ++c)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float4 v = sl[(k + u) * Q + c];
                    const float d0 = x[4 * c] - v.x, d1 = x[4 * c + 1] - v.y;
                    const float d2c = x[4 * c + 2] - v.z, d3 = x[4 * c + 3] - v.w;
                    d2[u] = fmaf(d3, d3, fmaf(d2c, d2c, fmaf(d1, d1, fmaf(d0, d0, d2[u]))));
                }
        };
        int k = 0;
        for (; k + 4 <= kc; k += 4) {
            float d2[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            dist(k, d2);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (d2[u] < best) { best = d2[u]; arg = k0 + k + u; }
        }
        for (; k < kc; ++k) {
            float d2[1] = {0.0f};
            dist(k, d2);
            if (d2[0] < best) { best = d2[0]; arg = k0 + k; }
        }
    }
    if (i < N) {
        key[i] = ((uint64_t)(uint32_t)arg << 32) | (uint64_t)i;
        ids[i] = (int32_t)i;
    }
}

// Super-blocked order of the tile list: key = (super-block of (I, J), tile
// code), super-blocks of S x S tiles in row-major order, tiles inside one in
// row-major order.  With the XCD-contiguous workgroup index, the tiles of a
// super-block run on one XCD and share its L2 for their 2 S row fragments.
__global__ void k_sp_tile_keys(const uint32_t* __restrict__ tiles, int64_t nt, int S, int NSB,
                               uint64_t* __restrict__ keys) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    const uint32_t ij = tiles[t];
    const uint32_t I = ij >> 16, J = ij & 0xFFFFu;
    keys[t] = ((uint64_t)((I / S) * (uint32_t)NSB + J / S) << 32) | (uint64_t)ij;
}

__global__ void k_sp_tile_codes(const uint64_t* __restrict__ keys, int64_t nt, uint32_t* __restrict__ tiles) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < nt) tiles[t] = (uint32_t)(keys[t] & 0xFFFFFFFFull);
}

// Rows of X and labels in the new order: Xp[r] = X[order[r]].
__global__ void k_sp_permute(const float* __restrict__ X, const float* __restrict__ y, int64_t N, int64_t m,
                             const int32_t* __restrict__ order, float* __restrict__ Xp, float* __restrict__ yp) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N * m) return;
    const int64_t r = t / m, c = t % m;
    Xp[t] = X[(int64_t)order[r] * m + c];
    if (c == 0) yp[r] = y[order[r]];
}

// Centroid (FP64) and radius (max distance to it, FP64) of each block of
// 256 reordered points; one workgroup per block.
__global__ __launch_bounds__(WG) void k_sp_block_bounds(const float* __restrict__ Xp, int64_t N, int64_t m,
                                                        double* __restrict__ cent, double* __restrict__ rad) {
    __shared__ double sh[WG];
    __shared__ double sh4[4];
    const int64_t b = blockIdx.x;
    const int64_t r0 = b * TILE;
    const int64_t nr = (N - r0 < TILE) ? N - r0 : TILE;
    for (int64_t c = 0; c < m; ++c) {
        double v = (threadIdx.x < nr) ? (double)Xp[(r0 + threadIdx.x) * m + c] : 0.0;
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int o = WG / 2; o > 0; o >>= 1) {
            if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
            __syncthreads();
        }
        if (threadIdx.x == 0) cent[b * m + c] = sh[0] / (double)nr;
        __syncthreads();
    }
    double d2 = 0.0;
    if (threadIdx.x < nr)
        for (int64_t c = 0; c < m; ++c) {
            const double d = (double)Xp[(r0 + threadIdx.x) * m + c] - cent[b * m + c];
            d2 += d * d;
        }
    d2 = block_max(threadIdx.x < nr ? d2 : 0.0, sh4);
    if (threadIdx.x == 0) rad[b] = sqrt(d2);
}

// keep[t] = 1 unless every pair of tile t is provably beyond the cut:
// ||x_i - x_j|| >= ||c_I - c_J|| - r_I - r_J.  The margin makes the test
// conservative against the rounding of the bounds and of the device's own
// distances (a skipped pair has d^2 > 1.001 cut).
__global__ void k_sp_prune(const uint32_t* __restrict__ tiles, int64_t nt, int64_t m, const double* __restrict__ cent,
                           const double* __restrict__ rad, double cut, uint8_t* __restrict__ keep) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nt) return;
    const uint32_t ij = tiles[t];
    const int I = (int)(ij >> 16), J = (int)(ij & 0xFFFFu);
    double dc2 = 0.0;
    for (int64_t c = 0; c < m; ++c) {
        const double d = cent[(int64_t)I * m + c] - cent[(int64_t)J * m + c];
        dc2 += d * d;
    }
    const double gap = sqrt(dc2) - (rad[I] + rad[J]) * (1.0 + 1e-6) - 1e-6;
    keep[t] = (gap > 0.0 && gap * gap > 1.001 * cut) ? 0 : 1;
}

// Augmented rows of the build: A row i gets (n_i, 1) in columns m, m + 1,
// B row i (a copy of A's first m columns) gets (-1/2, -n_i/2), each value
// split into the Gram kind's planes as the features are (hi, then the BF16
// remainders), so that sum_k a_ik b_jk = x_i . x_j - n_i/2 - n_j/2 for the
// products the kind forms.  Columns past m + 1 stay 0.  One thread per value,
// so that accesses are contiguous (a thread per row: 327 us, a thread per value 31 us
// for 200,000 rows), 2^30 threads at most: a launch holds fewer than 2^32, and the
// largest staged matrices have more values.
__global__ void k_sp_augment(int64_t NPAD, int m, int m_pad, int kind, const float* __restrict__ nrm,
                             float* f32a, uint16_t* hia, uint16_t* loa, uint16_t* lo2a, float* f32b,
                             uint16_t* hib, uint16_t* lob, uint16_t* lo2b) {
    const bool x3 = (kind == GRAM_BF16X3 || kind == GRAM_BF16X6), x6 = (kind == GRAM_BF16X6);
    for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < NPAD * m_pad;
         o += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = o / m_pad;
        const int k = (int)(o - i * m_pad);
        const float n = nrm[i];
        // (A's value where it is not a feature, B's)
        const float va = k == m ? n : 1.0f, vb = k == m ? -0.5f : k == m + 1 ? -0.5f * n : 0.0f;
        const bool extra = k == m || k == m + 1;
        if (kind == GRAM_F32) {
            if (extra) f32a[o] = va;
            f32b[o] = k < m ? f32a[o] : vb;
            continue;
        }
        uint16_t h, l, l2;
        split3(vb, h, l, l2);
        hib[o] = k < m ? hia[o] : h;
        if (x3) lob[o] = k < m ? loa[o] : l;
        if (x6) lo2b[o] = k < m ? lo2a[o] : l2;
        if (!extra) continue;
        split3(va, h, l, l2);
        hia[o] = h;
        if (x3) loa[o] = l;
        if (x6) lo2a[o] = l2;
    }
}

template <int KIND>
void sp_build_kind(bool fill, int mp, dim3 g, const Features& FA, const Features& FB, const uint32_t* tiles, int64_t stride, int64_t N,
                   float cut, float c, float lam2, int64_t* counts, int64_t cap, unsigned long long* cursor, int sh,
                   uint64_t* keys, float* kv, hipStream_t s) {
    const dim3 gf((unsigned)(((int64_t)g.x + SP_TPW - 1) / SP_TPW));
#define GABP_SP_LAUNCH(MPV)                                                                                  \
    do {                                                                                                     \
        if (fill)                                                                                            \
            hipLaunchKernelGGL((k_sp_fill<KIND, MPV>), gf, dim3(WG), 0, s, FA, FB, tiles, (int64_t)g.x, N, cut,   \
                               c, lam2, cap, cursor, sh, keys, kv);                                          \
        else                                                                                                 \
            hipLaunchKernelGGL((k_sp_count<KIND, MPV>), g, dim3(WG), 0, s, FA, FB, tiles, stride, N, cut,     \
                               counts);                                                                      \
    } while (0)
    // register-held fragments of two bands plus the prefetched B fragment
    // fit up to 64 features; beyond, fragments are reloaded per block
    if (mp <= 32) GABP_SP_LAUNCH(32);
    else if (mp <= 64) GABP_SP_LAUNCH(64);
    else GABP_SP_LAUNCH(0);
#undef GABP_SP_LAUNCH
}

hipError_t sp_build(bool fill, const Features& FA, const Features& FB, const uint32_t* tiles, int64_t ntiles,
                    int64_t stride, int64_t N, float cut, float c, float lam2, int64_t* counts, int64_t cap,
                    unsigned long long* cursor, int sh, uint64_t* keys, float* kv, hipStream_t s) {
    const dim3 g((unsigned)ntiles);
#define GABP_SP_KIND(K) sp_build_kind<K>(fill, FA.m_pad, g, FA, FB, tiles, stride, N, cut, c, lam2, counts, cap, cursor, sh, keys, kv, s)
    switch (FA.kind) {
        case GRAM_F32: GABP_SP_KIND(GRAM_F32); break;
        case GRAM_BF16: GABP_SP_KIND(GRAM_BF16); break;
        case GRAM_BF16X3: GABP_SP_KIND(GRAM_BF16X3); break;
        case GRAM_BF16X6: GABP_SP_KIND(GRAM_BF16X6); break;
        default: return hipErrorInvalidValue;
    }
#undef GABP_SP_KIND
    return hipGetLastError();
}

inline unsigned blocks(int64_t n) { return (unsigned)((n + WG - 1) / WG); }

}  // namespace

hipError_t launch_sp_count(const Features& FA, const Features& FB, const uint32_t* tiles, int64_t ntiles,
                           int64_t stride, int64_t N, float cut, int64_t* counts, hipStream_t s) {
    return in_launches(ntiles, [&](int64_t o, int64_t n) {
        return sp_build(false, FA, FB, tiles + o * stride, n, stride, N, cut, 0.0f, 0.0f, counts + o, 0, nullptr, 0,
                        nullptr, nullptr, s);
    });
}

hipError_t launch_sp_fill(const Features& FA, const Features& FB, const uint32_t* tiles, int64_t ntiles, int64_t N,
                          float cut, float neg_gamma_log2e, float lam2, int64_t cap, unsigned long long* cursor, int sh,
                          uint64_t* keys, float* kv, hipStream_t s) {
    // (kMaxBlocks tiles at a time, whose workgroups take SP_TPW each)
    return in_launches(ntiles, [&](int64_t o, int64_t n) {
        return sp_build(true, FA, FB, tiles + o, n, 1, N, cut, neg_gamma_log2e, lam2, nullptr, cap, cursor, sh, keys,
                        kv, s);
    });
}

hipError_t launch_sp_augment(int64_t NPAD, int64_t m, int m_pad, int kind, const float* nrm, float* f32a,
                             uint16_t* hia, uint16_t* loa, uint16_t* lo2a, float* f32b, uint16_t* hib,
                             uint16_t* lob, uint16_t* lo2b, hipStream_t s) {
    if (m + 2 > m_pad) return hipErrorInvalidValue;
    const unsigned g = blocks(std::min<int64_t>(NPAD * m_pad, (int64_t)1 << 30));
    hipLaunchKernelGGL(k_sp_augment, dim3(g), dim3(WG), 0, s, NPAD, (int)m, m_pad, kind, nrm, f32a, hia, loa, lo2a,
                       f32b, hib, lob, lo2b);
    return hipGetLastError();
}

hipError_t launch_sp_order(const float* X, int64_t N, int64_t m, const int32_t* lm, int K, uint64_t* key,
                           int32_t* ids, hipStream_t s) {
    // rows of up to 64 features fit the registers; beyond, from memory
#define GABP_ASSIGN(MR_) \
    if (m <= MR_) { \
        hipLaunchKernelGGL(k_sp_assign_reg<MR_>, dim3(blocks(N)), dim3(WG), 0, s, X, N, (int)m, lm, K, key, ids); \
        return hipGetLastError(); \
    }
    GABP_ASSIGN(8)
    GABP_ASSIGN(16)
    GABP_ASSIGN(24)
    GABP_ASSIGN(32)
    GABP_ASSIGN(64)
#undef GABP_ASSIGN
    const int chunk = (int)(8192 / m) > 0 ? (int)(8192 / m) : 1;
    const size_t lds = (size_t)std::min<int64_t>(chunk, K) * m * sizeof(float);
    hipLaunchKernelGGL(k_sp_assign, dim3(blocks(N)), dim3(WG), lds, s, X, N, m, lm, K, key, ids);
    return hipGetLastError();
}

hipError_t launch_sp_permute(const float* X, const float* y, int64_t N, int64_t m, const int32_t* order, float* Xp,
                             float* yp, hipStream_t s) {
    hipLaunchKernelGGL(k_sp_permute, dim3(blocks(N * m)), dim3(WG), 0, s, X, y, N, m, order, Xp, yp);
    return hipGetLastError();
}

hipError_t launch_sp_prune(const float* Xp, int64_t N, int64_t m, int NB, const uint32_t* tiles, int64_t nt,
                           double cut, double* cent, double* rad, uint8_t* keep, hipStream_t s) {
    hipLaunchKernelGGL(k_sp_block_bounds, dim3((unsigned)NB), dim3(WG), 0, s, Xp, N, m, cent, rad);
    hipLaunchKernelGGL(k_sp_prune, dim3(blocks(nt)), dim3(WG), 0, s, tiles, nt, m, cent, rad, cut, keep);
    return hipGetLastError();
}

hipError_t sp_select(void* tmp, size_t* bytes, const uint32_t* in, const uint8_t* flags, uint32_t* out,
                     int64_t* nsel, int64_t n, hipStream_t s) {
    return hipcub::DeviceSelect::Flagged(tmp, *bytes, in, flags, out, nsel, (int)n, s);
}

hipError_t sp_tile_order(void* tmp, size_t* bytes, uint32_t* tiles, int64_t nt, int S, int NB, uint64_t* k0,
                         uint64_t* k1, hipStream_t s) {
    if (tmp == nullptr) return hipcub::DeviceRadixSort::SortKeys(tmp, *bytes, k0, k1, (int)nt, 0, 64, s);
    if (nt <= 0) return hipSuccess;
    const int NSB = (NB + S - 1) / S;
    hipLaunchKernelGGL(k_sp_tile_keys, dim3(blocks(nt)), dim3(WG), 0, s, tiles, nt, S, NSB, k0);
    hipError_t e = hipcub::DeviceRadixSort::SortKeys(tmp, *bytes, k0, k1, (int)nt, 0, 64, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sp_tile_codes, dim3(blocks(nt)), dim3(WG), 0, s, k1, nt, tiles);
    return hipGetLastError();
}

hipError_t sp_scan(void* tmp, size_t* bytes, const int64_t* in, int64_t* out, int64_t n, hipStream_t s) {
    return hipcub::DeviceScan::ExclusiveSum(tmp, *bytes, in, out, (int)n, s);
}

hipError_t sp_sort_keys(void* tmp, size_t* bytes, const uint64_t* kin, uint64_t* kout, const float* vin,
                        float* vout, int64_t n, int bits, hipStream_t s) {
    return hipcub::DeviceRadixSort::SortPairs(tmp, *bytes, kin, kout, vin, vout, (int)n, 0, bits, s);
}

hipError_t sp_sort_ids(void* tmp, size_t* bytes, const uint64_t* kin, uint64_t* kout, const int32_t* vin,
                       int32_t* vout, int64_t n, hipStream_t s) {
    return hipcub::DeviceRadixSort::SortPairs(tmp, *bytes, kin, kout, vin, vout, (int)n, 0, 64, s);
}

hipError_t launch_sp_unpack(const uint64_t* keys, int64_t E, int sh, int32_t* ei, int32_t* ej, uint64_t* keys_t,
                            hipStream_t s) {
    if (E > 0) hipLaunchKernelGGL(k_sp_unpack, dim3(blocks(E)), dim3(WG), 0, s, keys, E, sh, ei, ej, keys_t);
    return hipGetLastError();
}

hipError_t launch_sp_offsets(const uint64_t* keys, int64_t E, int sh, int64_t N, int64_t* off, hipStream_t s) {
    hipLaunchKernelGGL(k_sp_offsets, dim3(blocks(N + 1)), dim3(WG), 0, s, keys, E, sh, N, off);
    return hipGetLastError();
}

hipError_t launch_sp_rowlen(int64_t N, const int64_t* off_i, const int64_t* off_j, int64_t* len, hipStream_t s) {
    hipLaunchKernelGGL(k_sp_rowlen, dim3(blocks(N + 1)), dim3(WG), 0, s, N, off_i, off_j, len);
    return hipGetLastError();
}

hipError_t launch_sp_rows(int64_t E, int64_t N, int sh, const int32_t* ei, const int32_t* ej, const float* kv,
                          const uint64_t* keys_t, const float* kv_t, const int64_t* off_i, const int64_t* off_j,
                          const int64_t* row, int32_t* col, float* rkv, int32_t* qrow, hipStream_t s) {
    hipLaunchKernelGGL(k_sp_rows, dim3(blocks(std::max(E, N))), dim3(WG), 0, s, E, N, sh, ei, ej, kv, keys_t, kv_t,
                       off_i, off_j, row, col, rkv, qrow);
    return hipGetLastError();
}

hipError_t launch_sp_rowsum(int64_t N, const int64_t* row, const float* kv, double* psum, double* pmax, hipStream_t s) {
    hipLaunchKernelGGL(k_sp_rowsum, dim3(blocks(16 * N)), dim3(WG), 0, s, N, row, kv, psum, pmax);
    return hipGetLastError();
}

hipError_t launch_sp_pack(int prec, int64_t N, const void* Pt, const void* S, void* PS, hipStream_t s) {
    if (prec == PREC_FP32)
        hipLaunchKernelGGL(k_sp_pack<float>, dim3(blocks(N)), dim3(WG), 0, s, N, (const float*)Pt, (const float*)S,
                           (float*)PS);
    else
        hipLaunchKernelGGL(k_sp_pack<double>, dim3(blocks(N)), dim3(WG), 0, s, N, (const double*)Pt, (const double*)S,
                           (double*)PS);
    return hipGetLastError();
}

hipError_t launch_sp_sweep(int prec, const SparseSweep& a, int t, hipStream_t s) {
    if (t < 1 || a.nq < 1) return hipErrorInvalidValue;
    const dim3 g(blocks(a.nq)), j(blocks((a.nq + WG - 1) / WG)), b(WG);
    auto run = [&](auto first, auto later, auto join) {
        hipLaunchKernelGGL(t == 1 ? first : later, g, b, 0, s, a, t);
        hipLaunchKernelGGL(join, j, b, 0, s, a, t);
        return hipGetLastError();
    };
    switch (prec) {
        case PREC_FP32:
            return run(k_sp_sweep<float, float, float, true>, k_sp_sweep<float, float, float, false>, k_sp_join<float>);
        case PREC_MIXED:
            return run(k_sp_sweep<float, double, double, true>, k_sp_sweep<float, double, double, false>,
                       k_sp_join<double>);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace gabp
