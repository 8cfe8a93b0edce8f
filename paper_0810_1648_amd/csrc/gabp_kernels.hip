// HIP kernels of the GaBP SVM solver for gfx950 (MI355X).
//
// Method: Bickson, Yom-Tov, Dolev, arXiv 0810.1648.  The sweep is Algorithm
// 2 (section "Algorithm Optimization") in synchronous rounds (section
// "Experimental Results"), with messages kept in information form
// E_ij = P_ij mu_ij:
//     Q_ij = P~_i - P_ji,   P_ij <- -A_ij^2 / Q_ij,   E_ij <- -A_ij (S_i - E_ji) / Q_ij,
//     P~_j = A_jj + sum_i P_ij,   S_j = b_j + sum_i E_ij,   mu_j = S_j / P~_j.
// Labels are folded into the right-hand side: with Y = diag(y), A = Y(K'+W)Y,
// so GaBP on (K' + W, b = y) yields the same iterates up to exact sign flips
// and alpha = y * mu.  The kernels therefore never multiply by labels.
//
// Data layout: the unordered pairs {i, j}, i < j, live in TILE x TILE tiles of
// the upper triangle, row-major inside a tile.  Pair-record planes keep both
// directions of a pair at the same offset (P_ij, P_ji, E_ij, E_ji), so the
// update of a pair reads and writes one position of five planes with no
// transpose.  Entries below the diagonal of diagonal tiles and entries of
// padded rows/columns hold K' = 0, which makes their messages exactly zero.
//
// Lane layout of the streaming kernels: a workgroup (4 wave64) owns one tile;
// wave w owns the 64-column strip [64w, 64w + 64); in step s, lane (g, q) =
// (lane / 16, lane % 16) handles row 4s + g and the four columns
// 64w + 4q .. 64w + 4q + 3, so each plane access of a wave is four 256-byte
// contiguous segments of 16-byte loads.  Row sums (messages received by the
// row node) are reduced over 16 lanes with DPP; column sums (messages
// received by the column node) accumulate in registers and are combined
// across the four lane groups once per tile.  Partial sums go to a
// [block][slot][TILE] array that a second kernel reduces in a fixed order,
// so results are bitwise reproducible.
//
// K' comes either from the materialised plane (one 16-byte load per lane
// and row) or is recomputed per 32-row band: each wave forms the Gram
// products of its 32 x 64 block on MFMA, applies exp, and passes the block
// through a wave-private LDS buffer into the row layout above.  Messages come
// either from the pair-record planes (stored edge state) or are rebuilt from
// a ring of earlier aggregates (stateless edge state): the message i -> j of
// sweep t needs only the reverse message of sweep t - 1, which needs i -> j
// of sweep t - 2, and so on, so unrolling L levels from zero reproduces the
// stored recursion exactly while t <= L and truncates it after.
#include "gabp_device.h"

namespace gabp {

// ------------------------------------------------------- setup kernels --

__global__ void k_fill_tiles(uint32_t* tiles, int NB) {
    const int I = blockIdx.x;
    for (int J = I + threadIdx.x; J < NB; J += blockDim.x)
        tiles[tile_index(I, J, NB)] = ((uint32_t)I << 16) | (uint32_t)J;
}

__global__ void k_validate(const float* __restrict__ X, const float* __restrict__ y, int64_t N,
                           int64_t m, int32_t* flag) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int bad = 0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < N * m; k += stride)
        if (!isfinite(X[k])) bad |= 1;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < N; k += stride)
        if (!(y[k] == 1.0f || y[k] == -1.0f)) bad |= 2;
    if (bad) atomicOr(flag, bad);
}

// Column means in FP64 (the RBF kernel is translation invariant, so
// centring is exact math; it shrinks ||x||^2 before the Gram expansion).
__global__ void k_colmean(const float* __restrict__ X, int64_t N, int64_t m, double* mean) {
    __shared__ double sh[WG];
    const int64_t k = blockIdx.x;
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < N; i += WG) acc += (double)X[i * m + k];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = WG / 2; o > 0; o >>= 1) {
        if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) mean[k] = sh[0] / (double)N;
}

// Staged rows: zero padded, and the squared norm computed from the values
// actually staged (so that d^2 of a point with itself is 0 up to the Gram's
// own rounding).  A workgroup takes 64 rows, 32 columns at a time through LDS,
// so that reads and writes are contiguous; the norms are one FMA chain per row
// in column order, by the first 64 threads (one thread per row doing all of it
// took 283 us for 100,000 rows of 54 features and 46 us for 10,007 of 100).
__global__ __launch_bounds__(WG) void k_stage(const float* __restrict__ X, const double* __restrict__ mean, int64_t N,
                                              int64_t m, int64_t NPAD, int m_pad, int kind, float* f32, uint16_t* hi,
                                              uint16_t* lo, uint16_t* lo2, double* f64, float* nrm) {
    constexpr int RW = 64, CW = 32;
    __shared__ float v[RW][CW + 1];
    const int64_t i0 = (int64_t)blockIdx.x * RW;
    float acc = 0.0f;
    for (int k0 = 0; k0 < m_pad; k0 += CW) {
        for (int t = threadIdx.x; t < RW * CW; t += WG) {
            const int r = t / CW, k = k0 + t % CW;
            const int64_t i = i0 + r;
            if (k >= m_pad || i >= NPAD) continue;
            const bool in = (i < N) && (k < m);
            const float raw = in ? X[i * m + k] : 0.0f;
            const int64_t o = i * m_pad + k;
            if (kind == GRAM_F64) {
                f64[o] = (double)raw;
                continue;
            }
            const float xc = in ? (float)((double)raw - mean[k]) : 0.0f;
            float s = xc;
            if (kind == GRAM_F32) {
                f32[o] = xc;
            } else {
                const uint16_t hb = f2bf(xc);
                s = bf2f(hb);
                hi[o] = hb;
                if (kind == GRAM_BF16X3 || kind == GRAM_BF16X6) {
                    const uint16_t l = f2bf(xc - s);
                    lo[o] = l;
                    if (kind == GRAM_BF16X6) {
                        const uint16_t l2 = f2bf((xc - s) - bf2f(l));
                        lo2[o] = l2;
                        s += bf2f(l) + bf2f(l2);
                    } else {
                        s += bf2f(l);
                    }
                }
            }
            v[r][t % CW] = s;
        }
        if (kind != GRAM_F64) {
            __syncthreads();
            if (threadIdx.x < RW)
                for (int c = 0; c < CW && k0 + c < m_pad; ++c) acc = fmaf(v[threadIdx.x][c], v[threadIdx.x][c], acc);
            __syncthreads();
        }
    }
    if (nrm && threadIdx.x < RW && i0 + threadIdx.x < NPAD) nrm[i0 + threadIdx.x] = (kind == GRAM_F64) ? 0.0f : acc;
}

// Materialise the K' tiles.  Wave w computes the 32-row bands w and w + 4,
// one 32 x 32 block at a time, and stores straight from the MFMA layout.
template <int KIND>
__global__ __launch_bounds__(WG) void k_gram_mfma(Features F, KernelParams kp,
                                                 const uint32_t* __restrict__ tiles,
                                                 float* __restrict__ Kp) {
    const TileCoord tc = tile_of(tiles);
    const size_t tbase = (size_t)blockIdx.x * TT;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, h = l >> 5, l32 = l & 31;
    for (int band = w; band < TILE / 32; band += 4) {
        const int64_t rowA = (int64_t)tc.I * TILE + band * 32 + l32;
        float ni[16];
#pragma unroll
        for (int r = 0; r < 16; ++r)
            ni[r] = F.nrm[(int64_t)tc.I * TILE + band * 32 + 8 * (r >> 2) + 4 * h + (r & 3)];
        for (int cb = 0; cb < TILE / 32; ++cb) {
            const int64_t colB = (int64_t)tc.J * TILE + cb * 32 + l32;
            const f32x16 acc = mfma_gram_32x32<KIND>(F, rowA, colB);
            const float nj = F.nrm[colB];
            const int col = cb * 32 + l32;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = band * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
                Kp[tbase + (size_t)row * TILE + col] =
                    kernel_entry(ni[r], nj, acc[r], (int64_t)tc.I * TILE + row, colB, kp);
            }
        }
    }
}

// Materialise the K' tiles and, in the same pass, the partial row and column
// sums and maxima of K' (>= 0) that the diagonal weighting needs, in the
// layout of k_rowsum.  Wave w computes the 32-row bands w and w + 4 with the
// band's A fragments in registers, walking the eight 32-column blocks.  Each
// 32 x 32 block goes through LDS once: column sums come from the MFMA layout
// (a lane holds 16 rows of one column), row sums and the 16-byte row stores
// from the transposed read (eight lanes per row).  All sums in a fixed order.
// BF16 Gram kinds: the four waves walk the same column blocks, so each
// block's B fragments are staged once in LDS in fragment order (BStage), the
// next block's chunks loaded into registers while the current one is
// multiplied (one barrier per block; the products in the same order as from
// registers, so K' is the same to the bit).
template <int KIND, int MP>
__global__ __launch_bounds__(WG) void k_gram_sums(Features F, KernelParams kp, const uint32_t* __restrict__ tiles,
                                                 float* __restrict__ Kp, int NB, double* __restrict__ psum,
                                                 double* __restrict__ pmax) {
    // tiles in list order (any order of the upper tiles, read XCD-contiguously);
    // each is written at its own position of the plane
    const uint32_t ij = tiles[xcd_contiguous(blockIdx.x, gridDim.x)];
    const TileCoord tc{(int)(ij >> 16), (int)(ij & 0xFFFFu)};
    const size_t tbase = (size_t)tile_index(tc.I, tc.J, NB) * TT;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, h = l >> 5, l32 = l & 31;
    __shared__ double csum[4][TILE];
    __shared__ float cmax[4][TILE];
    __shared__ float blk[4][32][33];
    const int64_t i0 = (int64_t)tc.I * TILE, j0 = (int64_t)tc.J * TILE;
    const int rr = l >> 3, cq = 4 * (l & 7);       // transposed read: row rr + 8 k, columns cq .. cq + 3
    constexpr bool STG = (KIND != GRAM_F32) && (MP > 0);
    using BS = BStage<KIND>;
    constexpr int CH = STG ? BS::NP * (MP / 16) * 64 : 1;                  // 16-byte chunks per block
    constexpr int PR = (CH + WG - 1) / WG;                                 // per thread
    __shared__ bf16x8 sb[2][CH];
    const int ns = F.m_pad / 16, ch = BS::NP * ns * 64;
    int cur = 0;
    if constexpr (STG) {
#pragma unroll
        for (int i = 0; i < PR; ++i) {
            const int k = tid + WG * i;
            if (k < ch) sb[0][BS::dst(ns, k)] = *BS::src(F, j0, ns, k);
        }
        __syncthreads();
    }
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
        const int band = w + 4 * pass;
        const int64_t rowA = i0 + band * 32 + l32;
        float ni[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) ni[r] = F.nrm[i0 + band * 32 + 8 * (r >> 2) + 4 * h + (r & 3)];
        RowFrag<KIND, MP> fa;
        fa.load(F, rowA);
        double rs[4] = {0.0, 0.0, 0.0, 0.0};
        float rm[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int cb = 0; cb < TILE / 32; ++cb) {
            const int64_t colB = j0 + cb * 32 + l32;
            // the next block (the first again after the last of pass 0)
            const bool more = STG && !(pass == 1 && cb == TILE / 32 - 1);
            const int64_t nb0 = j0 + ((cb + 1) % (TILE / 32)) * 32;
            bf16x8 pre[PR];
            if constexpr (STG) {
                if (more) {
#pragma unroll
                    for (int i = 0; i < PR; ++i) {
                        const int k = tid + WG * i;
                        if (k < ch) pre[i] = *BS::src(F, nb0, ns, k);
                    }
                }
            }
            f32x16 acc = {};
            if constexpr (STG) BS::template mma<MP>(fa, sb[cur], ns, l, acc);
            else acc = fa.gram(F, rowA, F, colB);
            const float nj = F.nrm[colB];
            double cs = 0.0;
            float cm = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 8 * (r >> 2) + 4 * h + (r & 3);
                const float kv = kernel_entry(ni[r], nj, acc[r], i0 + band * 32 + row, colB, kp);
                blk[w][row][l32] = kv;
                cs += (double)kv;
                cm = fmaxf(cm, kv);
            }
            // the column's 32 rows of this band: both lane halves
            cs = cs + __shfl_xor(cs, 32);
            cm = fmaxf(cm, __shfl_xor(cm, 32));
            const int col = cb * 32 + l32;
            if (h == 0) {
                if (pass == 0) { csum[w][col] = cs; cmax[w][col] = cm; }
                else { csum[w][col] += cs; cmax[w][col] = fmaxf(cmax[w][col], cm); }
            }
            wave_lds_sync();
            float* dst = Kp + tbase + (size_t)(band * 32 + rr) * TILE + cb * 32 + cq;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float* src = &blk[w][rr + 8 * k][cq];
                const f32x4v v = {src[0], src[1], src[2], src[3]};
                __builtin_nontemporal_store(v, reinterpret_cast<f32x4v*>(dst + (size_t)8 * k * TILE));
                rs[k] += ((double)v[0] + (double)v[1]) + ((double)v[2] + (double)v[3]);
                rm[k] = fmaxf(rm[k], fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
            }
            wave_lds_sync();
            if constexpr (STG) {
                if (more) {
#pragma unroll
                    for (int i = 0; i < PR; ++i) {
                        const int k = tid + WG * i;
                        if (k < ch) sb[cur ^ 1][BS::dst(ns, k)] = pre[i];
                    }
                }
                __syncthreads();
                cur ^= 1;
            }
        }
        // rows rr + 8 k: the eight lanes of each row add their column quads
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double v = rs[k];
            v = v + dpp<0xB1>(v);
            v = v + dpp<0x4E>(v);
            v = v + dpp<0x141>(v);
            float mv = rm[k];
            mv = fmaxf(mv, dpp<0xB1>(mv));
            mv = fmaxf(mv, dpp<0x4E>(mv));
            mv = fmaxf(mv, dpp<0x141>(mv));
            if ((l & 7) == 0) {
                const size_t o = ((size_t)tc.I * (NB + 1) + tc.J) * TILE + band * 32 + rr + 8 * k;
                psum[o] = v;
                pmax[o] = (double)mv;
            }
        }
    }
    __syncthreads();
    const int slot = (tc.I < tc.J) ? tc.I : NB;
    const size_t cb = ((size_t)tc.J * (NB + 1) + slot) * TILE + tid;
    psum[cb] = (csum[0][tid] + csum[1][tid]) + (csum[2][tid] + csum[3][tid]);
    pmax[cb] = (double)fmaxf(fmaxf(cmax[0][tid], cmax[1][tid]), fmaxf(cmax[2][tid], cmax[3][tid]));
}

template <int KIND>
void gram_sums_kind(int mp, dim3 g, const Features& F, const KernelParams& kp, const uint32_t* tiles, float* Kp,
                    int NB, double* psum, double* pmax, hipStream_t s) {
    if (mp <= 32)
        hipLaunchKernelGGL((k_gram_sums<KIND, 32>), g, dim3(WG), 0, s, F, kp, tiles, Kp, NB, psum, pmax);
    else if (mp <= 64)
        hipLaunchKernelGGL((k_gram_sums<KIND, 64>), g, dim3(WG), 0, s, F, kp, tiles, Kp, NB, psum, pmax);
    else if (mp <= 128)
        hipLaunchKernelGGL((k_gram_sums<KIND, 128>), g, dim3(WG), 0, s, F, kp, tiles, Kp, NB, psum, pmax);
    else
        hipLaunchKernelGGL((k_gram_sums<KIND, 0>), g, dim3(WG), 0, s, F, kp, tiles, Kp, NB, psum, pmax);
}

// FP64 K' from direct differences (no Gram expansion, no centring).  One
// workgroup per 32-row band of a tile, 16 features at a time through LDS, a
// lane holding 8 rows x 4 columns of sums (m_pad is a multiple of 16; the
// features in order, as one chain per pair).  (One workgroup per tile reading
// the column rows from memory for every row: 490 us for three tiles of 10
// features, one serial chain; now 14 us.)
__global__ __launch_bounds__(WG) void k_gram_f64(Features F, KernelParams kp,
                                                const uint32_t* __restrict__ tiles,
                                                double* __restrict__ Kp) {
    constexpr int KC = 16, BR = 32;
    __shared__ __attribute__((aligned(16))) double xj[KC][TILE];
    __shared__ double xi[KC][BR];
    const int64_t tile = blockIdx.x / (TILE / BR);
    const int band = blockIdx.x % (TILE / BR);
    const uint32_t ij = tiles[tile];
    const TileCoord tc{(int)(ij >> 16), (int)(ij & 0xFFFFu)};
    const size_t tbase = (size_t)tile * TT;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, g = l >> 4, q = l & 15;
    const int col0 = w * 64 + q * 4;
    const int mp = F.m_pad;
    const double* pj = F.f64 + ((int64_t)tc.J * TILE + tid) * mp;
    const double* pi = F.f64 + ((int64_t)tc.I * TILE + band * BR + (tid & (BR - 1))) * mp;
    double d2[BR / 4][4];
#pragma unroll
    for (int s = 0; s < BR / 4; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) d2[s][c] = 0.0;
    for (int k0 = 0; k0 < mp; k0 += KC) {
#pragma unroll
        for (int k = 0; k < KC; ++k) xj[k][tid] = pj[k0 + k];
#pragma unroll
        for (int k = tid / BR; k < KC; k += WG / BR) xi[k][tid & (BR - 1)] = pi[k0 + k];
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < KC; ++k) {
            const V4<double> x = ld4(&xj[k][col0]);
#pragma unroll
            for (int s = 0; s < BR / 4; ++s) {
                const double a = xi[k][4 * s + g];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double d = a - x.v[c];
                    d2[s][c] = fma(d, d, d2[s][c]);
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int s = 0; s < BR / 4; ++s) {
        const int r = band * BR + 4 * s + g;
        const int64_t i = (int64_t)tc.I * TILE + r;
        V4<double> out;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int64_t j = (int64_t)tc.J * TILE + col0 + c;
            out.v[c] = (i < j && j < kp.N) ? exp(-kp.gamma * d2[s][c]) + kp.lam2 : 0.0;
        }
        st4(Kp + tbase + (size_t)r * TILE + col0, out);
    }
}

// K' taken from a caller-supplied dense N x N matrix (upper triangle).
template <class ST>
__global__ __launch_bounds__(WG) void k_gather_dense(const double* __restrict__ K, KernelParams kp,
                                                    const uint32_t* __restrict__ tiles,
                                                    ST* __restrict__ Kp) {
    const TileCoord tc = tile_of(tiles);
    const size_t tbase = (size_t)blockIdx.x * TT;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, q = l & 15;
    const int col0 = w * 64 + q * 4;
    for (int s = 0; s < TILE / 4; ++s) {
        const int r = 4 * s + g;
        const int64_t i = (int64_t)tc.I * TILE + r;
        V4<ST> out;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int64_t j = (int64_t)tc.J * TILE + col0 + c;
            out.v[c] = (i < j && j < kp.N) ? (ST)K[i * kp.N + j] : (ST)0;
        }
        st4(Kp + tbase + (size_t)r * TILE + col0, out);
    }
}

__global__ void k_dense_diag(const double* __restrict__ K, int64_t N, double* kdiag) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) kdiag[i] = K[i * N + i];
}

__global__ void k_fill_value(double* dst, int64_t n, double v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = v;
}

// --------------------------------------------------- diagonal weighting --

// Partial sums r_i = sum_{j != i} |K'_ij| and maxima max_{j != i} |K'_ij| per
// tile slot (FP64), from the K' plane or from K' recomputed per band.
template <class ST, int KSRC, int GK>
__global__ __launch_bounds__(WG) void k_rowsum(const ST* __restrict__ Kp, Features F, KernelParams kp,
                                              const uint32_t* __restrict__ tiles, int NB,
                                              double* __restrict__ psum, double* __restrict__ pmax) {
    const TileCoord tc = tile_of(tiles);
    const size_t tbase = (size_t)blockIdx.x * TT;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, g = l >> 4, q = l & 15;
    const int col0 = w * 64 + q * 4;
    __shared__ double rows[4][TILE], rmax[4][TILE];
    __shared__ float kband[KSRC == KSRC_RECOMPUTE ? 4 : 1][KSRC == KSRC_RECOMPUTE ? 32 * 64 : 1];
    double cs[4] = {0.0, 0.0, 0.0, 0.0}, cm[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = 0; b < TILE / 32; ++b) {
        if constexpr (KSRC == KSRC_RECOMPUTE) {
            gram_band<GK>(F, kp, tc.I, tc.J, 32 * b, 64 * w, kband[w]);
            wave_lds_sync();
        }
        for (int s2 = 0; s2 < 8; ++s2) {
            const int r = 32 * b + 4 * s2 + g;
            V4<ST> k;
            if constexpr (KSRC == KSRC_RECOMPUTE) {
                const float4 kk = *reinterpret_cast<const float4*>(&kband[w][(4 * s2 + g) * 64 + 4 * q]);
                k = V4<ST>{{(ST)kk.x, (ST)kk.y, (ST)kk.z, (ST)kk.w}};
            } else {
                k = ld4(Kp + tbase + (size_t)r * TILE + col0);
            }
            double rs = 0.0, rm = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double a = fabs((double)k.v[c]);
                cs[c] += a;
                rs += a;
                cm[c] = fmax(cm[c], a);
                rm = fmax(rm, a);
            }
            rs = sum16(rs);
            rm = fmax(rm, dpp<0xB1>(rm));
            rm = fmax(rm, dpp<0x4E>(rm));
            rm = fmax(rm, dpp<0x141>(rm));
            rm = fmax(rm, dpp<0x140>(rm));
            if (q == 0) { rows[w][r] = rs; rmax[w][r] = rm; }
        }
        if constexpr (KSRC == KSRC_RECOMPUTE) wave_lds_sync();
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        cs[c] = sum_groups(cs[c]);
        cm[c] = fmax(cm[c], __shfl_xor(cm[c], 16));
        cm[c] = fmax(cm[c], __shfl_xor(cm[c], 32));
    }
    __syncthreads();
    const size_t rs_ = ((size_t)tc.I * (NB + 1) + tc.J) * TILE + tid;
    psum[rs_] = (rows[0][tid] + rows[1][tid]) + (rows[2][tid] + rows[3][tid]);
    pmax[rs_] = fmax(fmax(rmax[0][tid], rmax[1][tid]), fmax(rmax[2][tid], rmax[3][tid]));
    if (g == 0) {
        const int slot = (tc.I < tc.J) ? tc.I : NB;
        const size_t cb = ((size_t)tc.J * (NB + 1) + slot) * TILE + col0;
#pragma unroll
        for (int c = 0; c < 4; ++c) { psum[cb + c] = cs[c]; pmax[cb + c] = cm[c]; }
    }
}

// Residual certificate of a finished solve: partial products
// sum_{j != i} K'_ij w_j (w_j = y_j alpha_j) per tile slot, in FP64, in the
// layout and lane order of k_rowsum (row part: slot J of block I; column
// part: slot I of block J, or slot NB for a diagonal tile).
template <class ST, int KSRC, int GK>
__global__ __launch_bounds__(WG) void k_apply(const ST* __restrict__ Kp, Features F, KernelParams kp,
                                             const uint32_t* __restrict__ tiles, int NB,
                                             const double* __restrict__ w, double* __restrict__ part) {
    const TileCoord tc = tile_of(tiles);
    const size_t tbase = (size_t)blockIdx.x * TT;
    const int tid = threadIdx.x, wv = tid >> 6, l = tid & 63, g = l >> 4, q = l & 15;
    const int col0 = wv * 64 + q * 4;
    __shared__ double rows[4][TILE];
    __shared__ float kband[KSRC == KSRC_RECOMPUTE ? 4 : 1][KSRC == KSRC_RECOMPUTE ? 32 * 64 : 1];
    const double* wI = w + (size_t)tc.I * TILE;
    const double* wJ = w + (size_t)tc.J * TILE;
    double wc[4], cs[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < 4; ++c) wc[c] = wJ[col0 + c];
    for (int b = 0; b < TILE / 32; ++b) {
        if constexpr (KSRC == KSRC_RECOMPUTE) {
            gram_band<GK>(F, kp, tc.I, tc.J, 32 * b, 64 * wv, kband[wv]);
            wave_lds_sync();
        }
        for (int s2 = 0; s2 < 8; ++s2) {
            const int r = 32 * b + 4 * s2 + g;
            V4<ST> k;
            if constexpr (KSRC == KSRC_RECOMPUTE) {
                const float4 kk = *reinterpret_cast<const float4*>(&kband[wv][(4 * s2 + g) * 64 + 4 * q]);
                k = V4<ST>{{(ST)kk.x, (ST)kk.y, (ST)kk.z, (ST)kk.w}};
            } else {
                k = ld4(Kp + tbase + (size_t)r * TILE + col0);
            }
            const double wr = wI[r];
            double rs = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double a = (double)k.v[c];
                rs = fma(a, wc[c], rs);
                cs[c] = fma(a, wr, cs[c]);
            }
            rs = sum16(rs);
            if (q == 0) rows[wv][r] = rs;
        }
        if constexpr (KSRC == KSRC_RECOMPUTE) wave_lds_sync();
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) cs[c] = sum_groups(cs[c]);
    __syncthreads();
    part[((size_t)tc.I * (NB + 1) + tc.J) * TILE + tid] = (rows[0][tid] + rows[1][tid]) + (rows[2][tid] + rows[3][tid]);
    if (g == 0) {
        const int slot = (tc.I < tc.J) ? tc.I : NB;
        const size_t cb = ((size_t)tc.J * (NB + 1) + slot) * TILE + col0;
#pragma unroll
        for (int c = 0; c < 4; ++c) part[cb + c] = cs[c];
    }
}

// w_i = y_i alpha_i on [0, N), zero on the padded rows.
__global__ void k_weights(int64_t N, int64_t NPAD, const double* __restrict__ alpha,
                          const float* __restrict__ y, double* __restrict__ w) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < NPAD) w[i] = (i < N) ? (double)y[i] * alpha[i] : 0.0;
}

// Per node: (A alpha)_i = A_ii alpha_i + y_i sum_{j != i} K'_ij w_j from the
// slot partials in slot order; per block: max_i |1 - (A alpha)_i| (+inf for a
// non-finite value) and min_i (A_ii - r_i).
__global__ __launch_bounds__(WG) void k_residual_blocks(int64_t N, int NB, const double* __restrict__ part,
                                                        const double* __restrict__ Adiag,
                                                        const double* __restrict__ rsum,
                                                        const double* __restrict__ alpha,
                                                        const float* __restrict__ y, double* __restrict__ bres,
                                                        double* __restrict__ bgap) {
    __shared__ double sh4[4];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double res = 0.0, ngap = -INFINITY;
    if (i < N) {
        const int64_t B = i / TILE, t = i % TILE;
        double acc = 0.0;
        for (int sl = 0; sl <= NB; ++sl) acc += part[((size_t)B * (NB + 1) + sl) * TILE + t];
        const double r = 1.0 - (Adiag[i] * alpha[i] + (double)y[i] * acc);
        res = isfinite(r) ? fabs(r) : INFINITY;
        ngap = -(Adiag[i] - rsum[i]);
    }
    res = block_max(res, sh4);
    __syncthreads();
    ngap = block_max(ngap, sh4);
    if (threadIdx.x == 0) { bres[blockIdx.x] = res; bgap[blockIdx.x] = ngap; }
}

// out[0] = ||1 - A alpha||_inf, out[1] = min_i (A_ii - r_i), out[2] = Varah's
// bound out[0] / out[1] on ||alpha - A^-1 1||_inf (+inf unless out[1] > 0).
__global__ __launch_bounds__(WG) void k_residual_final(int nb, const double* __restrict__ bres,
                                                       const double* __restrict__ bgap, double* __restrict__ out) {
    __shared__ double sh4[4];
    double r = 0.0, ng = -INFINITY;
    for (int k = threadIdx.x; k < nb; k += blockDim.x) { r = fmax(r, bres[k]); ng = fmax(ng, bgap[k]); }
    r = block_max(r, sh4);
    __syncthreads();
    ng = block_max(ng, sh4);
    if (threadIdx.x == 0) {
        const double gap = -ng;
        out[0] = r;
        out[1] = gap;
        out[2] = (gap > 0.0) ? r / gap : INFINITY;
    }
}

// Weighted diagonal (subsection "GaBP Algorithm Convergence") and the row
// maxima of |K'|.  For the uniform rule this kernel leaves the per-block max
// of A_ii - K'_ii for k_diag_shift.
__global__ void k_diag(int64_t N, int NB, const double* __restrict__ psum,
                       const double* __restrict__ pmax, const double* __restrict__ kdiag, int mode,
                       double C, double delta, double* __restrict__ Adiag,
                       double* __restrict__ rowmax, double* __restrict__ rsum, double* __restrict__ blk) {
    __shared__ double sh4[4];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double wv = -INFINITY;
    if (i < N) {
        const int64_t B = i / TILE, t = i % TILE;
        double r = 0.0, mx = 0.0;
        for (int s = 0; s <= NB; ++s) {
            const size_t o = ((size_t)B * (NB + 1) + s) * TILE + t;
            r += psum[o];
            mx = fmax(mx, pmax[o]);
        }
        const double kii = kdiag[i];
        const double soft = kii + 1.0 / C, dom = (1.0 + delta) * r;
        double a;
        switch (mode) {
            case 0: a = kii; break;
            case 1: a = soft; break;
            default: a = fmax(soft, dom); break;
        }
        Adiag[i] = a;
        rowmax[i] = mx;
        rsum[i] = r;
        wv = a - kii;
    }
    if (mode == 3) {
        wv = block_max(wv, sh4);
        if (threadIdx.x == 0) blk[blockIdx.x] = wv;
    }
}

// Maxima of consecutive arrays of n values, one workgroup each.
__global__ void k_max_reduce(int n, const double* __restrict__ in, double* out) {
    __shared__ double sh4[4];
    double v = -INFINITY;
    for (int k = threadIdx.x; k < n; k += blockDim.x) v = fmax(v, in[(size_t)blockIdx.x * n + k]);
    v = block_max(v, sh4);
    if (threadIdx.x == 0) out[blockIdx.x] = v;
}

__global__ void k_diag_shift(int64_t N, const double* __restrict__ kdiag,
                             const double* __restrict__ shift, double* __restrict__ Adiag) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) Adiag[i] = kdiag[i] + *shift;
}

__global__ void k_reset_status(DevStatus* st) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        st->t = 0; st->done = 0; st->reason = R_NONE; st->since_best = 0; st->bad = 0; st->g = 0; st->ticket = 0;
        st->delta = 0.0; st->amax = 0.0; st->best_delta = INFINITY;
    }
}

// Sweep 0: aggregates of all-zero messages, P~ = A_ii, S = b = y, in ring
// slot 0.  Padded nodes get P~ = 1, S = 0 so that their (zero) messages stay
// finite.
template <class AT>
__global__ void k_init(int64_t N, int64_t NPAD, int R, const double* __restrict__ Adiag,
                       const float* __restrict__ y, AT* __restrict__ Pt, AT* __restrict__ S,
                       double* __restrict__ alpha, DevStatus* st, double boxC) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NPAD) return;
    if (i < N) {
        const AT a = (AT)Adiag[i];
        AT b = (AT)y[i];
        double an = (double)(b / a) * (double)y[i];
        if (boxC > 0.0) {              // box projection of the initial means
            an = fmin(fmax(an, 0.0), boxC);
            b = a * (AT)(an * (double)y[i]);
        }
        Pt[i] = a;
        S[i] = b;
        alpha[i] = an;
        if (!(a > (AT)0) || !isfinite((double)a)) st->bad = 1;
        // slots of the sweeps before sweep 0 (stateless ring): P~ = +inf and
        // S = 0 make every message rebuilt from them exactly zero, which is
        // what the messages of sweep 0 are, so a fixed number of levels is
        // exact from sweep 1 on
        for (int r = 1; r < R; ++r) {
            Pt[(int64_t)r * NPAD + i] = (AT)INFINITY;
            S[(int64_t)r * NPAD + i] = (AT)0;
        }
    } else {
        // padding rows are never finalized: set them in every ring slot
        for (int r = 0; r < R; ++r) {
            Pt[(int64_t)r * NPAD + i] = (AT)1;
            S[(int64_t)r * NPAD + i] = (AT)0;
        }
    }
}

// Aggregates of the FB nodes of finalize block `blk` from the partial sums
// (fixed order), the new alpha and the block's change / magnitude maxima.
// boxC > 0: the belief mean is clipped to [0, boxC] (alpha space) and S is
// replaced by P~ times the clipped mean.  The block's slots are split into
// four contiguous ranges, one per wave, a lane adding one node over its
// wave's range, eight slots' loads in flight (the additions keep the slot
// order); wave 0 adds the four parts and forms the node.  The reads of the
// partials are a short latency chain, so the node range is spread over as
// many workgroups as it has waves: with 256 nodes per workgroup and one slot
// in flight a 158-slot group visit took 17.8 us and an 80-slot sweep 10.6 us.
template <class AT, class PT>
__device__ inline void finalize_block(int64_t blk, int64_t N, int stride, int slots, const PT* __restrict__ partP,
                                      const PT* __restrict__ partE,
                                      const double* __restrict__ Adiag,
                                      const float* __restrict__ y, AT* __restrict__ Pt,
                                      AT* __restrict__ S, double* __restrict__ alpha,
                                      double* __restrict__ blk_delta,
                                      double* __restrict__ blk_amax, DevStatus* st, double boxC,
                                      AT* __restrict__ Inv, AT* __restrict__ Mean) {
    __shared__ AT shp[4][FB], she[4][FB];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int64_t i = blk * FB + l;
    {
        const int qn = (slots + 3) / 4;
        const int s0 = w * qn, s1 = (s0 + qn < slots) ? s0 + qn : slots;
        const size_t o = (size_t)(i / TILE) * stride * TILE + (size_t)(i % TILE);
        const PT* pp = partP + o;
        const PT* pe = partE + o;
        AT ap = 0, ae = 0;
        int s = s0;
        for (; s + 8 <= s1; s += 8) {
            PT vp[8], ve[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) { vp[k] = pp[(size_t)(s + k) * TILE]; ve[k] = pe[(size_t)(s + k) * TILE]; }
#pragma unroll
            for (int k = 0; k < 8; ++k) { ap += (AT)vp[k]; ae += (AT)ve[k]; }
        }
        for (; s < s1; ++s) { ap += (AT)pp[(size_t)s * TILE]; ae += (AT)pe[(size_t)s * TILE]; }
        shp[w][l] = ap;
        she[w][l] = ae;
    }
    __syncthreads();
    if (w != 0) return;
    double d = 0.0, am = 0.0;
    bool bad = false;
    if (i < N) {
        AT p = (AT)Adiag[i] + ((shp[0][l] + shp[1][l]) + (shp[2][l] + shp[3][l]));
        AT e = (AT)y[i] + ((she[0][l] + she[1][l]) + (she[2][l] + she[3][l]));
        double an = (double)(e / p) * (double)y[i];
        bad = !(p > (AT)0) || !isfinite((double)p) || !isfinite((double)e);
        if (boxC > 0.0) {
            an = fmin(fmax(an, 0.0), boxC);
            e = p * (AT)(an * (double)y[i]);
        }
        Pt[i] = p;
        S[i] = e;
        if (Inv) { Inv[i] = (AT)1 / p; Mean[i] = e / p; }
        d = fabs(an - alpha[i]);
        am = fabs(an);
        alpha[i] = an;
    }
    if (__any(bad) && l == 0) store_agent(&st->bad, 1);
    d = wave_max(d);
    am = wave_max(am);
    if (l == 0) { store_agent(blk_delta + blk, d); store_agent(blk_amax + blk, am); }
}

// One finalize launch; with `trace` the workgroup that takes the last ticket
// applies the stop rule (no workgroup waits).  Each workgroup's maxima are
// written through to device scope and have completed before its ticket, and
// the last workgroup reads them at device scope, so no cache is written back
// for them (a fence per workgroup costs more than the launch it saves).
template <class AT, class PT>
__global__ __launch_bounds__(WG) void k_finalize(FinalizeArgs f) {
    if (f.st->done) return;
    __shared__ int last;
    const int64_t blk = f.b0 * (TILE / FB) + blockIdx.x;
    const int slots = f.split > 1 ? part_slots((int)(blk / (TILE / FB)), f.NB, f.split) : f.stride;
    finalize_block<AT, PT>(blk, f.N, f.stride, slots, static_cast<const PT*>(f.partP),
                           static_cast<const PT*>(f.partE), f.Adiag, f.y, static_cast<AT*>(f.Pt),
                           static_cast<AT*>(f.S), f.alpha, f.blk_delta, f.blk_amax, f.st, f.boxC,
                           static_cast<AT*>(f.Inv), static_cast<AT*>(f.Mean));
    if (!f.trace) return;
    if (threadIdx.x == 0) {
        wait_vm<0>();
        last = atomicAdd(&f.st->ticket, 1u) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    if (threadIdx.x == 0) f.st->ticket = 0;
    status_update((int)((f.N + FB - 1) / FB), f.blk_delta, f.blk_amax, f.st, f.trace, f.rule);
}

// 1/P~ and S/P~ of every ring slot (series sweeps): P~ = +inf, S = 0 give 0
// and 0, the values a tile would form from them.
template <class AT>
__global__ void k_ring_recip(int64_t n, const AT* __restrict__ Pt, const AT* __restrict__ S,
                             AT* __restrict__ Inv, AT* __restrict__ Mean) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    Inv[i] = (AT)1 / Pt[i];
    Mean[i] = S[i] / Pt[i];
}

// The stop rule as a launch of its own.
__global__ __launch_bounds__(WG) void k_status(FinalizeArgs f) {
    if (f.st->done) return;
    status_update((int)((f.N + FB - 1) / FB), f.blk_delta, f.blk_amax, f.st, f.trace, f.rule);
}

// Served form: items are (request, block of 256 nodes), four finalize blocks
// each.
template <class AT>
__global__ __launch_bounds__(WG) void k_finalize_batched(const ReqDesc* __restrict__ reqs,
                                                        const uint2* __restrict__ items, int nitems) {
    constexpr int SUB = TILE / FB;
    for (int it = blockIdx.x; it < nitems * SUB; it += gridDim.x) {
        const uint2 w = items[it / SUB];
        const ReqDesc& rd = reqs[w.x];
        const int64_t blk = (int64_t)w.y * SUB + it % SUB;
        if (rd.sw.st->done || blk * FB >= rd.N) continue;
        const int64_t wslot = (int64_t)((rd.sw.st->t + 1) % rd.sw.R) * rd.sw.NPAD;
        AT* const Pt = static_cast<AT*>(const_cast<void*>(rd.sw.HP)) + wslot;
        AT* const S = static_cast<AT*>(const_cast<void*>(rd.sw.HS)) + wslot;
        // NBc + 1 slots per block after a sweep over chunks
        const int stride = (rd.sw.chunk > 1) ? (rd.sw.NB + rd.sw.chunk - 1) / rd.sw.chunk + 1
                                             : part_stride(rd.sw.NB, rd.sw.split);
        const int ns = (rd.sw.chunk > 1) ? stride : part_slots((int)w.y, rd.sw.NB, rd.sw.split);
        if (rd.sw.part32)
            finalize_block<AT, float>(blk, rd.N, stride, ns, static_cast<const float*>(rd.sw.partP),
                                      static_cast<const float*>(rd.sw.partE), rd.Adiag, rd.y, Pt, S, rd.alpha,
                                      rd.blk_delta, rd.blk_amax, rd.sw.st, 0.0, nullptr, nullptr);
        else
            finalize_block<AT, AT>(blk, rd.N, stride, ns, static_cast<const AT*>(rd.sw.partP),
                                   static_cast<const AT*>(rd.sw.partE), rd.Adiag, rd.y, Pt, S, rd.alpha,
                                   rd.blk_delta, rd.blk_amax, rd.sw.st, 0.0, nullptr, nullptr);
        __syncthreads();
    }
}

// Stop rule of served requests, one workgroup per active request; also copies
// the request's status into a packed array the host reads back in one
// transfer.  A step visits one group of a grouped
// request (G groups; G = 1 for the synchronous schedule); after the visit of
// the last group the stop rule runs (one sweep done), and the group index
// advances for every request still running.
__global__ __launch_bounds__(WG) void k_status_grouped(const ReqDesc* __restrict__ reqs,
                                                      const int* __restrict__ slots, int n,
                                                      DevStatus* __restrict__ out) {
    const int k = blockIdx.x;
    if (k >= n) return;
    const ReqDesc& rd = reqs[slots[k]];
    DevStatus* st = rd.sw.st;
    const int done0 = st->done, g0 = st->g;
    __syncthreads();
    if (!done0) {
        if (g0 == rd.G - 1) status_update(rd.nblk, rd.blk_delta, rd.blk_amax, st, rd.trace, rd.rule);
        if (threadIdx.x == 0) st->g = (g0 + 1) % rd.G;
    }
    __syncthreads();
    if (threadIdx.x == 0) out[k] = *st;
}

// A-priori bound on the contraction of the message recursion.  With
// c_i = max_j |A_ij| * sum_{j != i} |A_ij|, every cavity precision satisfies
// Q_ij >= P~_i^(t-1) (messages are non-positive while Q > 0) and, by
// induction over sweeps, P~_i^t >= lo_i = A_ii - c_i / m* where
// m* = min_i (A_ii + sqrt(A_ii^2 - 4 c_i)) / 2 (the larger root of
// m^2 - A_ii m + c_i).  The induction needs every lo_i >= m* (then m* bounds
// every aggregate from below, P~^0 = A_ii included); lo_i equals m* at the
// node that defines it, so the comparison allows a 1e-12 relative rounding
// margin.  The reverse message enters the next one with a factor
// |A_ij| / Q_ij <= rowmax_i / lo_i, whose maximum is returned as rho (+inf if
// the bound does not exist).
__global__ void k_bound_root(int64_t N, const double* __restrict__ Adiag, const double* __restrict__ rowmax,
                             const double* __restrict__ rsum, double* __restrict__ blk) {
    __shared__ double sh4[4];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double v = -INFINITY;   // holds -root, so the block max is -(min root)
    if (i < N) {
        const double A = Adiag[i], c = rowmax[i] * rsum[i], disc = A * A - 4.0 * c;
        v = (disc >= 0.0 && A > 0.0) ? -0.5 * (A + sqrt(disc)) : INFINITY;
    }
    v = block_max(v, sh4);
    if (threadIdx.x == 0) blk[blockIdx.x] = v;
}

__global__ void k_bound_rho(int64_t N, const double* __restrict__ Adiag, const double* __restrict__ rowmax,
                            const double* __restrict__ rsum, const double* __restrict__ neg_mstar,
                            double* __restrict__ blk) {
    __shared__ double sh4[4];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const double m = -*neg_mstar;
    double v = 0.0;
    if (i < N) {
        const double lo = Adiag[i] - rowmax[i] * rsum[i] / m;
        v = (m > 0.0 && lo >= m * (1.0 - 1e-12)) ? rowmax[i] / lo : INFINITY;
    }
    v = block_max(v, sh4);
    const double mx = block_max(i < N ? rowmax[i] : 0.0, sh4);
    if (threadIdx.x == 0) {
        blk[blockIdx.x] = v;
        blk[gridDim.x + blockIdx.x] = mx;
    }
}

// ------------------------------------------------------------- queries --

template <class ST>
__global__ void k_entries(const ST* __restrict__ Kp, int NB, const int64_t* __restrict__ rows,
                          const int64_t* __restrict__ cols, int64_t n, double* __restrict__ out) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int64_t i = rows[k], j = cols[k];
    if (i > j) { const int64_t t = i; i = j; j = t; }
    const int I = (int)(i / TILE), J = (int)(j / TILE);
    out[k] = (double)Kp[(size_t)tile_index(I, J, NB) * TT + (size_t)(i % TILE) * TILE + (j % TILE)];
}

template <class AT>
__global__ void k_pack_out(int64_t N, const double* __restrict__ alpha, const AT* __restrict__ Pt, int stride,
                           const double* __restrict__ Adiag, const float* __restrict__ y,
                           const int32_t* __restrict__ order, double* __restrict__ out) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= N) return;
    const int64_t i = order ? order[r] : r;
    out[i] = alpha[r];
    out[N + i] = (double)Pt[r * stride];
    out[2 * N + i] = Adiag[r];
    reinterpret_cast<float*>(out + 3 * N)[i] = y[r];
}

// ----------------------------------------------------------- launchers --

static inline unsigned grid1(int64_t n) { return (unsigned)((n + WG - 1) / WG); }

hipError_t launch_fill_tiles(uint32_t* tiles, int NB, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_tiles, dim3(NB), dim3(WG), 0, s, tiles, NB);
    return hipGetLastError();
}

hipError_t launch_validate(const float* X, const float* y, int64_t N, int64_t m, int32_t* flag,
                           hipStream_t s) {
    int64_t n = std::max<int64_t>(N * m, N);
    unsigned g = (unsigned)std::min<int64_t>((n + WG - 1) / WG, 4096);
    if (g == 0) g = 1;
    hipLaunchKernelGGL(k_validate, dim3(g), dim3(WG), 0, s, X, y, N, m, flag);
    return hipGetLastError();
}

hipError_t launch_colmean(const float* X, int64_t N, int64_t m, double* mean, hipStream_t s) {
    hipLaunchKernelGGL(k_colmean, dim3((unsigned)m), dim3(WG), 0, s, X, N, m, mean);
    return hipGetLastError();
}

hipError_t launch_stage(const float* X, const double* mean, int64_t N, int64_t m, int64_t NPAD,
                        int m_pad, int kind, float* f32, uint16_t* hi, uint16_t* lo, uint16_t* lo2,
                        double* f64, float* nrm, hipStream_t s) {
    hipLaunchKernelGGL(k_stage, dim3((unsigned)((NPAD + 63) / 64)), dim3(WG), 0, s, X, mean, N, m, NPAD, m_pad, kind,
                       f32, hi, lo, lo2, f64, nrm);
    return hipGetLastError();
}

hipError_t launch_gram(const Features& F, const KernelParams& kp, const uint32_t* tiles,
                       int64_t ntiles, void* Kp, hipStream_t s) {
    const dim3 g((unsigned)ntiles), b(WG);
    switch (F.kind) {
        case GRAM_F32: hipLaunchKernelGGL(k_gram_mfma<GRAM_F32>, g, b, 0, s, F, kp, tiles, (float*)Kp); break;
        case GRAM_BF16: hipLaunchKernelGGL(k_gram_mfma<GRAM_BF16>, g, b, 0, s, F, kp, tiles, (float*)Kp); break;
        case GRAM_BF16X3: hipLaunchKernelGGL(k_gram_mfma<GRAM_BF16X3>, g, b, 0, s, F, kp, tiles, (float*)Kp); break;
        case GRAM_BF16X6: hipLaunchKernelGGL(k_gram_mfma<GRAM_BF16X6>, g, b, 0, s, F, kp, tiles, (float*)Kp); break;
        case GRAM_F64: hipLaunchKernelGGL(k_gram_f64, dim3((unsigned)(ntiles * (TILE / 32))), b, 0, s, F, kp, tiles, (double*)Kp); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gram_sums(const Features& F, const KernelParams& kp, const uint32_t* tiles, int64_t ntiles,
                            void* Kp, int NB, double* psum, double* pmax, hipStream_t s) {
    const dim3 g((unsigned)ntiles);
    float* K = (float*)Kp;
    switch (F.kind) {
        case GRAM_F32: gram_sums_kind<GRAM_F32>(F.m_pad, g, F, kp, tiles, K, NB, psum, pmax, s); break;
        case GRAM_BF16: gram_sums_kind<GRAM_BF16>(F.m_pad, g, F, kp, tiles, K, NB, psum, pmax, s); break;
        case GRAM_BF16X3: gram_sums_kind<GRAM_BF16X3>(F.m_pad, g, F, kp, tiles, K, NB, psum, pmax, s); break;
        case GRAM_BF16X6: gram_sums_kind<GRAM_BF16X6>(F.m_pad, g, F, kp, tiles, K, NB, psum, pmax, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gather_dense(const double* K, const KernelParams& kp, const uint32_t* tiles,
                               int64_t ntiles, void* Kp, int prec, double* kdiag, hipStream_t s) {
    const dim3 g((unsigned)ntiles), b(WG);
    if (prec == PREC_FP64)
        hipLaunchKernelGGL(k_gather_dense<double>, g, b, 0, s, K, kp, tiles, (double*)Kp);
    else
        hipLaunchKernelGGL(k_gather_dense<float>, g, b, 0, s, K, kp, tiles, (float*)Kp);
    hipLaunchKernelGGL(k_dense_diag, dim3(grid1(kp.N)), dim3(WG), 0, s, K, kp.N, kdiag);
    return hipGetLastError();
}

hipError_t launch_fill_value(double* dst, int64_t n, double v, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_value, dim3(grid1(n)), dim3(WG), 0, s, dst, n, v);
    return hipGetLastError();
}

hipError_t launch_rowsum(const void* Kp, int prec, int ksrc, const Features& F, const KernelParams& kp,
                         const uint32_t* tiles, int64_t ntiles, int NB, double* psum, double* pmax,
                         hipStream_t s) {
    if (ntiles > kMaxBlocks && ksrc == KSRC_PLANE) return hipErrorInvalidValue;
    if (ntiles > kMaxBlocks)
        return in_launches(ntiles, [&](int64_t o, int64_t n) {
            return launch_rowsum(Kp, prec, ksrc, F, kp, tiles + o, n, NB, psum, pmax, s);
        });
    const dim3 g((unsigned)ntiles), b(WG);
    if (ksrc == KSRC_PLANE) {
        if (prec == PREC_FP64)
            hipLaunchKernelGGL((k_rowsum<double, KSRC_PLANE, GRAM_F64>), g, b, 0, s, (const double*)Kp, F, kp, tiles, NB, psum, pmax);
        else
            hipLaunchKernelGGL((k_rowsum<float, KSRC_PLANE, GRAM_F32>), g, b, 0, s, (const float*)Kp, F, kp, tiles, NB, psum, pmax);
    } else {
        switch (F.kind) {
            case GRAM_F32: hipLaunchKernelGGL((k_rowsum<float, KSRC_RECOMPUTE, GRAM_F32>), g, b, 0, s, nullptr, F, kp, tiles, NB, psum, pmax); break;
            case GRAM_BF16: hipLaunchKernelGGL((k_rowsum<float, KSRC_RECOMPUTE, GRAM_BF16>), g, b, 0, s, nullptr, F, kp, tiles, NB, psum, pmax); break;
            case GRAM_BF16X3: hipLaunchKernelGGL((k_rowsum<float, KSRC_RECOMPUTE, GRAM_BF16X3>), g, b, 0, s, nullptr, F, kp, tiles, NB, psum, pmax); break;
            case GRAM_BF16X6: hipLaunchKernelGGL((k_rowsum<float, KSRC_RECOMPUTE, GRAM_BF16X6>), g, b, 0, s, nullptr, F, kp, tiles, NB, psum, pmax); break;
            default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

hipError_t launch_residual(const void* Kp, int prec, int ksrc, const Features& F, const KernelParams& kp,
                           const uint32_t* tiles, int64_t ntiles, int NB, int64_t N, int64_t NPAD,
                           const double* alpha, const float* y, const double* Adiag, const double* rsum,
                           double* w, double* part, double* blk1, double* blk2, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_weights, dim3(grid1(NPAD)), dim3(WG), 0, s, N, NPAD, alpha, y, w);
    if (ntiles > kMaxBlocks && ksrc == KSRC_PLANE) return hipErrorInvalidValue;
    const dim3 b(WG);
    if (ksrc == KSRC_PLANE) {
        const dim3 g((unsigned)ntiles);
        if (prec == PREC_FP64)
            hipLaunchKernelGGL((k_apply<double, KSRC_PLANE, GRAM_F64>), g, b, 0, s, (const double*)Kp, F, kp, tiles, NB, w, part);
        else
            hipLaunchKernelGGL((k_apply<float, KSRC_PLANE, GRAM_F32>), g, b, 0, s, (const float*)Kp, F, kp, tiles, NB, w, part);
    } else {
        const hipError_t e = in_launches(ntiles, [&](int64_t o, int64_t n) {
            const dim3 g((unsigned)n);
            const uint32_t* t = tiles + o;
            switch (F.kind) {
                case GRAM_F32: hipLaunchKernelGGL((k_apply<float, KSRC_RECOMPUTE, GRAM_F32>), g, b, 0, s, nullptr, F, kp, t, NB, w, part); break;
                case GRAM_BF16: hipLaunchKernelGGL((k_apply<float, KSRC_RECOMPUTE, GRAM_BF16>), g, b, 0, s, nullptr, F, kp, t, NB, w, part); break;
                case GRAM_BF16X3: hipLaunchKernelGGL((k_apply<float, KSRC_RECOMPUTE, GRAM_BF16X3>), g, b, 0, s, nullptr, F, kp, t, NB, w, part); break;
                case GRAM_BF16X6: hipLaunchKernelGGL((k_apply<float, KSRC_RECOMPUTE, GRAM_BF16X6>), g, b, 0, s, nullptr, F, kp, t, NB, w, part); break;
                default: return hipErrorInvalidValue;
            }
            return hipGetLastError();
        });
        if (e != hipSuccess) return e;
    }
    const unsigned nb = grid1(N);
    hipLaunchKernelGGL(k_residual_blocks, dim3(nb), dim3(WG), 0, s, N, NB, part, Adiag, rsum, alpha, y, blk1, blk2);
    hipLaunchKernelGGL(k_residual_final, dim3(1), dim3(WG), 0, s, (int)nb, blk1, blk2, out);
    return hipGetLastError();
}

hipError_t launch_diag(int64_t N, int NB, const double* psum, const double* pmax, const double* kdiag,
                       int mode, double C, double delta, double* Adiag, double* rowmax, double* rsum,
                       double* scratch_blk, double* scratch_one, hipStream_t s) {
    const unsigned nb = grid1(N);
    hipLaunchKernelGGL(k_diag, dim3(nb), dim3(WG), 0, s, N, NB, psum, pmax, kdiag, mode, C, delta, Adiag,
                       rowmax, rsum, scratch_blk);
    if (mode == 3) {
        hipLaunchKernelGGL(k_max_reduce, dim3(1), dim3(WG), 0, s, (int)nb, scratch_blk, scratch_one);
        hipLaunchKernelGGL(k_diag_shift, dim3(nb), dim3(WG), 0, s, N, kdiag, scratch_one, Adiag);
    }
    return hipGetLastError();
}

hipError_t launch_init(int prec, int64_t N, int64_t NPAD, int R, const double* Adiag, const float* y,
                       void* Pt, void* S, double* alpha, DevStatus* st, hipStream_t s, double boxC) {
    hipLaunchKernelGGL(k_reset_status, dim3(1), dim3(64), 0, s, st);
    if (prec == PREC_FP32)
        hipLaunchKernelGGL(k_init<float>, dim3(grid1(NPAD)), dim3(WG), 0, s, N, NPAD, R, Adiag, y,
                           (float*)Pt, (float*)S, alpha, st, boxC);
    else
        hipLaunchKernelGGL(k_init<double>, dim3(grid1(NPAD)), dim3(WG), 0, s, N, NPAD, R, Adiag, y,
                           (double*)Pt, (double*)S, alpha, st, boxC);
    return hipGetLastError();
}

// Per-precision sweep dispatch lives in gabp_sweep_{f32,mixed,f64}.hip.
hipError_t launch_sweep(int prec, int ksrc, int gram, int levels, bool first, int ser, const SweepArgs& a,
                        hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (levels == 0) ser = 0;
    switch (prec) {
        case PREC_FP32: return launch_sweep_f32(ksrc, gram, levels, first, ser, a, s, e0, e1);
        case PREC_MIXED: return launch_sweep_mixed(ksrc, gram, levels, first, ser, a, s, e0, e1);
        case PREC_FP64: return launch_sweep_f64(ksrc, gram, levels, first, ser, a, s, e0, e1);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sweep_grouped(int prec, int ksrc, int gram, int levels, int ser, const SweepArgs& a,
                                const uint32_t* within, int nwithin, const uint32_t* dir, int ndir, int t,
                                hipStream_t s) {
    if (levels == 0) ser = 0;
    switch (prec) {
        case PREC_FP32: return launch_sweep_grouped_f32(ksrc, gram, levels, ser, a, within, nwithin, dir, ndir, t, s);
        case PREC_MIXED: return launch_sweep_grouped_mixed(ksrc, gram, levels, ser, a, within, nwithin, dir, ndir, t, s);
        case PREC_FP64: return launch_sweep_grouped_f64(ksrc, gram, levels, ser, a, within, nwithin, dir, ndir, t, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_served_sweep(int prec, int levels, int ser, bool grouped, const ReqDesc* reqs, const uint2* items,
                               int n, hipStream_t s) {
    switch (prec) {
        case PREC_FP32: return launch_served_sweep_f32(levels, ser, grouped, reqs, items, n, s);
        case PREC_MIXED: return launch_served_sweep_mixed(levels, ser, grouped, reqs, items, n, s);
        case PREC_FP64: return launch_served_sweep_f64(levels, ser, grouped, reqs, items, n, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_served_finalize(bool agg_f32, const ReqDesc* reqs, const uint2* items, int n, hipStream_t s) {
    const int gf = std::max(1, std::min(n * (TILE / FB), 8192));
    if (agg_f32)
        hipLaunchKernelGGL(k_finalize_batched<float>, dim3(gf), dim3(WG), 0, s, reqs, items, n);
    else
        hipLaunchKernelGGL(k_finalize_batched<double>, dim3(gf), dim3(WG), 0, s, reqs, items, n);
    return hipGetLastError();
}

hipError_t launch_served_status(const ReqDesc* reqs, const int* slots, int nslots, DevStatus* status_out,
                                hipStream_t s) {
    hipLaunchKernelGGL(k_status_grouped, dim3(std::max(1, nslots)), dim3(WG), 0, s, reqs, slots, nslots, status_out);
    return hipGetLastError();
}

// Above this many finalize workgroups the stop rule is a launch of its own.
// One launch less saves 1.2 us a sweep at 47 workgroups (N = 3,001: 21.6 ->
// 20.4 us) and 0.8 at 125 (N = 8,000: 47.9 -> 47.1); the ticket that every
// workgroup waits for before it ends costs 1.1 us more at 313 (N = 20,000:
// 160.2 -> 161.3), 2.8 at 500 (369.2 -> 372.0) and 11 at 1,563 (3,324 -> 3,335).
constexpr int64_t kFuseStatusMax = 256;

hipError_t launch_finalize(int prec, const FinalizeArgs& f, hipStream_t s) {
    if ((f.Inv == nullptr) != (f.Mean == nullptr)) return hipErrorInvalidValue;
    const int64_t nb = (f.N + FB - 1) / FB, b0 = f.b0 * (TILE / FB);
    const int64_t b1 = f.b1 > 0 ? std::min(nb, f.b1 * (TILE / FB)) : nb;
    if (b1 <= b0) return f.trace ? hipErrorInvalidValue : hipSuccess;
    const dim3 g((unsigned)(b1 - b0)), b(WG);
    FinalizeArgs a = f;
    const bool own = f.trace && b1 - b0 > kFuseStatusMax;
    if (own) a.trace = nullptr;
    if (prec == PREC_FP32) hipLaunchKernelGGL((k_finalize<float, float>), g, b, 0, s, a);
    else if (f.part32) hipLaunchKernelGGL((k_finalize<double, float>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_finalize<double, double>), g, b, 0, s, a);
    if (own) hipLaunchKernelGGL(k_status, dim3(1), b, 0, s, f);
    return hipGetLastError();
}

hipError_t launch_ring_recip(int prec, int64_t NPAD, int R, const void* Pt, const void* S, void* Inv, void* Mean,
                             hipStream_t s) {
    const int64_t n = NPAD * (int64_t)R;
    if (prec == PREC_FP32)
        hipLaunchKernelGGL(k_ring_recip<float>, dim3(grid1(n)), dim3(WG), 0, s, n, (const float*)Pt,
                           (const float*)S, (float*)Inv, (float*)Mean);
    else
        hipLaunchKernelGGL(k_ring_recip<double>, dim3(grid1(n)), dim3(WG), 0, s, n, (const double*)Pt,
                           (const double*)S, (double*)Inv, (double*)Mean);
    return hipGetLastError();
}

hipError_t launch_rho_bound(int64_t N, const double* Adiag, const double* rowmax, const double* rsum,
                            double* blk, double* one, hipStream_t s) {
    const unsigned nb = grid1(N);
    hipLaunchKernelGGL(k_bound_root, dim3(nb), dim3(WG), 0, s, N, Adiag, rowmax, rsum, blk);
    hipLaunchKernelGGL(k_max_reduce, dim3(1), dim3(WG), 0, s, (int)nb, blk, one);
    hipLaunchKernelGGL(k_bound_rho, dim3(nb), dim3(WG), 0, s, N, Adiag, rowmax, rsum, one, blk);
    hipLaunchKernelGGL(k_max_reduce, dim3(2), dim3(WG), 0, s, (int)nb, blk, one + 1);
    return hipGetLastError();
}

hipError_t launch_kernel_entries(const void* Kp, int prec, int NB, const int64_t* rows,
                                 const int64_t* cols, int64_t n, double* out, hipStream_t s) {
    if (prec == PREC_FP64)
        hipLaunchKernelGGL(k_entries<double>, dim3(grid1(n)), dim3(WG), 0, s, (const double*)Kp, NB,
                           rows, cols, n, out);
    else
        hipLaunchKernelGGL(k_entries<float>, dim3(grid1(n)), dim3(WG), 0, s, (const float*)Kp, NB,
                           rows, cols, n, out);
    return hipGetLastError();
}

hipError_t launch_pack_out(int prec, int64_t N, const double* alpha, const void* Pt, int stride, const double* Adiag,
                           const float* y, const int32_t* order, double* out, hipStream_t s) {
    if (prec == PREC_FP32)
        hipLaunchKernelGGL(k_pack_out<float>, dim3(grid1(N)), dim3(WG), 0, s, N, alpha, (const float*)Pt, stride, Adiag,
                           y, order, out);
    else
        hipLaunchKernelGGL(k_pack_out<double>, dim3(grid1(N)), dim3(WG), 0, s, N, alpha, (const double*)Pt, stride,
                           Adiag, y, order, out);
    return hipGetLastError();
}

}  // namespace gabp

