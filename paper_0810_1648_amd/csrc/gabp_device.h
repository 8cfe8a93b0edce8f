// Device-side building blocks shared by the HIP translation units of the
// GaBP SVM solver: vector loads, wave reductions, MFMA Gram tiles, and the
// sweep of one tile (see gabp_kernels.hip for the data layout).
#pragma once

#include "gabp_internal.h"

#include <hip/hip_ext.h>

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace gabp {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4v __attribute__((ext_vector_type(4)));

// ----------------------------------------------------------------- helpers

template <class T> struct V4 { T v[4]; };

__device__ inline V4<float> ld4(const float* p) {
    const float4 x = *reinterpret_cast<const float4*>(p);
    return {{x.x, x.y, x.z, x.w}};
}
__device__ inline V4<double> ld4(const double* p) {
    const double2 a = *reinterpret_cast<const double2*>(p);
    const double2 b = *reinterpret_cast<const double2*>(p + 2);
    return {{a.x, a.y, b.x, b.y}};
}
__device__ inline void st4(float* p, const V4<float>& v) {
    *reinterpret_cast<float4*>(p) = make_float4(v.v[0], v.v[1], v.v[2], v.v[3]);
}
__device__ inline void st4(double* p, const V4<double>& v) {
    *reinterpret_cast<double2*>(p) = make_double2(v.v[0], v.v[1]);
    *reinterpret_cast<double2*>(p + 2) = make_double2(v.v[2], v.v[3]);
}

// Streaming accesses of the K' and pair-record planes: every element is used
// once per sweep, so loads and stores carry the non-temporal hint and leave
// the caches to the aggregates and partial sums.
__device__ inline V4<float> ld4nt(const float* p) {
    const f32x4v x = __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(p));
    return {{x[0], x[1], x[2], x[3]}};
}
__device__ inline void st4nt(float* p, const V4<float>& v) {
    const f32x4v x = {v.v[0], v.v[1], v.v[2], v.v[3]};
    __builtin_nontemporal_store(x, reinterpret_cast<f32x4v*>(p));
}
typedef double f64x2v __attribute__((ext_vector_type(2)));
__device__ inline V4<double> ld4nt(const double* p) {
    const f64x2v a = __builtin_nontemporal_load(reinterpret_cast<const f64x2v*>(p));
    const f64x2v b = __builtin_nontemporal_load(reinterpret_cast<const f64x2v*>(p + 2));
    return {{a[0], a[1], b[0], b[1]}};
}
__device__ inline void st4nt(double* p, const V4<double>& v) {
    const f64x2v a = {v.v[0], v.v[1]}, b = {v.v[2], v.v[3]};
    __builtin_nontemporal_store(a, reinterpret_cast<f64x2v*>(p));
    __builtin_nontemporal_store(b, reinterpret_cast<f64x2v*>(p + 2));
}

// K' row steps in flight per lane in the stateless sweep over an FP32 K'
// plane: each wave streams its row steps into an LDS ring by direct
// global-to-LDS loads, so the bytes in flight do not occupy registers.
#ifndef GABP_KRING
#define GABP_KRING 4
#endif
constexpr int KRING = GABP_KRING;

// LDS byte offset of a shared-memory pointer (wave-uniform here).
__device__ inline uint32_t lds_offset(const void* p) {
    return (uint32_t)reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)p);
}

// One direct global-to-LDS load of 16 bytes per lane: lane l's bytes at
// base + voff land at LDS offset lds + 16 l, with the non-temporal hint.  The
// compiler's wait counting does not see this load: callers wait for it with
// wait_vm before reading the LDS it writes, and issue it only after their
// last read of that LDS has completed.
__device__ inline void dma16(const float* base, uint32_t voff, uint32_t lds) {
    // the base and the LDS offset are wave-uniform: scalar operands
    lds = __builtin_amdgcn_readfirstlane(lds);
    // (the builtin returns a signed int: each half goes through uint32_t so
    // that the low half is zero-extended, never sign-extended)
    const uint64_t b = reinterpret_cast<uint64_t>(base);
    const uint32_t bh = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    const uint32_t bl = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    base = reinterpret_cast<const float*>(((uint64_t)bh << 32) | (uint64_t)bl);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                 :: "v"(voff), "s"(base), "s"(lds) : "memory", "m0");
}
// Waits until at most N vector-memory operations of this wave are in flight.
template <int N> __device__ inline void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// Device-scope accesses of values that workgroups of one launch hand to each
// other: written through to, and read from, where every XCD sees them.
template <class T> __device__ inline void store_agent(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T> __device__ inline T load_agent(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Address of a lane's element from a wave-uniform base (scalar registers)
// and a 32-bit lane offset: loads and stores then take the scalar-base form
// and the per-step address arithmetic stays off the vector ALU.
template <class T> __device__ inline T* lane_ptr(T* base, uint32_t elems) {
    using C = typename std::conditional<std::is_const<T>::value, const char, char>::type;
    return reinterpret_cast<T*>(reinterpret_cast<C*>(base) + elems * (uint32_t)sizeof(T));
}

template <int CTRL> __device__ inline int dpp_i(int v) {
    // every source lane of these patterns exists, so no fill value is needed
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}
template <int CTRL> __device__ inline float dpp(float v) {
    return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}
template <int CTRL> __device__ inline double dpp(double v) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const int lo = dpp_i<CTRL>((int)(unsigned)(u & 0xffffffffull));
    const int hi = dpp_i<CTRL>((int)(unsigned)(u >> 32));
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) |
                                            (unsigned long long)(unsigned)lo));
}
// Sum over the 16 lanes of a DPP row; every lane receives the same bits.
template <class T> __device__ inline T sum16(T v) {
    v = v + dpp<0xB1>(v);    // quad_perm(1,0,3,2): pairs
    v = v + dpp<0x4E>(v);    // quad_perm(2,3,0,1): quads
    v = v + dpp<0x141>(v);   // row_half_mirror: 8 lanes
    v = v + dpp<0x140>(v);   // row_mirror: 16 lanes
    return v;
}
// Sum over lanes q, q+16, q+32, q+48 in the fixed order (g0+g1)+(g2+g3).
template <class T> __device__ inline T sum_groups(T v) {
    v = v + __shfl_xor(v, 16);
    v = v + __shfl_xor(v, 32);
    return v;
}
__device__ inline double wave_max(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}
// Block (256 threads) max; result valid in every thread.
__device__ inline double block_max(double v, double* sh4) {
    v = wave_max(v);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sh4[w] = v;
    __syncthreads();
    v = fmax(fmax(sh4[0], sh4[1]), fmax(sh4[2], sh4[3]));
    __syncthreads();
    return v;
}

// Stop rule (Algorithm 2 step "Check", tested on alpha).
__device__ inline void status_update(int nblk, const double* __restrict__ bd,
                                     const double* __restrict__ ba, DevStatus* st,
                                     double* __restrict__ trace, const StopRule& rule) {
    __shared__ double sh4[4];
    double d = 0.0, a = 0.0;
    for (int k = threadIdx.x; k < nblk; k += blockDim.x) {
        d = fmax(d, load_agent(bd + k));
        a = fmax(a, load_agent(ba + k));
    }
    d = block_max(d, sh4);
    a = block_max(a, sh4);
    if (threadIdx.x == 0) {
        const int t = st->t + 1;
        st->t = t;
        st->delta = d;
        st->amax = a;
        trace[t - 1] = d;
        if (load_agent(&st->bad)) {
            st->done = 1; st->reason = R_DIVERGED;
        } else if (d <= rule.tol_abs + rule.tol_rel * a) {
            st->done = 1; st->reason = R_CONVERGED;
        } else {
            if (d < st->best_delta) { st->best_delta = d; st->since_best = 0; }
            else st->since_best = st->since_best + 1;
            if (rule.stag_window > 0 && st->since_best >= rule.stag_window && d <= rule.stag_rel * a) {
                st->done = 1; st->reason = R_STAGNATED;
            } else if (t >= rule.max_sweeps) {
                st->done = 1; st->reason = R_MAX_SWEEPS;
            }
        }
    }
}

__device__ inline uint16_t f2bf(float f) {  // round to nearest even
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// v = h + l + l2 in BF16 (each the rounding of the remainder left by the
// terms before it): h alone carries about 2^-9 of v, h + l about 2^-18,
// h + l + l2 about 2^-27.
__device__ inline void split3(float v, uint16_t& h, uint16_t& l, uint16_t& l2) {
    h = f2bf(v);
    const float r = v - bf2f(h);
    l = f2bf(r);
    l2 = f2bf(r - bf2f(l));
}

// Reciprocals: v_rcp_f32 (1 ulp) for FP32; for FP64, v_rcp_f64 refined by
// two Newton steps (the cavity precisions are far from the denormal range).
__device__ inline float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double rcp_fast(double x) {
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    return __builtin_isinf(x) ? 0.0 : r;    // 1/inf = 0 (Newton would give NaN)
}

// ... of a finite positive argument.
__device__ inline float rcp_pos(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ inline double rcp_pos(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// Workgroups go to the eight XCDs in turn (workgroup b to XCD b mod 8).
// This index of workgroup b in [0, n) (n = the grid) gives every XCD one
// contiguous range instead, so that work items sharing data (neighbouring
// nodes and edges, tiles of one super-block) meet in the same L2.
__device__ inline int64_t xcd_contiguous(int64_t b, int64_t n) {
    const int64_t x = b & 7, q = b >> 3, base = n >> 3, rem = n & 7;
    return x * base + (x < rem ? x : rem) + q;
}

struct TileCoord { int I, J; };
__device__ inline TileCoord tile_of(const uint32_t* tiles) {
    const uint32_t ij = tiles[blockIdx.x];
    return {(int)(ij >> 16), (int)(ij & 0xFFFFu)};
}

// ------------------------------------------------------------ K' build --

// One 32 x 32 block of the Gram matrix x_a . x_b on MFMA, for A rows
// rowA = base_a + lane % 32 and B rows colB = base_b + lane % 32.  The
// inner-product index is split between the two lane halves so that each lane
// reads contiguous features.  Output layout of the 32x32 MFMAs: register r of
// lane l holds row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
// The A rows come from FA and the B rows from FB (the same staging: m_pad
// and kind are taken from FA).
template <int KIND>
__device__ inline f32x16 mfma_gram_32x32(const Features& FA, int64_t rowA, const Features& FB, int64_t colB) {
    const int l = threadIdx.x & 63, h = l >> 5;
    const int mp = FA.m_pad;
    f32x16 acc = {};
    if constexpr (KIND == GRAM_F32) {
        const int half = mp >> 1;
        const float* pa = FA.f32 + rowA * mp + h * half;
        const float* pb = FB.f32 + colB * mp + h * half;
        for (int s = 0; s < half; s += 4) {
            const f32x4v a4 = *reinterpret_cast<const f32x4v*>(pa + s);
            const f32x4v b4 = *reinterpret_cast<const f32x4v*>(pb + s);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[0], b4[0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[1], b4[1], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[2], b4[2], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[3], b4[3], acc, 0, 0, 0);
        }
    } else {
        const int64_t oa = rowA * mp + 8 * h, ob = colB * mp + 8 * h;
        for (int s = 0; s < mp; s += 16) {
            const bf16x8 a = *reinterpret_cast<const bf16x8*>(FA.hi + oa + s);
            const bf16x8 b = *reinterpret_cast<const bf16x8*>(FB.hi + ob + s);
            if constexpr (KIND == GRAM_BF16X3 || KIND == GRAM_BF16X6) {
                // correction terms first, then the leading product
                const bf16x8 al = *reinterpret_cast<const bf16x8*>(FA.lo + oa + s);
                const bf16x8 bl = *reinterpret_cast<const bf16x8*>(FB.lo + ob + s);
                if constexpr (KIND == GRAM_BF16X6) {
                    const bf16x8 a2 = *reinterpret_cast<const bf16x8*>(FA.lo2 + oa + s);
                    const bf16x8 b2 = *reinterpret_cast<const bf16x8*>(FB.lo2 + ob + s);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b2, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, b, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bl, acc, 0, 0, 0);
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bl, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, b, acc, 0, 0, 0);
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
        }
    }
    return acc;
}

template <int KIND>
__device__ inline f32x16 mfma_gram_32x32(const Features& F, int64_t rowA, int64_t colB) {
    return mfma_gram_32x32<KIND>(F, rowA, F, colB);
}

// A operand (32 rows) of the MFMA Gram, held in registers while a wave walks
// many 32-row B blocks, when m_pad <= MP; MP = 0 reloads it every block.
template <int KIND, int MP> struct RowFrag {
    static constexpr int NS = (KIND == GRAM_F32) ? MP / 8 : MP / 16;
    static constexpr int NSA = NS > 0 ? NS : 1;
    f32x4v f[KIND == GRAM_F32 ? NSA : 1];
    bf16x8 hi[KIND == GRAM_F32 ? 1 : NSA];
    bf16x8 lo[(KIND == GRAM_BF16X3 || KIND == GRAM_BF16X6) ? NSA : 1];
    bf16x8 lo2[KIND == GRAM_BF16X6 ? NSA : 1];

    __device__ void load(const Features& Fq, int64_t rowA) {
        if constexpr (MP > 0) {
            const int l = threadIdx.x & 63, h = l >> 5, mp = Fq.m_pad;
            if constexpr (KIND == GRAM_F32) {
                const int half = mp >> 1;
                const float* pa = Fq.f32 + rowA * mp + h * half;
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (4 * s < half) f[s] = *reinterpret_cast<const f32x4v*>(pa + 4 * s);
            } else {
                const int64_t oa = rowA * mp + 8 * h;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (16 * s >= mp) continue;
                    hi[s] = *reinterpret_cast<const bf16x8*>(Fq.hi + oa + 16 * s);
                    if constexpr (KIND == GRAM_BF16X3 || KIND == GRAM_BF16X6)
                        lo[s] = *reinterpret_cast<const bf16x8*>(Fq.lo + oa + 16 * s);
                    if constexpr (KIND == GRAM_BF16X6)
                        lo2[s] = *reinterpret_cast<const bf16x8*>(Fq.lo2 + oa + 16 * s);
                }
            }
        }
    }

    // Two A blocks (a0, a1) against the same B rows: each B fragment is
    // loaded once for both MFMA chains.
    __device__ static void gram2(const RowFrag& a0, const RowFrag& a1, const Features& Fq, int64_t rowA0,
                                 int64_t rowA1, const Features& Ft, int64_t colB, f32x16& acc0, f32x16& acc1) {
        if constexpr (MP == 0) {
            acc0 = mfma_gram_32x32<KIND>(Fq, rowA0, Ft, colB);
            acc1 = mfma_gram_32x32<KIND>(Fq, rowA1, Ft, colB);
        } else {
            const int l = threadIdx.x & 63, h = l >> 5, mp = Ft.m_pad;
            acc0 = f32x16{};
            acc1 = f32x16{};
            if constexpr (KIND == GRAM_F32) {
                const int half = mp >> 1;
                const float* pb = Ft.f32 + colB * mp + h * half;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (4 * s >= half) continue;
                    const f32x4v b4 = *reinterpret_cast<const f32x4v*>(pb + 4 * s);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.f[s][e], b4[e], acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.f[s][e], b4[e], acc1, 0, 0, 0);
                    }
                }
            } else {
                const int64_t ob = colB * mp + 8 * h;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (16 * s >= mp) continue;
                    const bf16x8 b = *reinterpret_cast<const bf16x8*>(Ft.hi + ob + 16 * s);
                    if constexpr (KIND == GRAM_BF16X3 || KIND == GRAM_BF16X6) {
                        const bf16x8 bl = *reinterpret_cast<const bf16x8*>(Ft.lo + ob + 16 * s);
                        if constexpr (KIND == GRAM_BF16X6) {
                            const bf16x8 b2 = *reinterpret_cast<const bf16x8*>(Ft.lo2 + ob + 16 * s);
                            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0.hi[s], b2, acc0, 0, 0, 0);
                            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1.hi[s], b2, acc1, 0, 0, 0);
                            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0.lo2[s], b, acc0, 0, 0, 0);
                            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1.lo2[s], b, acc1, 0, 0, 0);
                            acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0.lo[s], bl, acc0, 0, 0, 0);
                            acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1.lo[s], bl, acc1, 0, 0, 0);
                        }
                        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0.hi[s], bl, acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1.hi[s], bl, acc1, 0, 0, 0);
                        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0.lo[s], b, acc0, 0, 0, 0);
                        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1.lo[s], b, acc1, 0, 0, 0);
                    }
                    acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0.hi[s], b, acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1.hi[s], b, acc1, 0, 0, 0);
                }
            }
        }
    }

    // Gram block of the 32 A rows with the B rows colB (one per lane % 32).
    __device__ f32x16 gram(const Features& Fq, int64_t rowA, const Features& Ft, int64_t colB) const {
        if constexpr (MP == 0) {
            return mfma_gram_32x32<KIND>(Fq, rowA, Ft, colB);
        } else {
            const int l = threadIdx.x & 63, h = l >> 5, mp = Ft.m_pad;
            f32x16 acc = {};
            if constexpr (KIND == GRAM_F32) {
                const int half = mp >> 1;
                const float* pb = Ft.f32 + colB * mp + h * half;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (4 * s >= half) continue;
                    const f32x4v b4 = *reinterpret_cast<const f32x4v*>(pb + 4 * s);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[s][0], b4[0], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[s][1], b4[1], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[s][2], b4[2], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[s][3], b4[3], acc, 0, 0, 0);
                }
            } else {
                const int64_t ob = colB * mp + 8 * h;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    if (16 * s >= mp) continue;
                    const bf16x8 b = *reinterpret_cast<const bf16x8*>(Ft.hi + ob + 16 * s);
                    if constexpr (KIND == GRAM_BF16X3 || KIND == GRAM_BF16X6) {
                        const bf16x8 bl = *reinterpret_cast<const bf16x8*>(Ft.lo + ob + 16 * s);
                        if constexpr (KIND == GRAM_BF16X6) {
                            const bf16x8 b2 = *reinterpret_cast<const bf16x8*>(Ft.lo2 + ob + 16 * s);
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi[s], b2, acc, 0, 0, 0);
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo2[s], b, acc, 0, 0, 0);
                            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo[s], bl, acc, 0, 0, 0);
                        }
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi[s], bl, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo[s], b, acc, 0, 0, 0);
                    }
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi[s], b, acc, 0, 0, 0);
                }
            }
            return acc;
        }
    }
};

// acc += A B^T for register-held fragments of 32 A rows and 32 B rows (both
// loaded with RowFrag::load; MP > 0), in the products order of
// mfma_gram_32x32 (correction terms first).  Loading the next B fragment
// before this call hides its latency behind the MFMA chain.
template <int KIND, int MP>
__device__ inline void frag_mma(const RowFrag<KIND, MP>& a, const RowFrag<KIND, MP>& b, f32x16& acc, int mp) {
    static_assert(MP > 0, "register fragments only");
    constexpr int NS = RowFrag<KIND, MP>::NS;
    if constexpr (KIND == GRAM_F32) {
        const int half = mp >> 1;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (4 * s >= half) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.f[s][e], b.f[s][e], acc, 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (16 * s >= mp) continue;
            if constexpr (KIND == GRAM_BF16X3 || KIND == GRAM_BF16X6) {
                if constexpr (KIND == GRAM_BF16X6) {
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi[s], b.lo2[s], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.lo2[s], b.hi[s], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.lo[s], b.lo[s], acc, 0, 0, 0);
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi[s], b.lo[s], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.lo[s], b.hi[s], acc, 0, 0, 0);
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi[s], b.hi[s], acc, 0, 0, 0);
        }
    }
}

// B fragments of a 32-row block staged in LDS (BF16 splits), shared by the
// waves of a workgroup.  Chunk k of a block (k < planes x 64 x ns, ns =
// m_pad / 16) is 16 bytes of one staged row: plane k / (64 ns), row and
// 16-byte column of the row-major features, so that consecutive threads load
// consecutive bytes; its slot is the fragment order (plane, k-step, lane),
// lane = 32 (column / 2 parity) + row, so that a wave reads the operand of
// k-step s as 64 consecutive chunks.
template <int KIND> struct BStage {
    static constexpr int NP = (KIND == GRAM_BF16X6) ? 3 : (KIND == GRAM_BF16X3) ? 2 : 1;
    __device__ static const bf16x8* src(const Features& F, int64_t row0, int ns, int k) {
        const int pl = k / (64 * ns), rem = k - pl * 64 * ns, row = rem / (2 * ns), cc = rem - row * 2 * ns;
        const uint16_t* base = (pl == 0) ? F.hi : (pl == 1) ? F.lo : F.lo2;
        return reinterpret_cast<const bf16x8*>(base + (row0 + row) * F.m_pad + 8 * cc);
    }
    __device__ static int dst(int ns, int k) {
        const int pl = k / (64 * ns), rem = k - pl * 64 * ns, row = rem / (2 * ns), cc = rem - row * 2 * ns;
        return (pl * ns + (cc >> 1)) * 64 + (cc & 1) * 32 + row;
    }
    // acc += A B^T with A in registers and B staged at sb (the products of
    // frag_mma, in its order)
    template <int MP>
    __device__ static void mma(const RowFrag<KIND, MP>& a, const bf16x8* sb, int ns, int l, f32x16& acc) {
#pragma unroll
        for (int st = 0; st < MP / 16; ++st) {
            if (st >= ns) continue;
            const bf16x8 bh = sb[(0 * ns + st) * 64 + l];
            if constexpr (NP >= 2) {
                const bf16x8 bl = sb[(1 * ns + st) * 64 + l];
                if constexpr (NP >= 3) {
                    const bf16x8 bl2 = sb[(2 * ns + st) * 64 + l];
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi[st], bl2, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.lo2[st], bh, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.lo[st], bl, acc, 0, 0, 0);
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi[st], bl, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.lo[st], bh, acc, 0, 0, 0);
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi[st], bh, acc, 0, 0, 0);
        }
    }
};

// K' = exp(-gamma d^2) + lambda^2 with d^2 = max(0, n_i + n_j - 2 G_ij), zero
// for pairs that are not strictly upper (i >= j) or are padding (j >= N).
// K' from a Gram entry: exp2 of the scaled, clamped distance on the
// hardware exp2 (v_exp_f32; results below 2^-126 flush to zero, which the
// lambda^2 added next absorbs), plus lambda^2.
__device__ inline float kernel_value(float ni, float nj, float g, const KernelParams& kp) {
    const float d2 = fmaxf(ni + nj - 2.0f * g, 0.0f);
    return __builtin_amdgcn_exp2f(kp.neg_gamma_log2e * d2) + (float)kp.lam2;
}
// ... and zero outside the strict upper triangle and past N.
__device__ inline float kernel_entry(float ni, float nj, float g, int64_t i, int64_t j,
                                     const KernelParams& kp) {
    const float kv = kernel_value(ni, nj, g, kp);
    return (i < j && j < kp.N) ? kv : 0.0f;
}

// K' for the 32 x 64 band [row0, row0 + 32) x [col0, col0 + 64) of tile
// (I, J), computed by one wave into its LDS buffer kb[32][64] (row-major).
template <int KIND>
__device__ inline void gram_band(const Features& F, const KernelParams& kp, int I, int J, int row0,
                                 int col0, float* kb) {
    const int l = threadIdx.x & 63, h = l >> 5, l32 = l & 31;
    const int64_t rowA = (int64_t)I * TILE + row0 + l32;
    // the index test matters only on diagonal tiles and in the last column block
    const bool plain = (I < J) && ((int64_t)J * TILE + col0 + 64 <= kp.N);
    if constexpr (KIND != GRAM_F32) {
        if (F.aug0) {
            // augmented rows: the MFMA output is the exponent (clamped at 0,
            // the largest value of -gamma log2(e) d^2), K' = exp2 + lambda^2
            Features FA = F, FB = F;
            FA.hi = F.aug0; FA.lo = F.aug0 + F.aug_plane; FA.lo2 = F.aug0 + 2 * F.aug_plane;
            FB.hi = F.aug1; FB.lo = F.aug1 + F.aug_plane; FB.lo2 = F.aug1 + 2 * F.aug_plane;
            const float lam2 = (float)kp.lam2;
#pragma unroll 1
            for (int cb = 0; cb < 2; ++cb) {
                const int64_t colB = (int64_t)J * TILE + col0 + 32 * cb + l32;
                const f32x16 acc = mfma_gram_32x32<KIND>(FA, rowA, FB, colB);
                float* kl = kb + 4 * h * 64 + 32 * cb + l32;
                if (plain) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        kl[(8 * (r >> 2) + (r & 3)) * 64] = __builtin_amdgcn_exp2f(fminf(acc[r], 0.0f)) + lam2;
                } else {
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int64_t i = (int64_t)I * TILE + row0 + 8 * (r >> 2) + 4 * h + (r & 3);
                        const float kv = __builtin_amdgcn_exp2f(fminf(acc[r], 0.0f)) + lam2;
                        kl[(8 * (r >> 2) + (r & 3)) * 64] = (i < colB && colB < kp.N) ? kv : 0.0f;
                    }
                }
            }
            return;
        }
    }
    float ni[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) ni[r] = F.nrm[(int64_t)I * TILE + row0 + 8 * (r >> 2) + 4 * h + (r & 3)];
#pragma unroll 1
    for (int cb = 0; cb < 2; ++cb) {
        const int64_t colB = (int64_t)J * TILE + col0 + 32 * cb + l32;
        const f32x16 acc = mfma_gram_32x32<KIND>(F, rowA, colB);
        const float nj = F.nrm[colB];
        // the lane's column of its row half: the 16 rows sit at constant offsets
        float* kl = kb + 4 * h * 64 + 32 * cb + l32;
        if (plain) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                kl[(8 * (r >> 2) + (r & 3)) * 64] = kernel_value(ni[r], nj, acc[r], kp);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 8 * (r >> 2) + 4 * h + (r & 3);
                kl[(8 * (r >> 2) + (r & 3)) * 64] =
                    kernel_entry(ni[r], nj, acc[r], (int64_t)I * TILE + row0 + row, colB, kp);
            }
        }
    }
}

__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------ sweep --

// Sums of one tile's messages: the row sums of node `threadIdx.x` of the row
// block, and the column sums of the lane's four columns (every row group of
// a wave holds the same values).
template <class AT>
struct TileSums {
    AT rp, re;
    AT cp[4], ce[4];
};

// Offsets of a tile's partial sums (part_stride, part_slots).
struct PartSlots {
    int NB, split;
    __device__ size_t at(int K, int slot) const { return ((size_t)K * part_stride(NB, split) + slot) * TILE; }
    __device__ size_t row(int I, int J) const { return at(I, I * split + J - I); }
    __device__ size_t col(int I, int J, int sub) const {
        return at(J, I < J ? I * split + sub : J * split + NB - J + sub);
    }
};

// Stores one partial sum of a tile: in FP32 when the plan keeps its partials
// in FP32 (the FP32-message form, whose tile sums are FP32 sums rounded once
// more here), else in the aggregate type.
template <class AT>
__device__ inline void put_part(void* base, size_t o, AT v, bool p32) {
    if (p32) static_cast<float*>(base)[o] = (float)v;
    else static_cast<AT*>(base)[o] = v;
}

// Type of the message arithmetic.  The MIXED path (FP32 storage, FP64
// aggregates) with series reciprocals computes its messages in FP32: the
// cavity denominator P~ - P_reverse is never formed (the series factor
// 1 + e + e^2 has |e| <= rho^2, bounded a priori, so nothing cancels), the
// per-node 1/P~ and S/P~ are rounded once from FP64, and FP32 sums of a few
// messages are added into the FP64 aggregates.  Every other path computes
// its messages in MT.
template <class ST, class MT, class AT, int SER>
struct MsgT {
    static constexpr bool F32 = SER && std::is_same<ST, float>::value && std::is_same<AT, double>::value;
    using T = typename std::conditional<F32, float, MT>::type;
};

// A tile's sums to its partial slots, or, with `out`, to the caller (a chunk
// adds them up first).
template <class AT>
__device__ inline void put_tile_sums(const SweepArgs& a, const TileCoord& tc, AT rowP, AT rowE, const AT (&cP)[4],
                                     const AT (&cE)[4], TileSums<AT>* out, int split, int sub) {
    if (out) {
        out->rp = rowP; out->re = rowE;
#pragma unroll
        for (int c = 0; c < 4; ++c) { out->cp[c] = cP[c]; out->ce[c] = cE[c]; }
        return;
    }
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, rows = TILE / split;
    const bool p32 = a.part32 != 0;
    const PartSlots ps{a.NB, split};
    if (tid / rows == sub) {
        const size_t rowslot = ps.row(tc.I, tc.J) + tid;
        put_part(a.partP, rowslot, rowP, p32);
        put_part(a.partE, rowslot, rowE, p32);
    }
    if (l < 16) {
        const size_t cb = ps.col(tc.I, tc.J, sub) + w * 64 + l * 4;
#pragma unroll
        for (int c = 0; c < 4; ++c) { put_part(a.partP, cb + c, cP[c], p32); put_part(a.partE, cb + c, cE[c], p32); }
    }
}

// Series sweeps of at most three levels as sums over powers of a = K'_ij
// (mom_plan): with u = 1/P~, primes marking the level (u, S of sweep t - 1; u',
// m' = S'/P~' of t - 2; m'' of t - 3) the series' messages into node j expand to
//   P_ij = -a^2 u_i + a^4 u_i^2 u'_j
//   E_ij = -a u_i S_i - a^2 u_i m'_j + a^3 u'_j (u_i^2 S_i - u_i m''_i) + a^4 u_i^2 u'_j m'_j
// (one level: the first term of each; two: m'' = 0; three levels of form 3
// leave out a^5 u_i^2 u'_j^2 m''_i, rr^4, under the rr^3 that form 3 errs by),
// so that a node's sums are its own factors times sums of a^k x_k with
// x_1 = u S, x_2 = u, x_3 = u^2 S - u m'', x_4 = u^2 of its neighbours: per
// pair the powers of a and one FMA per power and direction, 11 VALU slots
// (one level: 5) where the recursion level by level takes 17.  The a^4 terms
// are rr^2 of the message sums: without them a sweep over the plane of 100,000
// points takes 3.26 instead of 3.27 ms and one recomputed from 120,000 points
// 4.97 instead of 5.47, with the precisions P~ off by rr^3.
template <int D, int SER> constexpr bool mom_plan() {   // (not with kSerLevels)
    return SER > 0 && (D == 1 || (D == 2 && SER == 1) || (D == 3 && SER == 3));
}
template <class XT, int D> struct Mom {
    static constexpr bool Q = D >= 2;   // the powers beyond a^2
    XT x1, x2, x3, x4;           // of a node as the source of messages
    XT ku, km;                   // u', m' of a node as their target
};

// W consecutive values of a ring (W = 4: 16-byte aligned).
template <int W, class T> __device__ inline void ld_nodes(const T* p, T (&v)[W]) {
    if constexpr (W == 4) {
        const V4<T> x = ld4(p);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = x.v[c];
    } else {
        static_assert(W == 1, "one node or four");
        v[0] = p[0];
    }
}

// Factors of W consecutive nodes for the moment sums.
template <int W, class XT, int D, class AT>
__device__ inline void mom_nodes(const SweepArgs& a, int slot_top, int64_t node, Mom<XT, D> (&m)[W]) {
    const AT* HP = static_cast<const AT*>(a.HP);
    const AT* HS = static_cast<const AT*>(a.HS);
    const AT* HI = static_cast<const AT*>(a.HI);
    const AT* HM = static_cast<const AT*>(a.HM);
    // 1/P~ and S/P~ from the rings when the finalize formed them (the same
    // IEEE quotients)
    auto inv = [&](int64_t o, AT (&v)[W]) {
        ld_nodes<W>((HI ? HI : HP) + o, v);
        if (!HI)
#pragma unroll
            for (int c = 0; c < W; ++c) v[c] = (AT)1 / v[c];
    };
    auto mean = [&](int64_t o, AT (&v)[W]) {
        ld_nodes<W>((HM ? HM : HS) + o, v);
        if (!HM) {
            AT p[W];
            ld_nodes<W>(HP + o, p);
#pragma unroll
            for (int c = 0; c < W; ++c) v[c] = v[c] / p[c];
        }
    };
    const int64_t o = (int64_t)slot_top * a.NPAD + node;
    const int64_t o1 = (int64_t)((slot_top - 1 + a.R) % a.R) * a.NPAD + node;
    const int64_t o2 = (int64_t)((slot_top - 2 + a.R) % a.R) * a.NPAD + node;
    AT u[W], s[W], ku[W], km[W], mm[W];
    inv(o, u);
    ld_nodes<W>(HS + o, s);
    if constexpr (D >= 2) { inv(o1, ku); mean(o1, km); }
    if constexpr (D >= 3) mean(o2, mm);
#pragma unroll
    for (int c = 0; c < W; ++c) {
        m[c].x1 = (XT)(u[c] * s[c]);
        m[c].x2 = (XT)u[c];
        m[c].x4 = (XT)(u[c] * u[c]);
        if constexpr (D >= 2) {
            m[c].ku = (XT)ku[c];
            m[c].km = (XT)km[c];
            AT z = u[c] * s[c];
            if constexpr (D >= 3) z -= mm[c];
            m[c].x3 = (XT)(u[c] * z);
        } else {
            m[c].x3 = m[c].ku = m[c].km = 0;
        }
    }
}

// Sums of a node's messages from its moment sums.
template <class T, bool Q>
__device__ inline void mom_sums(T m1, T m2, T m3, T m4, T ku, T km, T& p, T& e) {
    if constexpr (Q) {
        p = fma(ku, m4, -m2);
        e = fma(ku, fma(km, m4, m3), -fma(km, m2, m1));
    } else {
        p = -m2;
        e = -m1;
    }
}

// sweep_tile for the plans of mom_plan.
template <class ST, class MT, class AT, int KSRC, int GK, int D, int SER>
__device__ inline void sweep_tile_mom(const SweepArgs& a, int64_t tile, int slot_top, TileSums<AT>* out, int split,
                                      int sub) {
    using XT = typename MsgT<ST, MT, AT, SER>::T;
    constexpr bool XF = MsgT<ST, MT, AT, SER>::F32;
    using MM = Mom<XT, D>;
    constexpr bool Q = MM::Q;
    const uint32_t ij = a.tiles[tile];
    const TileCoord tc{(int)(ij >> 16), (int)(ij & 0xFFFFu)};
    const size_t tbase = (size_t)tile * TT;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, g = l >> 4, q = l & 15;
    const int col0 = w * 64 + q * 4;
    const ST* Kp = static_cast<const ST*>(a.Kp);
    const uint32_t lo = (uint32_t)(g * TILE + col0);
    const int bb0 = sub * (TILE / 32 / split), bb1 = bb0 + TILE / 32 / split;
    const int u0 = 8 * bb0, u1 = 8 * bb1;
    constexpr bool RING = (KSRC == KSRC_PLANE) && std::is_same<ST, float>::value;
    constexpr int KR = RING ? KRING : 1;
    __shared__ __attribute__((aligned(16))) float kring[KR][4][RING ? 256 : 4];
    if constexpr (RING) {
#pragma unroll
        for (int u = 0; u < KR; ++u)
            dma16(reinterpret_cast<const float*>(Kp) + tbase + (size_t)(u0 + u) * 4 * TILE, lo * 4u,
                  lds_offset(&kring[u][w][0]));
    }
    // row nodes: x_1 .. x_4 and (u', m'); column nodes: (u', m'), needed at
    // the end only
    typedef XT X4 __attribute__((ext_vector_type(4)));
    typedef XT X2 __attribute__((ext_vector_type(2)));
    __shared__ X4 sx[TILE];
    __shared__ X2 sk[Q ? TILE : 1], sc[Q ? TILE : 1];
    using RT = typename std::conditional<XF, XT, AT>::type;
    __shared__ RT rP[4][TILE], rE[4][TILE];
    __shared__ RT red[4][2][2][64];
    __shared__ float kband[KSRC == KSRC_RECOMPUTE ? 4 : 1][KSRC == KSRC_RECOMPUTE ? 32 * 64 : 1];
    {
        MM m[1];
        mom_nodes<1, XT, D, AT>(a, slot_top, (int64_t)tc.I * TILE + tid, m);
        sx[tid] = X4{m[0].x1, m[0].x2, m[0].x3, m[0].x4};
        if constexpr (Q) sk[tid] = X2{m[0].ku, m[0].km};
    }
    XT y1[4], y2[4], y3[4], y4[4];
    {
        MM m[4];
        mom_nodes<4, XT, D, AT>(a, slot_top, (int64_t)tc.J * TILE + col0, m);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            y1[c] = m[c].x1; y2[c] = m[c].x2; y3[c] = m[c].x3; y4[c] = m[c].x4;
            if constexpr (Q) {
                if (g == 0) sc[col0 + c] = X2{m[c].ku, m[c].km};
            }
        }
    }
    XT c1[4] = {0, 0, 0, 0}, c2[4] = {0, 0, 0, 0}, c3[4] = {0, 0, 0, 0}, c4[4] = {0, 0, 0, 0};
    __syncthreads();

    size_t off = tbase + (size_t)u0 * 4 * TILE;
    V4<ST> k{};
    if constexpr (!RING && KSRC == KSRC_PLANE) k = ld4nt(lane_ptr(Kp + off, lo));
    for (int b = bb0; b < bb1; ++b) {
        if constexpr (KSRC == KSRC_RECOMPUTE) {
            gram_band<GK>(a.F, a.kp, tc.I, tc.J, 32 * b, 64 * w, kband[w]);
            wave_lds_sync();
        }
        // (not unrolled: four steps with static ring slots take 137 instead of 97 VGPRs
        // and 154 instead of 147 us at N = 20,000)
#pragma unroll 1
        for (int s2 = 0; s2 < 8; ++s2) {
            const int r = 32 * b + 4 * s2 + g;
            const int u = b * 8 + s2;                 // row step
            const size_t off2 = (u + 1 < u1) ? off + 4 * TILE : off;
            V4<ST> k2;
            if constexpr (RING) {
                if (u + KR <= u1) wait_vm<KR - 1>();
                else wait_vm<0>();
                const float4 kk = *reinterpret_cast<const float4*>(&kring[u % KR][w][4 * l]);
                k = V4<ST>{{(ST)kk.x, (ST)kk.y, (ST)kk.z, (ST)kk.w}};
            } else if constexpr (KSRC == KSRC_PLANE) {
                k2 = ld4nt(lane_ptr(Kp + off2, lo));
            } else {
                const float4 kk = *reinterpret_cast<const float4*>(&kband[w][(4 * s2 + g) * 64 + 4 * q]);
                k = V4<ST>{{(ST)kk.x, (ST)kk.y, (ST)kk.z, (ST)kk.w}};
            }
            const X4 x = sx[r];
            XT m1 = 0, m2 = 0, m3 = 0, m4 = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const XT av = (XT)k.v[c], a2 = av * av;
                c1[c] = fma(av, x[0], c1[c]);
                m1 = fma(av, y1[c], m1);
                c2[c] = fma(a2, x[1], c2[c]);
                m2 = fma(a2, y2[c], m2);
                if constexpr (Q) {
                    const XT a3 = a2 * av, a4 = a2 * a2;
                    c3[c] = fma(a3, x[2], c3[c]);
                    m3 = fma(a3, y3[c], m3);
                    c4[c] = fma(a4, x[3], c4[c]);
                    m4 = fma(a4, y4[c], m4);
                }
            }
            XT rp, re;
            const X2 f = Q ? sk[r] : X2{0, 0};
            mom_sums<XT, Q>(m1, m2, m3, m4, f[0], f[1], rp, re);
            // row sums over the 16 column lanes through LDS every two row
            // steps (as in sweep_tile)
            red[w][0][s2 & 1][l] = (RT)rp;
            red[w][1][s2 & 1][l] = (RT)re;
            if (s2 & 1) {
                wave_lds_sync();
                const int qty = l >> 5, idx = l & 31, stp = idx >> 4, gg = (idx >> 2) & 3, pt = idx & 3;
                const RT* src = &red[w][qty][stp][16 * gg + 4 * pt];
                RT v = (src[0] + src[1]) + (src[2] + src[3]);
                v = v + dpp<0xB1>(v);
                v = v + dpp<0x4E>(v);
                const int row = 32 * b + 4 * ((s2 & 6) + stp) + gg;
                if (pt == 0) {
                    if (qty == 0) rP[w][row] = v;
                    else rE[w][row] = v;
                }
                wave_lds_sync();
            }
            if constexpr (RING) {
                if (u + KR < u1)
                    dma16(reinterpret_cast<const float*>(Kp) + tbase + (size_t)(u + KR) * 4 * TILE, lo * 4u,
                          lds_offset(&kring[u % KR][w][0]));
            } else if constexpr (KSRC == KSRC_PLANE) {
                k = k2;
            }
            off = off2;
        }
        if constexpr (KSRC == KSRC_RECOMPUTE) wave_lds_sync();
    }
    AT cP[4], cE[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const X2 f = Q ? sc[col0 + c] : X2{0, 0};
        mom_sums<AT, Q>((AT)c1[c], (AT)c2[c], (AT)c3[c], (AT)c4[c], (AT)f[0], (AT)f[1], cP[c], cE[c]);
        cP[c] = sum_groups(cP[c]);
        cE[c] = sum_groups(cE[c]);
    }
    __syncthreads();
    const AT rowP = ((AT)rP[0][tid] + (AT)rP[1][tid]) + ((AT)rP[2][tid] + (AT)rP[3][tid]);
    const AT rowE = ((AT)rE[0][tid] + (AT)rE[1][tid]) + ((AT)rE[2][tid] + (AT)rE[3][tid]);
    put_tile_sums<AT>(a, tc, rowP, rowE, cP, cE, out, split, sub);
}

// One synchronous sweep over all tiles.  Template parameters:
//   ST storage type of K' and the message planes, MT type of the top-level
//   update (cavity denominators, reciprocals), AT aggregate type;
//   KSRC: K' from the materialised plane or recomputed per 32-row band;
//   GK: Gram kind of the recompute;
//   D: 0 = stored edge state (pair-record planes read and written);
//      D >= 1 = stateless: the messages of the previous sweep are rebuilt
//      from the aggregates of the D - 1 earlier sweeps held in the ring (a
//      slot from before sweep 0 holds P~ = inf, S = 0 and yields exactly zero
//      messages), lower levels in LT (see below);
//   FIRST: the stored planes are all zero (sweep 1) and are not read;
//   XL, WR (stored state): the planes hold the messages of XL sweeps before
//      the previous one, and the XL sweeps between are formed again from the
//      aggregates of their time (ring slots slot_top - XL .. slot_top - 1),
//      each message rounded to ST as it was when stored elsewhere, so that the
//      result is the same to the bit; WR: this sweep's messages are written.
//      Writing every kStoredPeriod-th sweep only takes 20 + 16 / period bytes
//      per FP32 pair instead of 36.
// Work of one tile: its row and column sums go to the tile's partial slots,
// or, with `out`, to the caller (a chunk adds them up first).  split > 1: only
// the sub-th of `split` equal row parts of the tile.  SER (stateless
// only; 0 = exact reciprocals): the
// reciprocals of the cavity precisions Q = P~ (1 - e), e = P_reverse / P~,
// are formed from the per-node u = 1/P~ by the series
// 1/Q = (1 + e + e^2 + ...) u, one term at the lower levels and SER terms at
// the top (SER = 3: one term at the top, none at the lower levels).
// |e| <= rho^2 holds for every message by the a-priori contraction bound (no
// run-time check is needed); the host picks the series only when the
// neglected terms are below the arithmetic's precision.  KSER: SER, with
// kSerLevels where powers of K' would leave the range (series_kernels).  The
// lower levels carry G = P / (-a^2) and F = E / a, which the one-term series
// turns into G_ij = u_i - a^2 u_i^2 G_ji and F_ij = G_ij (a F_ji - S_i): the
// deepest level (reverse messages zero) is G = u, F = -S/P~ of its source and
// costs nothing, a middle level costs four operations per direction (two with
// G = u).
template <class ST, class MT, class AT, int KSRC, int GK, int D, bool FIRST, int KSER, int XL = 0, bool WR = true>
__device__ inline void sweep_tile(const SweepArgs& a, int64_t tile, int slot_top, TileSums<AT>* out = nullptr,
                                  int split = 1, int sub = 0) {
    constexpr int SER = KSER & ~kSerLevels;
    if constexpr (mom_plan<D, KSER>()) {
        sweep_tile_mom<ST, MT, AT, KSRC, GK, D, SER>(a, tile, slot_top, out, split, sub);
        return;
    } else {
    DevStatus* st = a.st;
    // lower levels: FP32 storage precision; with the series and up to three
    // levels they run in the top level's type (FP64 FMA issues at the FP32
    // rate on CDNA4, and no conversions are needed between levels; deeper
    // unrolls keep FP32 to bound the per-column register history)
    using XT = typename MsgT<ST, MT, AT, SER>::T;
    constexpr bool XF = MsgT<ST, MT, AT, SER>::F32;
    using LT = typename std::conditional<(SER && D <= 3) || std::is_same<ST, double>::value, XT, float>::type;
    constexpr bool STORED = (D == 0);
    constexpr bool LEAN = (SER == 3);         // lower levels: G = u (no series term)
    constexpr int DL = (D > 1) ? D - 1 : 1;   // lower levels held per node
    constexpr int NL = STORED ? 1 : DL;
    constexpr int NT = STORED ? 1 : TILE;
    // series: S and u^2 only at the middle levels 1 .. D - 2, S/P~ only at
    // the deepest level D - 1; exact reciprocals: S at every lower level
    constexpr int NSL = SER ? ((D > 2) ? D - 2 : 1) : NL;
    constexpr int NTS = (SER && D <= 2) ? 1 : NT;
    constexpr int NTQ = (SER && SER != 3 && D > 2) ? NT : 1;
    constexpr int NTD = (SER && D >= 2) ? NT : 1;
    const uint32_t ij = a.tiles[tile];
    const TileCoord tc{(int)(ij >> 16), (int)(ij & 0xFFFFu)};
    const size_t tbase = (size_t)tile * TT;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, g = l >> 4, q = l & 15;
    const int col0 = w * 64 + q * 4;
    constexpr int L = D;                      // stateless: levels unrolled in this launch
    const AT* HP = static_cast<const AT*>(a.HP);
    const AT* HS = static_cast<const AT*>(a.HS);
    // series: 1/P~ and S/P~ from the rings when the finalize formed them
    // (the same IEEE quotients as here)
    const AT* HI = static_cast<const AT*>(a.HI);
    const AT* HM = static_cast<const AT*>(a.HM);
    // branch-free around the loads (the ring pointers are uniform), so that
    // the node loads of the tile's prologue issue back to back
    const AT* HIs = HI ? HI : HP;
    const AT* HMs = HM ? HM : HS;
    auto inv_at = [&](int64_t o) -> AT {
        const AT v = HIs[o];
        return HI ? v : (AT)1 / v;
    };
    auto mean_at = [&](int64_t o) -> AT {
        const AT v = HMs[o], p = HP[o];
        return HM ? v : v / p;
    };
    const ST* Kp = static_cast<const ST*>(a.Kp);
    ST* Pf = static_cast<ST*>(a.Pf);
    ST* Pb = static_cast<ST*>(a.Pb);
    ST* Ef = static_cast<ST*>(a.Ef);
    ST* Eb = static_cast<ST*>(a.Eb);
    // the lane's offset inside a row group of a tile
    const uint32_t lo = (uint32_t)(g * TILE + col0);

    // stateless over an FP32 K' plane: row steps stream through a per-wave
    // LDS ring KR steps ahead (K' is the only stream; one register prefetch
    // per lane does not cover the HBM latency), the first KR issued before
    // the node data is loaded; other forms prefetch one row step ahead in
    // registers
    constexpr bool RING = (KSRC == KSRC_PLANE) && !STORED && std::is_same<ST, float>::value;
    constexpr int KR = RING ? KRING : 1;
    constexpr int SU = (RING && 8 % KR == 0) ? KR : 1;   // row steps unrolled (static ring slots)
    // this part's 32-row bands [bb0, bb1), its first row step and the end
    const int bb0 = sub * (TILE / 32 / split), bb1 = bb0 + TILE / 32 / split;
    const int u0 = 8 * bb0, u1 = 8 * bb1;
    __shared__ __attribute__((aligned(16))) float kring[KR][4][RING ? 256 : 4];
    if constexpr (RING) {
#pragma unroll
        for (int u = 0; u < KR; ++u)
            dma16(reinterpret_cast<const float*>(Kp) + tbase + (size_t)(u0 + u) * 4 * TILE, lo * 4u,
                  lds_offset(&kring[u][w][0]));
    }

    // row-node data: top level (P~ or, with SER, 1/P~) and lower levels
    __shared__ XT sPt[TILE], sS[TILE];
    __shared__ LT sPtL[NL][NT], sSL[NSL][NTS], sUQL[NSL][NTQ], sSIL[NTD];
    // row partials per wave strip (XF: FP32 sums of 64 messages; exact in AT)
    using RT = typename std::conditional<XF, XT, AT>::type;
    __shared__ RT rP[4][TILE], rE[4][TILE];
    __shared__ float kband[KSRC == KSRC_RECOMPUTE ? 4 : 1][KSRC == KSRC_RECOMPUTE ? 32 * 64 : 1];
    // stateless: per-lane row partials of two row steps, reduced over the 16
    // column lanes through LDS once per two steps (a DPP tree per row step
    // costs 24 VALU slots in FP64; this costs about 5); XF reduces in FP32
    __shared__ RT red[STORED ? 1 : 4][2][2][64];

    const int64_t top = (int64_t)slot_top * a.NPAD;
    {
        const int64_t o = top + (int64_t)tc.I * TILE + tid;
        sPt[tid] = SER ? (XT)inv_at(o) : (XT)HP[o];
        sS[tid] = (XT)HS[o];
    }
    // one-term series: the top level forms 1/Q = u - a^2 u^2 G_rev from u and
    // u^2 (two operations per direction instead of three)
    constexpr bool SQ1 = (SER == 1 || SER == 3);
    __shared__ XT sPq[SQ1 ? TILE : 1];
    XT ptj[4], sj[4], pqj[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int64_t o = top + (int64_t)tc.J * TILE + col0 + c;
        ptj[c] = SER ? (XT)inv_at(o) : (XT)HP[o];
        sj[c] = (XT)HS[o];
        pqj[c] = ptj[c] * ptj[c];
    }
    if constexpr (SQ1) sPq[tid] = sPt[tid] * sPt[tid];
    // stored state, sweeps between: aggregates of their time per row and column
    constexpr int XN = XL > 0 ? XL : 1, XR = XL > 0 ? TILE : 1;
    __shared__ __attribute__((aligned(16))) XT xrP[XN][XR], xrS[XN][XR], xcP[XN][XR], xcS[XN][XR];
    if constexpr (XL > 0) {
#pragma unroll
        for (int m = 0; m < XL; ++m) {
            const int64_t base = (int64_t)((slot_top - XL + m + a.R) % a.R) * a.NPAD;
            xrP[m][tid] = (XT)HP[base + (int64_t)tc.I * TILE + tid];
            xrS[m][tid] = (XT)HS[base + (int64_t)tc.I * TILE + tid];
            xcP[m][tid] = (XT)HP[base + (int64_t)tc.J * TILE + tid];
            xcS[m][tid] = (XT)HS[base + (int64_t)tc.J * TILE + tid];
        }
    }
    // lower levels per node: P~ (exact) or u = 1/P~ (series) at every level;
    // exact: S at every level; series: S and u^2 at the middle levels, S/P~
    // at the deepest
    LT ptjL[DL][4], sjL[NSL][4], cuqL[NSL][4], sijL[4];
    if constexpr (!STORED) {
#pragma unroll
        for (int k = 1; k < D; ++k) {
            if (k < L) {
                const int64_t base = (int64_t)((slot_top - k + a.R) % a.R) * a.NPAD;
                const int64_t o = base + (int64_t)tc.I * TILE + tid;
                if constexpr (SER) {
                    // form 3: the deepest level's G (= u) is never read
                    if (!(LEAN && k == D - 1)) sPtL[k - 1][tid] = (LT)inv_at(o);
                    if (k == D - 1) {
                        sSIL[tid] = (LT)mean_at(o);
                    } else {
                        if constexpr (!LEAN) {
                            const AT u = inv_at(o);
                            sUQL[k - 1][tid] = (LT)(u * u);
                        }
                        sSL[k - 1][tid] = (LT)HS[o];
                    }
                } else {
                    sPtL[k - 1][tid] = (LT)HP[o];
                    sSL[k - 1][tid] = (LT)HS[o];
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int64_t o = base + (int64_t)tc.J * TILE + col0 + c;
                    if constexpr (SER) {
                        const AT u = inv_at(o);
                        if (!(LEAN && k == D - 1)) ptjL[k - 1][c] = (LT)u;
                        if (k == D - 1) {
                            sijL[c] = (LT)mean_at(o);
                        } else {
                            if constexpr (!LEAN) cuqL[k - 1][c] = (LT)(u * u);
                            sjL[k - 1][c] = (LT)HS[o];
                        }
                    } else {
                        ptjL[k - 1][c] = (LT)HP[o];
                        sjL[k - 1][c] = (LT)HS[o];
                    }
                }
            }
        }
    }
    AT cP[4] = {0, 0, 0, 0}, cE[4] = {0, 0, 0, 0};
    XT cPm[4] = {0, 0, 0, 0}, cEm[4] = {0, 0, 0, 0};   // XF: FP32 column sums over the tile's 256 rows
    bool bad = false;
    __syncthreads();

    // row offset (wave-uniform: tile base plus 4 TILE per row step)
    size_t off = tbase + (size_t)u0 * 4 * TILE;
    V4<ST> k{}, pf{}, pb{}, ef{}, eb{};
    if constexpr (!RING && KSRC == KSRC_PLANE) k = ld4nt(lane_ptr(Kp + off, lo));
    if constexpr (STORED && !FIRST) {
        pf = ld4nt(lane_ptr(Pf + off, lo)); pb = ld4nt(lane_ptr(Pb + off, lo));
        ef = ld4nt(lane_ptr(Ef + off, lo)); eb = ld4nt(lane_ptr(Eb + off, lo));
    }

    for (int b = bb0; b < bb1; ++b) {
        if constexpr (KSRC == KSRC_RECOMPUTE) {
            gram_band<GK>(a.F, a.kp, tc.I, tc.J, 32 * b, 64 * w, kband[w]);
            wave_lds_sync();
        }
#pragma unroll SU
        for (int s2 = 0; s2 < 8; ++s2) {
            const int r = 32 * b + 4 * s2 + g;
            // prefetch the lane's next row (the last row re-reads itself: the
            // offset stays inside the tile and no branch is needed)
            const bool more = (b * 8 + s2 + 1) < u1;
            const size_t off2 = more ? off + 4 * TILE : off;
            V4<ST> k2, pf2, pb2, ef2, eb2;
            const int u = b * 8 + s2;                 // row step
            if constexpr (RING) {
                // this step's slot has landed once at most KR - 1 loads are
                // in flight (every later step issued one), or all of them near
                // the tile's end
                if (u + KR <= u1) wait_vm<KR - 1>();
                else wait_vm<0>();
                const float4 kk = *reinterpret_cast<const float4*>(&kring[u % KR][w][4 * l]);
                k = V4<ST>{{(ST)kk.x, (ST)kk.y, (ST)kk.z, (ST)kk.w}};
            } else if constexpr (KSRC == KSRC_PLANE) {
                k2 = ld4nt(lane_ptr(Kp + off2, lo));
            }
            if constexpr (STORED && !FIRST) {
                pf2 = ld4nt(lane_ptr(Pf + off2, lo)); pb2 = ld4nt(lane_ptr(Pb + off2, lo));
                ef2 = ld4nt(lane_ptr(Ef + off2, lo)); eb2 = ld4nt(lane_ptr(Eb + off2, lo));
            }
            if constexpr (KSRC == KSRC_RECOMPUTE) {
                const float4 kk = *reinterpret_cast<const float4*>(&kband[w][(4 * s2 + g) * 64 + 4 * q]);
                k = V4<ST>{{(ST)kk.x, (ST)kk.y, (ST)kk.z, (ST)kk.w}};
            }
            const XT pti = sPt[r], si = sS[r];
            const XT pqi = SQ1 ? sPq[r] : (XT)0;
            AT rp = 0, re = 0;
            XT rpm = 0, rem = 0;                         // XF: FP32 row sums (4 columns, then 64 per wave)
            V4<ST> npf, npb, nef, neb;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const XT av = (XT)k.v[c];
                // messages of the previous sweep: stored, or rebuilt level by level
                XT opf, opb, oef, oeb;
                if constexpr (STORED) {
                    opf = (XT)pf.v[c]; opb = (XT)pb.v[c]; oef = (XT)ef.v[c]; oeb = (XT)eb.v[c];
                    if constexpr (XL > 0) {
                        const XT a2 = av * av;
#pragma unroll
                        for (int m = 0; m < XL; ++m) {
                            // (a product fused into the next difference would
                            // skip the rounding that storing it brought)
#pragma clang fp contract(off)
                            const XT rf = rcp_fast(xrP[m][r] - opb), rb = rcp_fast(xcP[m][col0 + c] - opf);
                            const XT nef = (XT)(ST)(-av * (xrS[m][r] - oeb) * rf);
                            const XT neb = (XT)(ST)(-av * (xcS[m][col0 + c] - oef) * rb);
                            opf = (XT)(ST)(-a2 * rf);
                            opb = (XT)(ST)(-a2 * rb);
                            oef = nef;
                            oeb = neb;
                        }
                    }
                } else if constexpr (SER) {
                    // G = P / (-a^2), F = E / a of the previous sweep's messages,
                    // rebuilt from the deepest level up (XT = LT on this path)
                    const LT al = (LT)k.v[c], a2l = al * al;
                    LT gf = 0, gb = 0, ff = 0, fb = 0;
                    constexpr int kd = L - 1;
#pragma unroll
                    for (int kk = D - 1; kk >= 1; --kk) {
                        if (kk == kd) {               // deepest level: reverse messages zero
                            if constexpr (!LEAN) {    // (form 3 never reads this level's G)
                                gf = sPtL[kk - 1][r];
                                gb = ptjL[kk - 1][c];
                            }
                            ff = -sSIL[r];
                            fb = -sijL[c];
                        } else if (kk < kd) {
                            LT ngf, ngb;
                            if constexpr (LEAN) {
                                ngf = sPtL[kk - 1][r];
                                ngb = ptjL[kk - 1][c];
                            } else {
                                ngf = fma(-a2l * sUQL[kk - 1][r], gb, sPtL[kk - 1][r]);
                                ngb = fma(-a2l * cuqL[kk - 1][c], gf, ptjL[kk - 1][c]);
                            }
                            const LT nff = ngf * fma(al, fb, -sSL[kk - 1][r]);
                            const LT nfb = ngb * fma(al, ff, -sjL[kk - 1][c]);
                            gf = ngf; gb = ngb; ff = nff; fb = nfb;
                        }
                    }
                    opf = (XT)gf; opb = (XT)gb; oef = (XT)ff; oeb = (XT)fb;
                } else {
                    const LT al = (LT)k.v[c], a2l = al * al;
                    LT lpf = 0, lpb = 0, lef = 0, leb = 0;
#pragma unroll
                    for (int kk = D - 1; kk >= 1; --kk) {
                        if (kk < L) {
                            const LT qf = sPtL[kk - 1][r] - lpb, qb = ptjL[kk - 1][c] - lpf;
                            bad |= !(qf > (LT)0) | !(qb > (LT)0);
                            const LT rf = rcp_fast(qf), rb = rcp_fast(qb);
                            const LT npf_ = -a2l * rf, npb_ = -a2l * rb;
                            const LT nef_ = -al * (sSL[kk - 1][r] - leb) * rf;
                            const LT neb_ = -al * (sjL[kk - 1][c] - lef) * rb;
                            lpf = npf_; lpb = npb_; lef = nef_; leb = neb_;
                        }
                    }
                    opf = (XT)lpf; opb = (XT)lpb; oef = (XT)lef; oeb = (XT)leb;
                }
                XT pij_m, eij_m, pji_m, eji_m;
                if constexpr (SER) {
                    // opf, opb, oef, oeb hold G_ij, G_ji, F_ij, F_ji here
                    const XT a2 = av * av;
                    XT gt_f, gt_b;                                                  // (1 + e + ...) / P~
                    if constexpr (SER == 2) {
                        const XT e_f = -(a2 * opb) * pti, e_b = -(a2 * opf) * ptj[c];   // P_ji / P~_i, P_ij / P~_j
                        gt_f = fma(pti, fma(e_f, e_f, e_f), pti);
                        gt_b = fma(ptj[c], fma(e_b, e_b, e_b), ptj[c]);
                    } else {
                        gt_f = fma(-(a2 * pqi), opb, pti);                          // u (1 + e), e = -a^2 u G_rev
                        gt_b = fma(-(a2 * pqj[c]), opf, ptj[c]);
                    }
                    pij_m = -a2 * gt_f;
                    pji_m = -a2 * gt_b;
                    eij_m = (av * gt_f) * fma(av, oeb, -si);      // a G (E_ji - S_i)
                    eji_m = (av * gt_b) * fma(av, oef, -sj[c]);
                } else {
                    const XT a2 = av * av;
                    const XT qf = pti - opb;        // P~_i - P_ji
                    const XT qb = ptj[c] - opf;     // P~_j - P_ij
                    bad |= !(qf > (XT)0) | !(qb > (XT)0);
                    const XT rf = rcp_fast(qf), rb = rcp_fast(qb);
                    pij_m = -a2 * rf;
                    eij_m = -av * (si - oeb) * rf;
                    pji_m = -a2 * rb;
                    eji_m = -av * (sj[c] - oef) * rb;
                }
                if constexpr (STORED) {
                    // the aggregates add the values as stored (also where this
                    // sweep's are not: no product fused into the sum)
#pragma clang fp contract(off)
                    const ST pij = (ST)pij_m, eij = (ST)eij_m, pji = (ST)pji_m, eji = (ST)eji_m;
                    if constexpr (WR) { npf.v[c] = pij; nef.v[c] = eij; npb.v[c] = pji; neb.v[c] = eji; }
                    cP[c] += (AT)pij; cE[c] += (AT)eij;     // received by column node j
                    rp += (AT)pji; re += (AT)eji;            // received by row node i
                } else if constexpr (XF) {
                    cPm[c] += pij_m; cEm[c] += eij_m;
                    rpm += pji_m; rem += eji_m;
                } else {
                    cP[c] += (AT)pij_m; cE[c] += (AT)eij_m;
                    rp += (AT)pji_m; re += (AT)eji_m;
                }
            }
            if constexpr (STORED) {
                if constexpr (WR) {
                    st4nt(lane_ptr(Pf + off, lo), npf); st4nt(lane_ptr(Pb + off, lo), npb);
                    st4nt(lane_ptr(Ef + off, lo), nef); st4nt(lane_ptr(Eb + off, lo), neb);
                }
                rp = sum16(rp);
                re = sum16(re);
                if (q == 0) { rP[w][r] = rp; rE[w][r] = re; }
            } else {
                red[w][0][s2 & 1][l] = XF ? (RT)rpm : (RT)rp;
                red[w][1][s2 & 1][l] = XF ? (RT)rem : (RT)re;
                if (s2 & 1) {
                    // lane l sums quantity l / 32 of row step (l % 32) / 16 and
                    // row group ((l % 32) / 4) % 4 over the column lanes
                    // 4 (l % 4) .. +3; the quad then adds its four parts (the
                    // same sum in every lane: IEEE addition commutes)
                    wave_lds_sync();
                    const int qty = l >> 5, idx = l & 31, stp = idx >> 4, gg = (idx >> 2) & 3, pt = idx & 3;
                    const RT* src = &red[w][qty][stp][16 * gg + 4 * pt];
                    RT v = (src[0] + src[1]) + (src[2] + src[3]);
                    v = v + dpp<0xB1>(v);
                    v = v + dpp<0x4E>(v);
                    const int row = 32 * b + 4 * ((s2 & 6) + stp) + gg;
                    if (pt == 0) {
                        if (qty == 0) rP[w][row] = v;
                        else rE[w][row] = v;
                    }
                    wave_lds_sync();
                }
            }
            if constexpr (RING) {
                // the slot's next row step (k was read from it and used above)
                if (u + KR < u1)
                    dma16(reinterpret_cast<const float*>(Kp) + tbase + (size_t)(u + KR) * 4 * TILE, lo * 4u,
                          lds_offset(&kring[u % KR][w][0]));
            } else if constexpr (KSRC == KSRC_PLANE) {
                k = k2;
            }
            if constexpr (STORED && !FIRST) { pf = pf2; pb = pb2; ef = ef2; eb = eb2; }
            off = off2;
        }
        if constexpr (KSRC == KSRC_RECOMPUTE) wave_lds_sync();
    }
    if constexpr (XF) {
#pragma unroll
        for (int c = 0; c < 4; ++c) { cP[c] = (AT)cPm[c]; cE[c] = (AT)cEm[c]; }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) { cP[c] = sum_groups(cP[c]); cE[c] = sum_groups(cE[c]); }
    __syncthreads();
    if (__any(bad) && l == 0) st->bad = 1;
    const AT rowP = ((AT)rP[0][tid] + (AT)rP[1][tid]) + ((AT)rP[2][tid] + (AT)rP[3][tid]);
    const AT rowE = ((AT)rE[0][tid] + (AT)rE[1][tid]) + ((AT)rE[2][tid] + (AT)rE[3][tid]);
    put_tile_sums<AT>(a, tc, rowP, rowE, cP, cE, out, split, sub);
    }
}

template <class ST, class MT, class AT, int KSRC, int GK, int D, bool FIRST, int SER>
__global__ __launch_bounds__(WG) void k_sweep(SweepArgs a) {
    if (a.st->done) return;
    sweep_tile<ST, MT, AT, KSRC, GK, D, FIRST, SER>(a, blockIdx.x / a.split, a.slot_top, nullptr, a.split,
                                                    blockIdx.x % a.split);
}

// stored records over the plane, written every kStoredPeriod sweeps
template <class ST, class MT, class AT, int KSRC, int GK, bool FIRST, int XL, bool WR>
__global__ __launch_bounds__(WG) void k_sweep_st(SweepArgs a) {
    if (a.st->done) return;
    sweep_tile<ST, MT, AT, KSRC, GK, 0, FIRST, 0, XL, WR>(a, blockIdx.x / a.split, a.slot_top, nullptr, a.split,
                                                    blockIdx.x % a.split);
}

// The sweeps chunk_plan selects (a.chunk = 2, single solves and served
// alike) run over 2 x 2 chunks of tiles; every other sweep takes one tile per
// workgroup.
template <class ST, class MT, class AT, int KSRC, int D, int SER>
constexpr bool chunk_sweep_ok() {
    return KSRC == KSRC_PLANE && std::is_same<ST, float>::value &&
           chunk_plan(std::is_same<AT, float>::value || MsgT<ST, MT, AT, SER>::F32, D, SER & ~kSerLevels);
}

// Synchronous sweep over chunks of C x C tiles (a.chunks: Ic << 16 | Jc,
// Ic <= Jc; the diagonal chunk holds its tiles with I <= J).  One workgroup
// per chunk adds each row's sums over the chunk's columns and each column's
// over its rows before storing them: a chunk stores one partial vector per
// row block and per column block, where single tiles store two per tile
// (C = 2 halves the partial-sum bytes, which reach HBM in small write bursts
// between the K' stream's reads).  The slots of block K (Kc = K / C, NBc =
// ceil(NB / C)) are those of the single-tile scheme with chunks in place of
// blocks: s < Kc the column sums of chunk (s, Kc), s = Kc the row sums of the
// diagonal chunk, Kc < s < NBc the row sums of chunk (Kc, s), s = NBc the
// column sums of the diagonal chunk.  Sums over a chunk are kept in CT: FP32
// where the partials are stored in FP32.
template <class ST, class MT, class AT, int GK, int D, int SER, int C>
__device__ inline void sweep_chunk(const SweepArgs& a, int Ic, int Jc, int slot_top) {
    using CT = typename std::conditional<MsgT<ST, MT, AT, SER>::F32, float, AT>::type;
    const int NB = a.NB, NBc = (NB + C - 1) / C;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, g = l >> 4, q = l & 15;
    const int col0 = w * 64 + q * 4;
    const bool p32 = a.part32 != 0;
    // row sums per row block of the chunk, in LDS (each thread its own row);
    // the column sums stay in registers
    __shared__ CT rs[C][2][TILE];
#pragma unroll
    for (int ii = 0; ii < C; ++ii) { rs[ii][0][tid] = 0; rs[ii][1][tid] = 0; }
    bool first = true;
    // one copy of the tile code (loops not unrolled)
#pragma unroll 1
    for (int jj = 0; jj < C; ++jj) {
        const int J = Jc * C + jj;
        if (J >= NB) break;
        CT csP[4] = {0, 0, 0, 0}, csE[4] = {0, 0, 0, 0};
#pragma unroll 1
        for (int ii = 0; ii < C; ++ii) {
            const int I = Ic * C + ii;
            if (I > J) break;          // (I >= NB implies I > J)
            if (!first) __syncthreads();
            first = false;
            TileSums<AT> o;
            sweep_tile<ST, MT, AT, KSRC_PLANE, GK, D, false, SER>(a, tile_index(I, J, NB), slot_top, &o);
            rs[ii][0][tid] += (CT)o.rp;
            rs[ii][1][tid] += (CT)o.re;
#pragma unroll
            for (int c = 0; c < 4; ++c) { csP[c] += (CT)o.cp[c]; csE[c] += (CT)o.ce[c]; }
        }
        if (g == 0) {
            const int slot = (Ic < Jc) ? Ic : NBc;
            const size_t cb = ((size_t)J * (NBc + 1) + slot) * TILE + col0;
#pragma unroll
            for (int c = 0; c < 4; ++c) { put_part(a.partP, cb + c, (AT)csP[c], p32); put_part(a.partE, cb + c, (AT)csE[c], p32); }
        }
    }
#pragma unroll
    for (int ii = 0; ii < C; ++ii) {
        const int I = Ic * C + ii;
        if (I >= NB) break;
        const size_t o = ((size_t)I * (NBc + 1) + Jc) * TILE + tid;
        put_part(a.partP, o, (AT)rs[ii][0][tid], p32);
        put_part(a.partE, o, (AT)rs[ii][1][tid], p32);
    }
}

template <class ST, class MT, class AT, int GK, int D, int SER, int C>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_sweep_chunk(SweepArgs a) {
    if (a.st->done) return;
    const uint32_t cc = a.chunks[blockIdx.x];
    sweep_chunk<ST, MT, AT, GK, D, SER, C>(a, (int)(cc >> 16), (int)(cc & 0xFFFFu), a.slot_top);
}

// Stateless sweep with K' recomputed per band: the Gram fragments, the
// band's K' (LDS) and the recursion's per-column state share the registers;
// at least three waves per SIMD keep the band computations of some waves
// overlapping the message steps of others.
template <class ST, class MT, class AT, int GK, int D, int SER>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_sweep_rc(SweepArgs a) {
    if (a.st->done) return;
    sweep_tile<ST, MT, AT, KSRC_RECOMPUTE, GK, D, false, SER>(a, blockIdx.x / a.split, a.slot_top, nullptr, a.split,
                                                              blockIdx.x % a.split);
}

// Sums of v[r] over the 32 lanes of a half, row r in the lanes whose low four
// bits are r's in reverse; each step halves the rows a lane holds, so all 16
// take 16 additions instead of 80.
__device__ inline double sum_rows16(const float (&v)[16], int l) {
    double s[8];
    const bool b0 = l & 1, b1 = l & 2, b2 = l & 4, b3 = l & 8;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float keep = b0 ? v[k + 8] : v[k], give = b0 ? v[k] : v[k + 8];
        s[k] = (double)keep + (double)__shfl_xor(give, 1);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double keep = b1 ? s[k + 4] : s[k], give = b1 ? s[k] : s[k + 4];
        s[k] = keep + __shfl_xor(give, 2);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double keep = b2 ? s[k + 2] : s[k], give = b2 ? s[k] : s[k + 2];
        s[k] = keep + __shfl_xor(give, 4);
    }
    const double keep = b3 ? s[1] : s[0], give = b3 ? s[0] : s[1];
    s[0] = keep + __shfl_xor(give, 8);
    return s[0] + __shfl_xor(s[0], 16);
}

// Three-level series sweep (form 3, FP32 messages) with K' recomputed from
// augmented rows of MP features, in the MFMA's own layout: a wave forms 32 x 32
// blocks of its 32-row band against the tile's eight column blocks (B
// fragments staged once per workgroup, as in k_gram_sums), a lane holding 16
// rows of one column.  Each K' entry goes from the MFMA output through exp2
// straight into the moment sums (mom_plan): the rows' factors and sums stay in
// registers over the band, a column's over the block.  No K' band passes
// through LDS, and nothing is reduced across lanes but one vector per band.
// 16 VALU slots per pair (exp2 4, + lambda^2, a^2, a^3, a^4, eight FMAs) beside the
// MFMAs; the VALU is busy for three quarters of the time.  N = 120,000, m =
// 20: 8.0 (bands through LDS, level by level) -> 5.5 ms per sweep; N = 300,000:
// 50.4 -> 34.3 ms (5.0 and 31.3 without the fourth power).  231 VGPRs of the
// three-term split at 32 features and 252 at 64 leave two waves per SIMD.
template <int KIND, int MP>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_sweep_rc_mom(SweepArgs a) {
    if (a.st->done) return;
    using MM = Mom<float, 3>;
    using BS = BStage<KIND>;
    typedef float X4 __attribute__((ext_vector_type(4)));
    typedef float X2 __attribute__((ext_vector_type(2)));
    constexpr int CH = BS::NP * (MP / 16) * 64, PR = (CH + WG - 1) / WG, NS = MP / 16;
    __shared__ bf16x8 sb[2][CH];
    __shared__ __attribute__((aligned(16))) float sx[4][TILE];   // x_1 .. x_4 of the row nodes
    __shared__ X4 sy[TILE];                     // ... of the column nodes
    __shared__ X2 sk[TILE], sc[TILE];           // u', m'
    __shared__ float cs[4][4][TILE];            // column sums per wave
    const int split = a.split, sub = blockIdx.x % split;
    const uint32_t ij = a.tiles[blockIdx.x / split];
    const TileCoord tc{(int)(ij >> 16), (int)(ij & 0xFFFFu)};
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, h = l >> 5, l32 = l & 31;
    const int64_t i0 = (int64_t)tc.I * TILE, j0 = (int64_t)tc.J * TILE;
    const float lam2 = (float)a.kp.lam2;
    // this thread's 16-byte chunks of a staged block: plane, row and column of
    // the row-major planes, in the order of BStage
    const uint16_t* const bt = a.F.aug1 + j0 * MP;
    int64_t so[PR];
#pragma unroll
    for (int i = 0; i < PR; ++i) {
        const int k = tid + WG * i, pl = k / (64 * NS), rem = k % (64 * NS);
        so[i] = pl * a.F.aug_plane + rem / (2 * NS) * MP + rem % (2 * NS) * 8;
        if (k < CH) sb[0][BS::dst(NS, k)] = *reinterpret_cast<const bf16x8*>(bt + so[i]);
    }
    {
        MM m[1];
        mom_nodes<1, float, 3, double>(a, a.slot_top, i0 + tid, m);
        sx[0][tid] = m[0].x1; sx[1][tid] = m[0].x2; sx[2][tid] = m[0].x3; sx[3][tid] = m[0].x4;
        sk[tid] = X2{m[0].ku, m[0].km};
        mom_nodes<1, float, 3, double>(a, a.slot_top, j0 + tid, m);
        sy[tid] = X4{m[0].x1, m[0].x2, m[0].x3, m[0].x4};
        sc[tid] = X2{m[0].ku, m[0].km};
    }
    __syncthreads();
    const int passes = 2 / split;
    const bool p32 = a.part32 != 0;
    const PartSlots ps{a.NB, split};
    int cur = 0;
#pragma unroll 1
    for (int pass = 0; pass < passes; ++pass) {
        const int band = 4 * (sub * passes + pass) + w;
        RowFrag<KIND, MP> fa;
        {
            const uint16_t* const at = a.F.aug0 + (i0 + band * 32 + l32) * MP + 8 * h;
#pragma unroll
            for (int st = 0; st < NS; ++st) {
                fa.hi[st] = *reinterpret_cast<const bf16x8*>(at + 16 * st);
                if constexpr (BS::NP >= 2) fa.lo[st] = *reinterpret_cast<const bf16x8*>(at + a.F.aug_plane + 16 * st);
                if constexpr (BS::NP >= 3)
                    fa.lo2[st] = *reinterpret_cast<const bf16x8*>(at + 2 * a.F.aug_plane + 16 * st);
            }
        }
        float r1[16], r2[16], r3[16], r4[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) r1[r] = r2[r] = r3[r] = r4[r] = 0.0f;
#pragma unroll 1
        for (int cb = 0; cb < TILE / 32; ++cb) {
            // the next block (the first again after the last of a pass)
            const bool more = !(pass == passes - 1 && cb == TILE / 32 - 1);
            const int nb0 = ((cb + 1) % (TILE / 32)) * 32 * MP;
            bf16x8 pre[PR];
            if (more) {
#pragma unroll
                for (int i = 0; i < PR; ++i) {
                    const int k = tid + WG * i;
                    if (k < CH) pre[i] = *reinterpret_cast<const bf16x8*>(bt + so[i] + nb0);
                }
            }
            f32x16 acc = {};
            BS::template mma<MP>(fa, sb[cur], NS, l, acc);
            const int col = cb * 32 + l32;
            const X4 y = sy[col];
            // the index test matters only on diagonal tiles and past N
            if (!((tc.I < tc.J) && (j0 + cb * 32 + 32 <= a.kp.N))) {
                const int64_t j = j0 + col;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t i = i0 + band * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
                    const float kv = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(acc[r]), 0.0f, 1.0f) + lam2;
                    acc[r] = (i < j && j < a.kp.N) ? kv : 0.0f;
                }
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc[r] = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(acc[r]), 0.0f, 1.0f) + lam2;
            }
            float c1 = 0.0f, c2 = 0.0f, c3 = 0.0f, c4 = 0.0f;
            // four consecutive rows at a time (one 16-byte LDS read per factor)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int o = band * 32 + 8 * t + 4 * h;
                const X4 x1 = *reinterpret_cast<const X4*>(&sx[0][o]), x2 = *reinterpret_cast<const X4*>(&sx[1][o]),
                         x3 = *reinterpret_cast<const X4*>(&sx[2][o]), x4 = *reinterpret_cast<const X4*>(&sx[3][o]);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 4 * t + v;
                    const float av = acc[r], a2 = av * av, a3 = a2 * av, a4 = a2 * a2;
                    c1 = fmaf(av, x1[v], c1);
                    r1[r] = fmaf(av, y[0], r1[r]);
                    c2 = fmaf(a2, x2[v], c2);
                    r2[r] = fmaf(a2, y[1], r2[r]);
                    c3 = fmaf(a3, x3[v], c3);
                    r3[r] = fmaf(a3, y[2], r3[r]);
                    c4 = fmaf(a4, x4[v], c4);
                    r4[r] = fmaf(a4, y[3], r4[r]);
                }
            }
            // (the row sums are formed here: the compiler otherwise carries the
            // powers of a over into the next block, 64 registers)
#pragma unroll
            for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(r1[r]), "+v"(r2[r]), "+v"(r3[r]), "+v"(r4[r]));
            // the column's 32 rows of this band: both lane halves
            c1 = c1 + __shfl_xor(c1, 32);
            c2 = c2 + __shfl_xor(c2, 32);
            c3 = c3 + __shfl_xor(c3, 32);
            c4 = c4 + __shfl_xor(c4, 32);
            if (h == 0) {
                if (pass > 0) { c1 += cs[w][0][col]; c2 += cs[w][1][col]; c3 += cs[w][2][col]; c4 += cs[w][3][col]; }
                cs[w][0][col] = c1; cs[w][1][col] = c2; cs[w][2][col] = c3; cs[w][3][col] = c4;
            }
            if (more) {
#pragma unroll
                for (int i = 0; i < PR; ++i) {
                    const int k = tid + WG * i;
                    if (k < CH) sb[cur ^ 1][BS::dst(NS, k)] = pre[i];
                }
            }
            __syncthreads();
            cur ^= 1;
        }
        // the band's row sums over the 32 lanes of a half, in FP64 (a lane's
        // eight columns are FP32 sums): step by step a lane keeps half of the
        // rows it holds and adds its partner's sums of them, so that lane l of
        // a half ends with row 8 (l & 1) + 4 (l >> 1 & 1) + 2 (l >> 2 & 1) + (l >> 3 & 1)
        float fp[16], fe[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const X2 f = sk[band * 32 + 8 * (r >> 2) + 4 * h + (r & 3)];
            mom_sums<float, true>(r1[r], r2[r], r3[r], r4[r], f[0], f[1], fp[r], fe[r]);
        }
        const double vp = sum_rows16(fp, l), ve = sum_rows16(fe, l);
        if (l32 < 16) {
            const int r = 8 * (l & 1) + 2 * (l & 2) + (l >> 1 & 2) + (l >> 3 & 1);
            const size_t o = ps.row(tc.I, tc.J) + band * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
            put_part(a.partP, o, vp, p32);
            put_part(a.partE, o, ve, p32);
        }
    }
    double m[4], p, e;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        m[k] = ((double)cs[0][k][tid] + (double)cs[1][k][tid]) + ((double)cs[2][k][tid] + (double)cs[3][k][tid]);
    const X2 f = sc[tid];
    mom_sums<double, true>(m[0], m[1], m[2], m[3], (double)f[0], (double)f[1], p, e);
    const size_t o = ps.col(tc.I, tc.J, sub) + tid;
    put_part(a.partP, o, p, p32);
    put_part(a.partE, o, e, p32);
}

// ------------------------------------------------ grouped (Gauss-Seidel) --
//
// Grouped schedule: the block rows are split into G ordered groups and a
// sweep visits them in order; the visit of group g recomputes every message
// INTO a node of g and then refreshes g's aggregates.  One launch per visit
// walks a list of (tile, direction) entries (GE_* bits): FWD = the messages
// i -> j into the column block J, BWD = j -> i into the row block I.

// Version of the source aggregates used at chain level k (k = 0: the message
// computed now; level k + 1: the reverse message it consumes) for a visit in
// sweep t, as an offset from t.  A message computed at a visit uses its
// source's aggregates as they stand then, and the reverse message as last
// computed, at the latest earlier visit of the source's group:
//   FWD across groups (row group earlier): row t+1, col t, row t, col t-1, ...
//   BWD across groups (column group later): col t, row t, col t-1, row t-1, ...
//   inside the group (Jacobi within g): t, t-1, t-2, ... as in the
//   synchronous schedule.
__device__ inline int level_version_offset(bool fwd, bool within, int k) {
    if (within) return -k;
    return fwd ? ((k & 1) ? -((k - 1) >> 1) : 1 - (k >> 1)) : -(k >> 1);
}
// Sweep of the visit that computed the level-k message, as an offset from t
// (FWD across: t, t, t-1, t-1, ...; BWD across: t, t-1, t-1, t-2, ...;
// inside: t - k).  A level whose visit precedes sweep 0 carries the zero
// start message; across groups its source version can still be 0, so the
// ring's pre-sweep slots alone do not make it zero.
__device__ inline int level_visit_offset(bool fwd, bool within, int k) {
    if (within) return -k;
    return fwd ? -(k >> 1) : -((k + 1) >> 1);
}

// LDS of one single-direction visit, declared by the kernel so that both
// directions share it.
template <class MT, class LT, class AT, class RT, int NRL, int RECOMP, int KRN = 0>
struct DirSmem {
    static constexpr int RING_STEPS = KRN;
    // K' ring (stateless visits over an FP32 plane): KRN row steps per wave
    __attribute__((aligned(16))) float kring[KRN > 0 ? KRN : 1][4][KRN > 0 ? 256 : 4];
    MT topP[TILE], topS[TILE];            // row source at level 0 (FWD)
    LT lowP[NRL][TILE], lowS[NRL][TILE];  // row source at lower levels
    LT lowSI[NRL][TILE];                  // series: S / P~
    LT lowUQ[NRL][TILE];                  // series: (1/P~)^2
    RT rP[4][TILE], rE[4][TILE];          // BWD row partials per wave strip (exact in AT)
    RT red[4][2][2][64];                  // BWD stateless: two row steps of lane partials
    float kband[RECOMP ? 4 : 1][RECOMP ? 32 * 64 : 1];
};

template <class ST, class MT, class AT, int D, int SER>
struct DirTypes {
    using XT = typename MsgT<ST, MT, AT, SER>::T;
    static constexpr bool XF = MsgT<ST, MT, AT, SER>::F32;
    using LT = typename std::conditional<(SER && D <= 3) || std::is_same<ST, double>::value, XT, float>::type;
    using RT = typename std::conditional<XF, XT, AT>::type;    // row reduction type
    static constexpr int NRL = (D / 2 > 0) ? D / 2 : 1;   // lower row-side levels
    static constexpr int NCL = (D / 2 > 0) ? D / 2 : 1;   // lower column-side levels
};

// One direction of one tile.  D = 0: stored pair records (the reverse
// message is read from its plane, the new one written to the other);
// D >= 1: the chain of D levels is rebuilt from the aggregate ring, the
// reverse message below the deepest level taken as zero.  The source's
// aggregates at version v sit in ring slot v mod R (R = 1 for stored
// records: every read is the node's latest value).
template <class ST, class MT, class AT, int KSRC, int GK, int D, int SER, bool FWD, class SM>
__device__ inline void sweep_tile_dir(const SweepArgs& a, int64_t tile, bool within, int t, SM& sm, int sub) {
    using DT = DirTypes<ST, MT, AT, D, SER>;
    using LT = typename DT::LT;
    using XT = typename DT::XT;
    constexpr bool XF = DT::XF;
    constexpr bool STORED = (D == 0);
    constexpr int L = STORED ? 1 : D;
    DevStatus* st = a.st;
    const uint32_t ij = a.tiles[tile];
    const TileCoord tc{(int)(ij >> 16), (int)(ij & 0xFFFFu)};
    const int NB = a.NB;
    const size_t tbase = (size_t)tile * TT;
    const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, g = l >> 4, q = l & 15;
    const int col0 = w * 64 + q * 4;
    const AT* HP = static_cast<const AT*>(a.HP);
    const AT* HS = static_cast<const AT*>(a.HS);
    const AT* HI = static_cast<const AT*>(a.HI);
    const AT* HM = static_cast<const AT*>(a.HM);
    const ST* Kp = static_cast<const ST*>(a.Kp);
    const uint32_t lo = (uint32_t)(g * TILE + col0);      // lane offset inside a row group
    // stateless visits over an FP32 K' plane (single solves): row steps
    // stream through the per-wave LDS ring as in the synchronous sweep, the
    // first KR issued first.  The served form keeps the one-step register
    // prefetch: its many small launches run more workgroups per CU without
    // the ring's LDS.
    constexpr bool RING = (SM::RING_STEPS > 0) && (KSRC == KSRC_PLANE) && !STORED && std::is_same<ST, float>::value;
    constexpr int KR = RING ? SM::RING_STEPS : 1;
    constexpr int SU = (RING && 8 % KR == 0) ? KR : 1;   // row steps unrolled (static ring slots)
    // the sub-th row part of the tile: bands [bb0, bb1), row steps [u0, u1)
    const int bb0 = sub * (TILE / 32 / a.split), bb1 = bb0 + TILE / 32 / a.split;
    const int u0 = 8 * bb0, u1 = 8 * bb1;
    if constexpr (RING) {
#pragma unroll
        for (int u = 0; u < KR; ++u)
            dma16(reinterpret_cast<const float*>(Kp) + tbase + (size_t)(u0 + u) * 4 * TILE, lo * 4u,
                  lds_offset(&sm.kring[u][w][0]));
    }
    auto slot_of = [&](int k) -> int64_t {
        if constexpr (STORED) return 0;
        const int v = t + level_version_offset(FWD, within, k);
        return (int64_t)(((v % a.R) + a.R) % a.R) * a.NPAD;
    };

    // source data per level: row side in LDS (per row), column side in
    // registers (the lane's four columns)
    XT ctP[4], ctS[4];                           // column source at level 0 (BWD)
    LT clP[DT::NCL][4], clS[DT::NCL][4], clSI[SER ? DT::NCL : 1][4], clUQ[SER ? DT::NCL : 1][4];
#pragma unroll
    for (int k = 0; k < L; ++k) {
        const bool row_side = FWD ? !(k & 1) : (k & 1);
        const int64_t base = slot_of(k);
        // levels computed before sweep 0: P~ = inf, S = 0 give exactly zero messages
        const bool live = STORED || t + level_visit_offset(FWD, within, k) >= 0;
        // per node: P~ (or, series, 1/P~), S and (series) S/P~; the rings'
        // 1/P~ and S/P~ when the finalize formed them (the same quotients)
        auto node = [&](int64_t o, AT& pv, AT& sv, AT& mv) {
            AT p = HP[o], s = HS[o];
            if (!live) { p = (AT)INFINITY; s = 0; }
            sv = s;
            if constexpr (SER) {
                pv = (HI && live) ? HI[o] : (AT)1 / p;
                mv = (HM && live) ? HM[o] : s / p;
            } else {
                pv = p;
                mv = 0;
            }
        };
        if (row_side) {
            AT pv, sv, mv;
            node(base + (int64_t)tc.I * TILE + tid, pv, sv, mv);
            if (k == 0) {
                sm.topP[tid] = (XT)pv;
                sm.topS[tid] = (XT)sv;
            } else {
                const int m = FWD ? (k >> 1) - 1 : (k >> 1);
                sm.lowP[m][tid] = (LT)pv;
                sm.lowS[m][tid] = (LT)sv;
                if constexpr (SER) { sm.lowSI[m][tid] = (LT)mv; sm.lowUQ[m][tid] = (LT)(pv * pv); }
            }
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                AT pv, sv, mv;
                node(base + (int64_t)tc.J * TILE + col0 + c, pv, sv, mv);
                if (k == 0) {
                    ctP[c] = (XT)pv;
                    ctS[c] = (XT)sv;
                } else {
                    const int m = FWD ? (k >> 1) : (k >> 1) - 1;
                    clP[m][c] = (LT)pv;
                    clS[m][c] = (LT)sv;
                    if constexpr (SER) { clSI[m][c] = (LT)mv; clUQ[m][c] = (LT)(pv * pv); }
                }
            }
        }
    }
    AT cP[4] = {0, 0, 0, 0}, cE[4] = {0, 0, 0, 0};
    XT cPm[4] = {0, 0, 0, 0}, cEm[4] = {0, 0, 0, 0};   // XF: FP32 column sums over the tile's 256 rows
    bool bad = false;
    __syncthreads();

    // stored records: FWD reads the reverse plane (P_ji, E_ji) and writes
    // the forward one; BWD the other way round
    ST* Prd = static_cast<ST*>(FWD ? a.Pb : a.Pf);
    ST* Erd = static_cast<ST*>(FWD ? a.Eb : a.Ef);
    ST* Pwr = static_cast<ST*>(FWD ? a.Pf : a.Pb);
    ST* Ewr = static_cast<ST*>(FWD ? a.Ef : a.Eb);

    size_t off = tbase + (size_t)u0 * 4 * TILE;                                   // wave-uniform row offset
    V4<ST> k4{}, pr{}, er{};
    if constexpr (KSRC == KSRC_PLANE && !RING) k4 = ld4nt(lane_ptr(Kp + off, lo));
    if constexpr (STORED) { pr = ld4nt(lane_ptr(Prd + off, lo)); er = ld4nt(lane_ptr(Erd + off, lo)); }

    for (int b = bb0; b < bb1; ++b) {
        if constexpr (KSRC == KSRC_RECOMPUTE) {
            gram_band<GK>(a.F, a.kp, tc.I, tc.J, 32 * b, 64 * w, sm.kband[w]);
            wave_lds_sync();
        }
#pragma unroll SU
        for (int s2 = 0; s2 < 8; ++s2) {
            const int r = 32 * b + 4 * s2 + g;
            const bool more = (b * 8 + s2 + 1) < u1;
            const size_t off2 = more ? off + 4 * TILE : off;
            V4<ST> k2, pr2, er2;
            const int u = b * 8 + s2;                 // row step
            if constexpr (RING) {
                if (u + KR <= u1) wait_vm<KR - 1>();
                else wait_vm<0>();
                const float4 kk = *reinterpret_cast<const float4*>(&sm.kring[u % KR][w][4 * l]);
                k4 = V4<ST>{{(ST)kk.x, (ST)kk.y, (ST)kk.z, (ST)kk.w}};
            } else if constexpr (KSRC == KSRC_PLANE) {
                k2 = ld4nt(lane_ptr(Kp + off2, lo));
            }
            if constexpr (STORED) { pr2 = ld4nt(lane_ptr(Prd + off2, lo)); er2 = ld4nt(lane_ptr(Erd + off2, lo)); }
            if constexpr (KSRC == KSRC_RECOMPUTE) {
                const float4 kk = *reinterpret_cast<const float4*>(&sm.kband[w][(4 * s2 + g) * 64 + 4 * q]);
                k4 = V4<ST>{{(ST)kk.x, (ST)kk.y, (ST)kk.z, (ST)kk.w}};
            }
            AT rp = 0, re = 0;
            XT rpm = 0, rem = 0;                         // XF: FP32 row sums (4 columns, then 64 per wave)
            V4<ST> np, ne;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const XT av = (XT)k4.v[c];
                // reverse message consumed by the top level
                XT opr, oer;
                if constexpr (STORED) {
                    opr = (XT)pr.v[c]; oer = (XT)er.v[c];
                } else {
                    const LT al = (LT)k4.v[c], a2l = al * al;
                    LT lp = 0, le = 0;
#pragma unroll
                    for (int k = L - 1; k >= 1; --k) {
                        const bool row_side = FWD ? !(k & 1) : (k & 1);
                        const int mr = FWD ? (k >> 1) - 1 : (k >> 1);
                        const int mc = FWD ? (k >> 1) : (k >> 1) - 1;
                        const LT pv = row_side ? sm.lowP[mr][r] : clP[mc][c];
                        const LT sv = row_side ? sm.lowS[mr][r] : clS[mc][c];
                        if constexpr (SER) {
                            // G = P / (-a^2) and F = E / a (as in the synchronous sweep)
                            if (k == L - 1) {            // deepest: reverse message zero
                                const LT siv = row_side ? sm.lowSI[mr][r] : clSI[mc][c];
                                lp = pv;
                                le = -siv;
                            } else {
                                LT ng;
                                if constexpr (SER == 3) {       // G = u (no series term)
                                    ng = pv;
                                } else {
                                    const LT uq = row_side ? sm.lowUQ[mr][r] : clUQ[mc][c];
                                    ng = fma(-a2l * uq, lp, pv);
                                }
                                const LT nf = ng * fma(al, le, -sv);
                                lp = ng; le = nf;
                            }
                        } else {
                            const LT qv = pv - lp;
                            bad |= !(qv > (LT)0);
                            const LT rv = rcp_fast(qv);
                            const LT np_ = -a2l * rv;
                            const LT ne_ = -al * (sv - le) * rv;
                            lp = np_; le = ne_;
                        }
                    }
                    opr = (XT)lp; oer = (XT)le;
                }
                // top level: the message into the target, from the source at level 0
                const XT pt = FWD ? sm.topP[r] : ctP[c];
                const XT sv = FWD ? sm.topS[r] : ctS[c];
                XT pm, em;
                if constexpr (SER) {
                    // opr, oer hold G, F of the reverse message here
                    const XT a2 = av * av;
                    const XT e = -(a2 * opr) * pt;
                    XT gt;
                    if constexpr (SER == 2) gt = fma(pt, fma(e, e, e), pt);
                    else gt = fma(pt, e, pt);
                    pm = -a2 * gt;
                    em = (av * gt) * fma(av, oer, -sv);
                } else {
                    const XT qv = pt - opr;
                    bad |= !(qv > (XT)0);
                    const XT rv = rcp_fast(qv);
                    pm = -(av * av) * rv;
                    em = -av * (sv - oer) * rv;
                }
                if constexpr (STORED) {
                    const ST ps = (ST)pm, es = (ST)em;
                    np.v[c] = ps; ne.v[c] = es;
                    if constexpr (FWD) { cP[c] += (AT)ps; cE[c] += (AT)es; }
                    else { rp += (AT)ps; re += (AT)es; }
                } else if constexpr (XF) {
                    if constexpr (FWD) { cPm[c] += pm; cEm[c] += em; }
                    else { rpm += pm; rem += em; }
                } else {
                    if constexpr (FWD) { cP[c] += (AT)pm; cE[c] += (AT)em; }
                    else { rp += (AT)pm; re += (AT)em; }
                }
            }
            if constexpr (STORED) { st4nt(lane_ptr(Pwr + off, lo), np); st4nt(lane_ptr(Ewr + off, lo), ne); }
            if constexpr (!FWD && STORED) {
                rp = sum16(rp);
                re = sum16(re);
                if (q == 0) { sm.rP[w][r] = rp; sm.rE[w][r] = re; }
            } else if constexpr (!FWD) {
                // row sums over the 16 column lanes through LDS every two row
                // steps (same scheme as the synchronous stateless sweep)
                using RT = typename DT::RT;
                sm.red[w][0][s2 & 1][l] = XF ? (RT)rpm : (RT)rp;
                sm.red[w][1][s2 & 1][l] = XF ? (RT)rem : (RT)re;
                if (s2 & 1) {
                    wave_lds_sync();
                    const int qty = l >> 5, idx = l & 31, stp = idx >> 4, gg = (idx >> 2) & 3, pt = idx & 3;
                    const RT* src = &sm.red[w][qty][stp][16 * gg + 4 * pt];
                    RT v = (src[0] + src[1]) + (src[2] + src[3]);
                    v = v + dpp<0xB1>(v);
                    v = v + dpp<0x4E>(v);
                    const int row = 32 * b + 4 * ((s2 & 6) + stp) + gg;
                    if (pt == 0) {
                        if (qty == 0) sm.rP[w][row] = v;
                        else sm.rE[w][row] = v;
                    }
                    wave_lds_sync();
                }
            }
            if constexpr (RING) {
                // the slot's next row step (k4 was read from it and used above)
                if (u + KR < u1)
                    dma16(reinterpret_cast<const float*>(Kp) + tbase + (size_t)(u + KR) * 4 * TILE, lo * 4u,
                          lds_offset(&sm.kring[u % KR][w][0]));
            } else if constexpr (KSRC == KSRC_PLANE) {
                k4 = k2;
            }
            if constexpr (STORED) { pr = pr2; er = er2; }
            off = off2;
        }
        if constexpr (KSRC == KSRC_RECOMPUTE) wave_lds_sync();
    }
    const bool p32 = a.part32 != 0;
    const PartSlots ps{NB, a.split};
    if constexpr (FWD) {
        if constexpr (XF) {
#pragma unroll
            for (int c = 0; c < 4; ++c) { cP[c] = (AT)cPm[c]; cE[c] = (AT)cEm[c]; }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) { cP[c] = sum_groups(cP[c]); cE[c] = sum_groups(cE[c]); }
        if (g == 0) {
            const size_t cb = ps.col(tc.I, tc.J, sub) + col0;
#pragma unroll
            for (int c = 0; c < 4; ++c) { put_part(a.partP, cb + c, cP[c], p32); put_part(a.partE, cb + c, cE[c], p32); }
        }
    } else {
        __syncthreads();
        if (tid >= 4 * u0 && tid < 4 * u1) {
            const size_t rowslot = ps.row(tc.I, tc.J) + tid;
            put_part(a.partP, rowslot, ((AT)sm.rP[0][tid] + (AT)sm.rP[1][tid]) + ((AT)sm.rP[2][tid] + (AT)sm.rP[3][tid]), p32);
            put_part(a.partE, rowslot, ((AT)sm.rE[0][tid] + (AT)sm.rE[1][tid]) + ((AT)sm.rE[2][tid] + (AT)sm.rE[3][tid]), p32);
        }
    }
    if (__any(bad) && l == 0) st->bad = 1;
}

// One visit of the grouped schedule over the entries list[0, n).
template <class ST, class MT, class AT, int KSRC, int GK, int D, int SER>
__global__ __launch_bounds__(WG) void k_sweep_dir(SweepArgs a, const uint32_t* __restrict__ list, int t) {
    using DT = DirTypes<ST, MT, AT, D, SER>;
    __shared__ DirSmem<typename DT::XT, typename DT::LT, AT, typename DT::RT, DT::NRL, KSRC == KSRC_RECOMPUTE,
                       (KSRC == KSRC_PLANE && D >= 1 && std::is_same<ST, float>::value) ? KRING : 0> sm;
    if (a.st->done) return;
    const uint32_t e = list[blockIdx.x / a.split];
    const int sub = blockIdx.x % a.split;
    const int64_t tile = (int64_t)(e & GE_TILE);
    const bool within = (e & GE_WITHIN) != 0;
    if (e & GE_BWD) sweep_tile_dir<ST, MT, AT, KSRC, GK, D, SER, false>(a, tile, within, t, sm, sub);
    else sweep_tile_dir<ST, MT, AT, KSRC, GK, D, SER, true>(a, tile, within, t, sm, sub);
}

// Served grouped visit: items are (request, list entry) pairs of every
// request's current group, built by the host per step; the sweep index of a
// request is its own count of completed sweeps.
template <class ST, class MT, class AT, int D, int SER>
__global__ __launch_bounds__(WG) void k_sweep_dir_batched(const ReqDesc* __restrict__ reqs,
                                                         const uint2* __restrict__ items, int nitems) {
    using DT = DirTypes<ST, MT, AT, D, SER>;
    __shared__ DirSmem<typename DT::XT, typename DT::LT, AT, typename DT::RT, DT::NRL, 0> sm;
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const uint2 w = items[it];
        const ReqDesc& rd = reqs[w.x & 0xFFFFu];
        const int sub = (int)(w.x >> 16);
        const DevStatus* st = rd.sw.st;
        if (st->done) continue;
        const uint32_t e = w.y;
        const int64_t tile = (int64_t)(e & GE_TILE);
        const bool within = (e & GE_WITHIN) != 0;
        if (e & GE_BWD) sweep_tile_dir<ST, MT, AT, KSRC_PLANE, GRAM_F32, D, SER, false>(rd.sw, tile, within, st->t, sm, sub);
        else sweep_tile_dir<ST, MT, AT, KSRC_PLANE, GRAM_F32, D, SER, true>(rd.sw, tile, within, st->t, sm, sub);
        __syncthreads();
    }
}

// Stored records inside a group: both directions from the previous values
// (Jacobi within the group), over the listed tiles.
template <class ST, class MT, class AT, int KSRC, int GK>
__global__ __launch_bounds__(WG) void k_sweep_listed(SweepArgs a, const uint32_t* __restrict__ list) {
    if (a.st->done) return;
    sweep_tile<ST, MT, AT, KSRC, GK, 0, false, 0>(a, (int64_t)(list[blockIdx.x / a.split] & GE_TILE), 0, nullptr,
                                                  a.split, blockIdx.x % a.split);
}

// Served form: one persistent grid walks the union work list of (request
// | row part << 16, tile) items of the active requests of one group (same precision, edge
// state and level count).  Each request keeps its own planes or aggregate
// ring, partial sums and status, so its arithmetic does not depend on the
// mix; the ring slot of the previous sweep follows from the request's own
// sweep count (ring slots of the sweeps before sweep 0 hold P~ = inf, S = 0,
// so a fixed level count is exact from the first sweep).
template <class ST, class MT, class AT, int D, int SER>
__global__ __launch_bounds__(WG) void k_sweep_batched(const ReqDesc* __restrict__ reqs,
                                                     const uint2* __restrict__ items, int nitems) {
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const uint2 w = items[it];
        const ReqDesc& rd = reqs[w.x & 0xFFFFu];
        const DevStatus* st = rd.sw.st;
        if (st->done) continue;
        sweep_tile<ST, MT, AT, KSRC_PLANE, GRAM_F32, D, false, SER>(rd.sw, (int64_t)w.y, st->t % rd.sw.R, nullptr,
                                                                    rd.sw.split, (int)(w.x >> 16));
        __syncthreads();
    }
}

// Launch groups whose plan may run over 2 x 2 chunks of tiles: a request
// whose single solve takes chunks (sw.chunk = 2) takes the same chunks here
// (items (request, Ic << 16 | Jc)), so that both sum in the same order; the
// others take whole tiles (items (request, tile)).
template <class ST, class MT, class AT, int D, int SER>
__global__ __launch_bounds__(WG) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_sweep_batched_chunk(
    const ReqDesc* __restrict__ reqs, const uint2* __restrict__ items, int nitems) {
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const uint2 w = items[it];
        const ReqDesc& rd = reqs[w.x & 0xFFFFu];
        const DevStatus* st = rd.sw.st;
        if (st->done) continue;
        if (rd.sw.chunk > 1)
            sweep_chunk<ST, MT, AT, GRAM_F32, D, SER, 2>(rd.sw, (int)(w.y >> 16), (int)(w.y & 0xFFFFu), st->t % rd.sw.R);
        else
            sweep_tile<ST, MT, AT, KSRC_PLANE, GRAM_F32, D, false, SER>(rd.sw, (int64_t)w.y, st->t % rd.sw.R, nullptr,
                                                                        rd.sw.split, (int)(w.x >> 16));
        __syncthreads();
    }
}

// Run-time (levels, reciprocal form) of a stateless launch to the
// compile-time pair (D, SER): exact reciprocals up to 8 levels, the series
// (one- or two-term top level) up to 6.  Every pair is its own
// instantiation, so the level loops are fully unrolled and branch-free.  The
// forms of kSerLevels run where the powers of K' leave the range.
template <class F>
inline hipError_t with_stateless(int levels, int ser, F&& f) {
    using std::integral_constant;
#define GABP_SL(S_, L_) \
    case (S_) * 16 + L_: f(integral_constant<int, L_>{}, integral_constant<int, S_>{}); return hipSuccess;
    switch (ser * 16 + levels) {
        GABP_SL(0, 1) GABP_SL(0, 2) GABP_SL(0, 3) GABP_SL(0, 4) GABP_SL(0, 5) GABP_SL(0, 6) GABP_SL(0, 7) GABP_SL(0, 8)
        GABP_SL(1, 1) GABP_SL(1, 2) GABP_SL(1, 3) GABP_SL(1, 4) GABP_SL(1, 5) GABP_SL(1, 6)
        GABP_SL(2, 1) GABP_SL(2, 2) GABP_SL(2, 3) GABP_SL(2, 4) GABP_SL(2, 5) GABP_SL(2, 6)
        GABP_SL(3, 3) GABP_SL(3, 4) GABP_SL(3, 5) GABP_SL(3, 6)
        GABP_SL(1 + kSerLevels, 2) GABP_SL(3 + kSerLevels, 3)
        default: return hipErrorInvalidValue;
    }
#undef GABP_SL
}

template <class ST, class MT, class AT, int D, int SER>
inline void served_d(bool grouped, const ReqDesc* reqs, const uint2* items, int n, hipStream_t s) {
    const int g = std::max(1, std::min(n, 2048));
    if (grouped)
        hipLaunchKernelGGL((k_sweep_dir_batched<ST, MT, AT, D, (SER & ~kSerLevels)>), dim3(g), dim3(WG), 0, s, reqs, items, n);
    else if constexpr (chunk_sweep_ok<ST, MT, AT, KSRC_PLANE, D, SER>())
        hipLaunchKernelGGL((k_sweep_batched_chunk<ST, MT, AT, D, SER>), dim3(g), dim3(WG), 0, s, reqs, items, n);
    else
        hipLaunchKernelGGL((k_sweep_batched<ST, MT, AT, D, SER>), dim3(g), dim3(WG), 0, s, reqs, items, n);
}

// levels 0: stored pair records; 1..8 stateless (1..6 with the series);
// grouped: the single-direction entries of one group visit (items
// (request, entry)); otherwise whole tiles (items (request, tile)).
template <class ST, class MT, class AT>
inline hipError_t served_sweep(int levels, int ser, bool grouped, const ReqDesc* reqs, const uint2* items, int n,
                               hipStream_t s) {
    if (levels == 0) {
        served_d<ST, MT, AT, 0, 0>(grouped, reqs, items, n, s);
        return hipGetLastError();
    }
    const hipError_t e = with_stateless(levels, ser, [&](auto L_, auto S_) {
        served_d<ST, MT, AT, decltype(L_)::value, decltype(S_)::value>(grouped, reqs, items, n, s);
    });
    return e != hipSuccess ? e : hipGetLastError();
}

// Launches `kern` on `s`. With an event pair the events take the dispatch's
// own begin and end timestamps (no marker packets around the kernel, so the
// span is the kernel's duration alone), either of which may be missing (one
// sweep in several launches); without, a plain launch.
template <class K, class... Args>
inline void launch_ev(K kern, dim3 g, dim3 b, hipStream_t s, hipEvent_t e0, hipEvent_t e1, Args... args) {
    if (e0 || e1)
        hipExtLaunchKernelGGL(kern, g, b, 0, s, e0, e1, 0, args...);
    else
        hipLaunchKernelGGL(kern, g, b, 0, s, args...);
}

// ---- sweep dispatch: precision x K' source x Gram kind x depth x first x series

template <class ST, class MT, class AT, int KSRC, int GK, int D, int SER>
inline hipError_t sweep_d(bool first, const SweepArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (a.ntiles * a.split > kMaxBlocks) {
        // (only without planes: K' of so many tiles does not fit the memory)
        if constexpr (KSRC == KSRC_RECOMPUTE && D >= 1) {
            if (a.split != 1) return hipErrorInvalidValue;
            return in_launches(a.ntiles, [&](int64_t o, int64_t n) {
                SweepArgs p = a;
                p.tiles = a.tiles + o;
                p.ntiles = n;
                return sweep_d<ST, MT, AT, KSRC, GK, D, SER>(first, p, s, o == 0 ? e0 : nullptr,
                                                             o + n == a.ntiles ? e1 : nullptr);
            });
        } else {
            return hipErrorInvalidValue;
        }
    }
    const dim3 g((unsigned)(a.ntiles * a.split)), blk(WG);
    if (a.chunk > 1) {
        if constexpr (chunk_sweep_ok<ST, MT, AT, KSRC, D, SER>()) {
            if (a.chunk != 2 || a.chunks == nullptr || a.nchunks <= 0) return hipErrorInvalidValue;
            launch_ev(k_sweep_chunk<ST, MT, AT, GK, D, SER, 2>, dim3((unsigned)a.nchunks), blk, s, e0, e1, a);
            return hipSuccess;
        } else {
            return hipErrorInvalidValue;
        }
    }
    if constexpr (D == 0 && KSRC == KSRC_PLANE) {
        if (a.period > 1) {
            // sweep a.between + 1 of its period: the planes written by the
            // last one only (before the first period's end they are zero)
            static_assert(kStoredPeriod == 3, "one instantiation per sweep of the period");
            if (a.period != kStoredPeriod || a.between < 0 || a.between >= kStoredPeriod) return hipErrorInvalidValue;
#define GABP_ST(F_, X_) launch_ev(k_sweep_st<ST, MT, AT, KSRC, GK, F_, X_, X_ == kStoredPeriod - 1>, g, blk, s, e0, e1, a)
            switch (a.between + (first ? kStoredPeriod : 0)) {
                case 0: GABP_ST(false, 0); break;
                case 1: GABP_ST(false, 1); break;
                case 2: GABP_ST(false, 2); break;
                case 3: GABP_ST(true, 0); break;
                case 4: GABP_ST(true, 1); break;
                default: GABP_ST(true, 2); break;
            }
#undef GABP_ST
            return hipSuccess;
        }
    }
    if constexpr (D == 0) {
        if (first) {
            launch_ev(k_sweep<ST, MT, AT, KSRC, GK, D, true, 0>, g, blk, s, e0, e1, a);
            return hipSuccess;
        }
    }
    if constexpr (KSRC == KSRC_RECOMPUTE && GK != GRAM_F32 && D == 3 && SER == 3 && MsgT<ST, MT, AT, SER>::F32) {
        // K' straight from the MFMA output: augmented rows of 32 or 64
        // features, at least one band per wave
        if (a.F.aug0 && a.split <= 2 && (a.F.m_pad == 32 || a.F.m_pad == 64)) {
            if (a.F.m_pad == 32) launch_ev(k_sweep_rc_mom<GK, 32>, g, blk, s, e0, e1, a);
            else launch_ev(k_sweep_rc_mom<GK, 64>, g, blk, s, e0, e1, a);
            return hipSuccess;
        }
    }
    if constexpr (KSRC == KSRC_RECOMPUTE && D >= 1)
        launch_ev(k_sweep_rc<ST, MT, AT, GK, D, SER>, g, blk, s, e0, e1, a);
    else
        launch_ev(k_sweep<ST, MT, AT, KSRC, GK, D, false, SER>, g, blk, s, e0, e1, a);
    return hipSuccess;
}

// `levels` = 0: stored edge state; >= 1: stateless with exactly that many
// levels; `ser`: 0 exact reciprocals, 1 / 2 series with a one- / two-term
// top level. e0 / e1 (optional): timestamps of the launch.
template <class ST, class MT, class AT, int KSRC, int GK>
inline hipError_t sweep_depth(int levels, bool first, int ser, const SweepArgs& a, hipStream_t s, hipEvent_t e0,
                              hipEvent_t e1) {
    if (levels == 0) {
        const hipError_t e = sweep_d<ST, MT, AT, KSRC, GK, 0, 0>(first, a, s, e0, e1);
        return e != hipSuccess ? e : hipGetLastError();
    }
    hipError_t ed = hipSuccess;
    const hipError_t e = with_stateless(levels, ser, [&](auto L_, auto S_) {
        ed = sweep_d<ST, MT, AT, KSRC, GK, decltype(L_)::value, decltype(S_)::value>(first, a, s, e0, e1);
    });
    if (e != hipSuccess) return e;
    return ed != hipSuccess ? ed : hipGetLastError();
}

// ---- grouped schedule dispatch: one group visit
template <class ST, class MT, class AT, int KSRC, int GK, int D, int SER>
inline void grouped_d(const SweepArgs& a, const uint32_t* list, int n, int t, hipStream_t s) {
    (void)in_launches((int64_t)n * a.split, [&](int64_t o, int64_t m) {     // (kMaxBlocks holds whole entries)
        hipLaunchKernelGGL((k_sweep_dir<ST, MT, AT, KSRC, GK, D, SER>), dim3((unsigned)m), dim3(WG), 0, s, a,
                           list + o / a.split, t);
        return hipSuccess;
    });
}

// Stored records (levels 0): the tiles inside the group in `within` (both
// directions), the others in `dir`; stateless: every entry in `dir`.
template <class ST, class MT, class AT, int KSRC, int GK>
inline hipError_t sweep_grouped(int levels, int ser, const SweepArgs& a, const uint32_t* within, int nwithin,
                                const uint32_t* dir, int ndir, int t, hipStream_t s) {
    if (levels == 0) {
        if (nwithin > 0)
            hipLaunchKernelGGL((k_sweep_listed<ST, MT, AT, KSRC, GK>), dim3((unsigned)(nwithin * a.split)), dim3(WG), 0, s, a,
                               within);
        grouped_d<ST, MT, AT, KSRC, GK, 0, 0>(a, dir, ndir, t, s);
        return hipGetLastError();
    }
    const hipError_t e = with_stateless(levels, ser, [&](auto L_, auto S_) {
        grouped_d<ST, MT, AT, KSRC, GK, decltype(L_)::value, (decltype(S_)::value & ~kSerLevels)>(a, dir, ndir, t, s);
    });
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace gabp
