// kernels.hip -- gfx950 kernels of the supernodal Cholesky numeric phase and
// of the triangular solves.
//
// Storage: supernode s is an m_s x w_s column-major panel at Lx + lptr[s]
// (leading dimension m_s); row k of the panel is global row rows[rptr[s]+k]
// of the permuted matrix, the first w_s rows are the columns of s.  Each
// supernode is cut into column blocks of kNB; the inverse of every block's
// diagonal triangle is kept (column-major nb x nb) at Linv + inv_off[blk].
//
// Kernels (paper Sec. 3, Listing 1 names the dense operations):
//   k_assemble     scatter A into the zeroed panels
//   k_level        what a level starts with: whole small and tiny supernodes,
//                  and POTRF of the first diagonal blocks of the wide ones,
//                  with the block inverses
//   k_tiles        MFMA tiles: TRSM (rows times the transposed block
//                  inverse), trailing SYRK/GEMM inside a supernode, and the
//                  SYRK/GEMM update scatter-added through relative indices
//                  into ancestor panels
//   k_solve_fwd / k_solve_bwd   block-level forward / backward substitution
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <mutex>
#include <type_traits>

#include "kernels.h"

namespace spc {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
    using acc = d4;
    // D(16x16) += A(16x4) B(4x16): lane l supplies A[l%16][l/16] and
    // B[l/16][l%16]; element v of lane l is D[l/16 + 4v][l%16] (measured on
    // gfx950: the four rows of a lane are interleaved by 4).
    static __device__ __forceinline__ acc run(double a, double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};
template <>
struct Mfma<float> {
    using acc = f4;
    // same operand layout; element v of lane l is D[4*(l/16) + v][l%16]
    static __device__ __forceinline__ acc run(float a, float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};

// BF16 updates (SPC_FP32_BF16UPD): D(16x16, FP32) += A(16x32) B(32x16) with
// both operands rounded to BF16 (round to nearest even).  Lane l supplies
// eight consecutive k of row l%16 of A and of column l%16 of B, k = 8 (l/16)
// .. 8 (l/16) + 7; the same k order for A and B is all a sum over k needs.
// D is laid out as in the FP32 16x16x4 shape: element v of lane l is
// D[4 (l/16) + v][l%16].
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f4 mfma_bf16(bf16x8 a, bf16x8 b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// Eight FP32 values as eight BF16 (16 bytes) for an LDS row of k.
__device__ __forceinline__ bf16x8 to_bf16x8(const float *v) {
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = (__bf16)v[e];
    return r;
}

__device__ __forceinline__ bool finite_pos(double d) { return d > 0.0 && d <= 1.7976931348623157e308; }
__device__ __forceinline__ bool finite_pos(float d) { return d > 0.0f && d <= 3.402823466e38f; }

template <typename T>
__global__ void k_zero(T *x, int64_t count) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < count; i += stride) x[i] = T(0);
}

__global__ void k_status_reset(unsigned long long *status, int count, int32_t *deverr, int32_t *flags, int nflags) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) status[i] = ~0ull;
    if (i < nflags) flags[i] = 0;
    if (i < 2) deverr[i] = 0;  // the device-error word and the raised-pivot count
}

// Data handed from one workgroup to another inside a launch (which may run
// on another XCD, with its own L2) moves through device-scope atomic loads
// and stores, and the flag that announces it is raised only after the
// writer's own stores have completed; no cache-wide fences.
template <typename T>
__device__ __forceinline__ T dev_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void dev_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Every wait on another workgroup is bounded: after a number of polls
// chosen by the host (about a second's worth by default) it gives up, sets
// the factor's device-error word and goes on, so every wave always exits;
// the host then reports SPC_DEVICE_ERROR.  The pivot status word is never
// used for this.
__device__ __forceinline__ void flag_device_error(int32_t *deverr) {
    __hip_atomic_fetch_or(deverr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Values handed over through memory that the reader polls (the persistent
// solve sweeps' buffers, the last panel of a handed-over block): filled with
// a signalling-NaN pattern before the sweep, which no arithmetic result
// takes (a NaN that arithmetic yields is quiet), so a reader polls the
// value itself and the writer needs no flag after it.
template <typename T>
struct Unset;
template <>
struct Unset<double> {
    using bits_t = unsigned long long;
    static constexpr bits_t bits = 0x7ff5a5a5a5a5a5a5ull;
};
template <>
struct Unset<float> {
    using bits_t = unsigned int;
    static constexpr bits_t bits = 0x7fa5a5a5u;
};
template <typename T>
__device__ __forceinline__ bool is_unset(T v) {
    return __builtin_bit_cast(typename Unset<T>::bits_t, v) == Unset<T>::bits;
}
// Bounded waits: poll an int until it holds `want`; after `spin` polls
// (about a second by default) give up, flag err and go on, so every wave
// always exits.  Once any wait has given up, the others stop waiting too.
__device__ __forceinline__ void wait_value(int32_t *p, int32_t want, int32_t *err, int32_t spin) {
    for (int it = 0; it < spin; ++it) {
        if (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == want) return;
        // once any wait has given up, the others stop waiting too
        if ((it & 255) == 255 && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
        __builtin_amdgcn_s_sleep(2);
    }
    flag_device_error(err);
}

template <typename T>
__global__ void k_assemble(const int64_t *amap, int64_t nnz, const double *values, T *Lx) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < nnz) Lx[amap[k]] = (T)values[k];
}

// Pivot floors of the BF16-update factorization: theta times the diagonal
// entry of A of each permuted column.
template <typename T>
__global__ void k_pivot_floor(const int64_t *dsrc, int64_t n, const double *values, double theta, T *floor) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) floor[j] = (T)(theta * values[dsrc[j]]);
}

// ---------------------------------------------------------------------------
// Global loads in the kernels below are issued unconditionally from clamped,
// always valid indices and masked afterwards, in groups, so that a wave has
// many loads in flight: a load under a branch makes the compiler wait for
// memory at the join, which serializes a loop of them.
// ---------------------------------------------------------------------------

template <typename T>
__device__ __forceinline__ T lane_read(T v, int src);
template <>
__device__ __forceinline__ double lane_read<double>(double v, int src) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), src);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <>
__device__ __forceinline__ float lane_read<float>(float v, int src) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}

// 1/sqrt(d): hardware estimate refined by Newton steps (two in double),
// so the pivot chain has no division.
__device__ __forceinline__ double rsqrt_nr(double d) {
    double y = __builtin_amdgcn_rsq(d);
    y = y * (1.5 - 0.5 * d * y * y);
    return y * (1.5 - 0.5 * d * y * y);
}
__device__ __forceinline__ float rsqrt_nr(float d) {
    float y = __builtin_amdgcn_rsqf(d);
    return y * (1.5f - 0.5f * d * y * y);
}

// Completes a wave's own LDS operations (and keeps the compiler from moving
// memory accesses across), so its later LDS reads of other lanes' data, and
// other waves after a flag, see them.  Global memory operations in flight
// are not waited for.
__device__ __forceinline__ void wave_lds_sync() {
    __asm__ volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __asm__ volatile("" ::: "memory");
}
// Value of lane C of each row of 16 lanes, in every lane of that row.
template <int C>
__device__ __forceinline__ double row_bcast(double v) {
    return __longlong_as_double(
        __builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), 0x150 + C, 0xf, 0xf, true));
}
template <int C>
__device__ __forceinline__ float row_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + C, 0xf, 0xf, true));
}

// Sums across lanes without a trip through LDS.  pair_add<CTRL>: v plus the
// value of the lane that the DPP control names (kXor1, kXor2: inside a quad;
// kRor4, kRor8: rotations of a row of 16); half_add<16 or 32>: v plus that of
// the lane 16 or 32 away.
constexpr int kXor1 = 0xb1, kXor2 = 0x4e, kRor4 = 0x124, kRor8 = 0x128;
template <int CTRL>
__device__ __forceinline__ float pair_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double pair_add(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return v + __longlong_as_double(((long long)hi << 32) | (uint32_t)lo);
}
template <int D>
__device__ __forceinline__ auto half_swap(uint32_t v) {
    static_assert(D == 16 || D == 32, "rows or halves of the wave");
    if constexpr (D == 16) return __builtin_amdgcn_permlane16_swap(v, v, false, false);
    else return __builtin_amdgcn_permlane32_swap(v, v, false, false);
}
template <int D>
__device__ __forceinline__ float half_add(float v) {
    const auto r = half_swap<D>((uint32_t)__float_as_int(v));
    return __int_as_float((int)r[0]) + __int_as_float((int)r[1]);
}
template <int D>
__device__ __forceinline__ double half_add(double v) {
    const long long b = __double_as_longlong(v);
    const auto lo = half_swap<D>((uint32_t)b), hi = half_swap<D>((uint32_t)(b >> 32));
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) +
           __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}

// 1/d: hardware estimate and one correction step (of third order in double,
// whose estimate is good to about 1e-8).
__device__ __forceinline__ double rcp_nr(double d) {
    const double y = __builtin_amdgcn_rcp(d), e = fma(-d, y, 1.0);
    return fma(y, fma(e, e, e), y);
}
__device__ __forceinline__ float rcp_nr(float d) {
    const float y = __builtin_amdgcn_rcpf(d);
    return fmaf(y, fmaf(-d, y, 1.0f), y);
}
// Diagonals of an elimination that takes 1/d: beyond these 1/d would be
// subnormal or overflow (the pivots themselves can be smaller than the
// diagonal by its rounding), and the tile is scaled first, each column by its
// own power of two (pivot_exponent: 2^e times 2^e is about d).
template <typename T>
struct PivotRange;
template <>
struct PivotRange<double> {
    static constexpr double big = 0x1p1000, small = 0x1p-960;
};
template <>
struct PivotRange<float> {
    static constexpr float big = 0x1p100f, small = 0x1p-100f;
};
template <typename T>
__device__ __forceinline__ bool pivot_far(T d) {
    return d > PivotRange<T>::big || (d > T(0) && d < PivotRange<T>::small);
}
__device__ __forceinline__ int pivot_exponent(double d) { return __builtin_amdgcn_frexp_exp(d) >> 1; }
__device__ __forceinline__ int pivot_exponent(float d) { return __builtin_amdgcn_frexp_expf(d) >> 1; }
__device__ __forceinline__ double pow2(double, int e) { return __builtin_amdgcn_ldexp(1.0, e); }
__device__ __forceinline__ float pow2(float, int e) { return __builtin_amdgcn_ldexpf(1.0f, e); }

// Elimination steps C.. of a 16x16 diagonal tile, by one wave.  Every row of
// 16 lanes holds the whole symmetric tile: t[k] of lane c is entry (k, c).
// Step C: w = u_Cc / d_C for the lanes c > C, and every row k > C loses
// u_kC w, u_kC broadcast inside the row of lanes; lane C keeps its column.
// The same w updates NX row tiles below (x[4 u + v], in the layout of an
// MFMA result: column = lane, so u_iC is a broadcast too), or, with INV, the
// rows z of an identity, which end as the inverse of the unit triangle.
// dl of lane C receives d_C.  The chain from pivot to pivot is a
// reciprocal and four dependent multiply-adds; there is no square root in
// it (the columns are scaled afterwards, all at once).
template <typename T, int NX, bool INV, bool BOOST, int C>
__device__ __forceinline__ void eliminate16(T (&t)[16], T (&x)[NX > 0 ? 4 * NX : 1], T (&z)[INV ? 16 : 1], T flo,
                                            T &dl, int &boosted, int l16) {
    if constexpr (C < 16) {
        T d = row_bcast<C>(t[C]);
        if constexpr (BOOST) {
            const T f = row_bcast<C>(flo);
            if (d < f) {  // a NaN compares false and fails the pivot check
                d = f;
                ++boosted;
            }
            t[C] = l16 == C ? d : t[C];
        }
        dl = l16 == C ? d : dl;
        const T y = rcp_nr(d);
        const T w = l16 > C ? t[C] * y : T(0);
#pragma unroll
        for (int k = C + 1; k < 16; ++k) t[k] -= row_bcast<C>(t[k]) * w;
#pragma unroll
        for (int e = 0; e < 4 * NX; ++e) x[e] -= row_bcast<C>(x[e]) * w;
        if constexpr (INV) {
            const T wz = z[C] * y;
#pragma unroll
            for (int k = C + 1; k < 16; ++k) z[k] -= row_bcast<C>(t[k]) * wz;
            // z is off the chain: without this its updates are put off (into
            // the block that stores z) and their broadcasts kept meanwhile,
            // in more registers than there are
#pragma unroll
            for (int k = C + 1; k < 16; ++k) __asm__ volatile("" : "+v"(z[k]));
        }
        eliminate16<T, NX, INV, BOOST, C + 1>(t, x, z, flo, dl, boosted, l16);
    }
}
template <typename T, int K>
__device__ __forceinline__ void scale_rows16(T (&z)[16], T rs) {
    if constexpr (K < 16) {
        z[K] *= row_bcast<K>(rs);
        scale_rows16<T, K + 1>(z, rs);
    }
}

// LDS scratch of potrf_lds beside the block itself: the inverses of the four
// 16x16 diagonal triangles, a tile for each wave but the second, and the
// diagonal of L.
template <typename T>
struct PotrfLds {
    T xd[4][16][17];
    T tile[3][16][17];
    T dg[kNB];
};

// Parts of a panel of a block that is handed out: waves 2 and 3 add 1 each to
// its flag once their part is out.  The last panel has no flag: what the
// tiles below need of it, the inverse of its diagonal triangle, goes straight
// from the wave that forms it to its place in the inverse store, and they
// poll the values there (unset by fill_last_inverse).  With a flag for it the
// tiles of a trailing launch ended 16.8 us (FP32) and 19.2 (FP64) after its
// start, now 14.9 and 17.8; a 34^3 FP32 refined step took 3445 us, now 3398.
constexpr int kPanelParts = 2;

// The last 16x16 diagonal tile of a full block's inverse at Vi, unset: done by
// whoever factors the block before it, in an earlier launch.
template <typename T>
__device__ __forceinline__ void fill_last_inverse(T *Vi) {
    const int a = threadIdx.x & 15, b = threadIdx.x >> 4;
    Vi[(48 + b) * kNB + 48 + a] = __builtin_bit_cast(T, Unset<T>::bits);
}

// Factor the block in A (nb <= 64; rows and columns >= nb hold the identity;
// only the lower triangle is read, what is above the diagonal is scratch),
// write L into P (columns c0.., leading dimension m, lower triangle only) and
// the inverse into Vi; a failed pivot lowers *status to g0 + its column.
// Called by all 256 threads of the workgroup.  With pflags (a full block, nb =
// 64), each panel p is also handed to workgroups of the same launch: its L and
// the inverse of its 16x16 diagonal triangle go out with device-scope atomic
// stores, and each of waves 2 and 3 adds 1 to pflags[p] once its part has
// completed (kPanelParts when the panel is out; the last panel by its values,
// above).  next_full: the supernode's next block is a full one, whose last
// tile of the inverse is unset here.
//
// Four 16-column panels, one workgroup barrier each.  In step p each of the
// panel's tiles below the diagonal (at most three) has a wave of its own (0,
// 2, 3): it brings the diagonal tile and its own up to date with panel p-1
// (16x16x4 MFMA, its own tile staying in registers), eliminates both
// (eliminate16; the diagonal tile by every such wave for itself, so nothing
// crosses between waves inside a panel) and scales the columns.  Wave 1 does
// the same for the diagonal tile with the identity beside it, which gives
// the inverse of its triangle.  Waves 2 and 3 also hand out panel q = p-1,
// apply it to the columns beyond panel p, and carry the block inverse on:
//   X_qj = -X_qq S_qj,  then  S_ij += L_iq X_qj  for i > q  (j <= q),
// with S_ij, later X_ij, in the tile (j, i) of A.  Only the last row's three
// products remain after the last panel.
// L^{-1} is stored column-major: Vi[k * nb + i] = (L^{-1})_ik.
// Bound by the 64 pivots, 125 to 170 cycles each: a chain of a reciprocal and
// four dependent multiply-adds, and a move and a multiply-add to issue for
// every row of the tile and of the one beside it (FP64: 90 to 120 cycles on
// average).  The form before kept a panel's 16 columns in the registers of
// lane = row of one wave, its multipliers read lane by lane into scalar
// registers, had a reciprocal square root in the chain and the inverse after
// it; one block alone took 19.6 us (FP64) and 16.9 (FP32) a launch, this one
// 12.6 and 11.3; the trailing launches of a 34^3 grid's top levels (FP32) 21.7
// and 18.4 on average.
template <typename T, bool BOOST = false>
__device__ __forceinline__ void potrf_lds(T (*A)[kNB + 1], PotrfLds<T> &W, int nb, T *P, int64_t m, int c0, T *Vi,
                                          unsigned long long *status, int64_t g0, int32_t *pflags, bool next_full,
                                          PivotFloor<T> pfl = {}) {
    constexpr int PW = 16;
    using M = Mfma<T>;
    using acc_t = typename M::acc;
    const int t = threadIdx.x;
    int lane = t & 63, l16 = lane & 15, lg = lane >> 4;
    // hides the lane's indices from the optimizer, so that the addresses of
    // one wave's role are not computed ahead of the loop by all of them
    auto fresh = [&] { __asm__ volatile("" : "+v"(lane), "+v"(l16), "+v"(lg)); };
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int npan = (nb + PW - 1) / PW;
    int bad = -1;  // wave 0: first pivot (block column) that failed
    int boosted = 0;
    // rows 16 ti.. and columns 16 tj.. of L L^T over panel q (as a result
    // tile: this lane's column 16 tj + l16)
    auto outer = [&](int ti, int tj, int q) {
        acc_t acc[2] = {acc_t{0, 0, 0, 0}, acc_t{0, 0, 0, 0}};
#pragma unroll
        for (int kk = 0; kk < PW; kk += 4)
            acc[kk >> 3] =
                M::run(A[16 * ti + l16][PW * q + kk + lg], A[16 * tj + l16][PW * q + kk + lg], acc[kk >> 3]);
        return acc[0] + acc[1];
    };
    // panel p: the diagonal tile, with the identity (wave 1) or with the tile
    // of rows 16 ti .. (ti > p; ti = p: none)
    auto panel = [&](int p, int ti, auto nxc, auto invc) {
        constexpr int NX = decltype(nxc)::value;
        constexpr bool INV = decltype(invc)::value;
        const int p0 = PW * p;
        T tt[16], x[NX > 0 ? 4 * NX : 1], z[INV ? 16 : 1], dl = T(1);
        // (xd[p] is written by wave 1 alone)
        T(*D)[17] = INV ? W.xd[p] : W.tile[wv == 0 ? 0 : wv - 1];
        T dmax;
        if (p > 0) {
            const acc_t a0 = outer(p, p, p - 1);
            T cold[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = M::row(lane, v);
                cold[v] = A[p0 + max(r, l16)][p0 + min(r, l16)];
            }
            if constexpr (NX > 0)
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = A[16 * ti + M::row(lane, v)][p0 + l16];
#pragma unroll
            for (int v = 0; v < 4; ++v) D[M::row(lane, v)][l16] = cold[v] - a0[v];
            if constexpr (NX > 0) {
                const acc_t ax = outer(ti, p, p - 1);
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] -= ax[v];
            }
            wave_lds_sync();
#pragma unroll
            for (int k = 0; k < 16; ++k) tt[k] = D[k][l16];
            dmax = D[l16][l16];
        } else {
#pragma unroll
            for (int k = 0; k < 16; ++k) tt[k] = A[max(k, l16)][min(k, l16)];
            if constexpr (NX > 0)
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = A[16 * ti + M::row(lane, v)][l16];
            dmax = A[l16][l16];
        }
        T flo = BOOST ? (p0 + l16 < nb ? pfl.v[g0 + p0 + l16] : T(0)) : T(0);
        // near the ends of the type's range the columns are scaled, S powers
        // of two: the elimination keeps the scale of each column (u becomes
        // u S, d becomes d s), about the root of the diagonal, and d s s is
        // about 1
        T sc = T(1);
        if (__any(pivot_far(dmax))) {
            sc = pow2(T(), -pivot_exponent(dmax));
#pragma unroll
            for (int k = 0; k < 16; ++k) tt[k] *= sc;
#pragma unroll
            for (int e = 0; e < 4 * NX; ++e) x[e] *= sc;
            flo *= sc;
        }
        if constexpr (INV)
#pragma unroll
            for (int k = 0; k < 16; ++k) z[k] = k == l16 ? T(1) : T(0);
        eliminate16<T, NX, INV, BOOST, 0>(tt, x, z, flo, dl, boosted, l16);
        const T rs = rsqrt_nr(dl * sc);  // 1 / (s sqrt(d))
        if constexpr (INV) {
            scale_rows16<T, 0>(z, rs * sc);
            if (lane < 16)
#pragma unroll
                for (int k = 0; k < 16; ++k) D[k][l16] = z[k];
            if (pflags && p == 3) {
                wave_lds_sync();
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = p0 + 4 * e + lg;
                    dev_store(Vi + k * nb + p0 + l16, D[l16][4 * e + lg]);
                }
            }
        } else {
            if constexpr (NX > 0)
#pragma unroll
                for (int v = 0; v < 4; ++v) A[16 * ti + M::row(lane, v)][p0 + l16] = x[v] * rs;
            if (wv == 0) {
                const unsigned long long fail = __ballot(!finite_pos(dl) && lane < 16 && p0 + lane < nb);
                if (fail && bad < 0) bad = p0 + __builtin_ctzll(fail);
                // L of the diagonal tile, transposed, above the diagonal, and
                // its diagonal apart: another wave may still have to read the
                // tile's values before the elimination
                if (lane < 16) {
                    W.dg[p0 + l16] = dl * rs;
#pragma unroll
                    for (int k = 1; k < 16; ++k)
                        if (k > l16) A[p0 + l16][p0 + k] = tt[k] * rs;
                }
            }
        }
    };
    // waves 2 and 3 (h = 0, 1): panel q goes out
    auto store = [&](T *dst, T v) {
        if (pflags) dev_store(dst, v);
        else *dst = v;
    };
    auto hand_out = [&](int q, int h) {
        // columns k0 .. k0 + 7, lane = row
        const int k0 = PW * q + 8 * h;
        T v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = k0 + e;
            v[e] = *(lane == k ? &W.dg[k] : (lane >> 4 == q ? &A[k][lane] : &A[lane][k]));
        }
        T *dst = P + (int64_t)(c0 + k0) * m + c0 + lane;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (k0 + e < nb && lane >= k0 + e && lane < nb) store(dst + e * m, v[e]);
        if (pflags)  // the panel's diagonal 16x16 block of the inverse (full blocks)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int k = 8 * h + 4 * e + lg;
                dev_store(Vi + (PW * q + k) * nb + PW * q + l16, W.xd[q][l16][k]);
            }
    };
    auto flag_out = [&](int q) {
        if (!pflags) return;
        __builtin_amdgcn_s_waitcnt(0);
        if (lane == 0) __hip_atomic_fetch_add(pflags + q, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // X_qj = -X_qq S_qj, in place in the tile (j, q) of A
    auto inverse_tile = [&](int q, int j) {
        acc_t acc[2] = {acc_t{0, 0, 0, 0}, acc_t{0, 0, 0, 0}};
#pragma unroll
        for (int kk = 0; kk < PW; kk += 4)
            acc[kk >> 3] = M::run(W.xd[q][l16][kk + lg], A[PW * j + kk + lg][PW * q + l16], acc[kk >> 3]);
#pragma unroll
        for (int v = 0; v < 4; ++v) A[PW * j + M::row(lane, v)][PW * q + l16] = -(acc[0][v] + acc[1][v]);
    };
    // S_ij += L_iq X_qj (a new sum for q = j), the tile (j, i) of A
    auto inverse_sum = [&](int i, int q, int j) {
        acc_t acc[2] = {acc_t{0, 0, 0, 0}, acc_t{0, 0, 0, 0}};
        if (q > j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[0][v] = A[PW * j + M::row(lane, v)][PW * i + l16];
#pragma unroll
        for (int kk = 0; kk < PW; kk += 4)
            acc[kk >> 3] = M::run(A[PW * i + l16][PW * q + kk + lg],
                                  q == j ? W.xd[q][kk + lg][l16] : A[PW * j + kk + lg][PW * q + l16], acc[kk >> 3]);
#pragma unroll
        for (int v = 0; v < 4; ++v) A[PW * j + M::row(lane, v)][PW * i + l16] = acc[0][v] + acc[1][v];
    };
    // rows 16 r .. of the block inverse to memory, by NTH threads (th)
    auto store_inverse_rows = [&](int r, int th, auto nthc) {
        constexpr int NTH = decltype(nthc)::value, N = PW * kNB / NTH;
        T v[N];
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int e = th + NTH * u, a = e & 15, k = e >> 4, tk = k >> 4, b = k & 15;
            const T *src = tk == r ? &W.xd[r][a][b] : &A[PW * min(tk, r) + a][PW * r + b];
            v[u] = tk <= r ? *src : T(0);
        }
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int e = th + NTH * u, i = PW * r + (e & 15), k = e >> 4;
            if (i < nb && k < nb) Vi[k * nb + i] = v[u];
        }
    };
    using Int0 = std::integral_constant<int, 0>;
    using Int1 = std::integral_constant<int, 1>;
    for (int p = 0; p < npan; ++p) {
        fresh();
        const int ti = p + (wv == 0 ? 1 : wv);  // this wave's tile below the diagonal
        if (wv == 1) panel(p, p, Int0{}, std::true_type{});
        else if (ti < npan) panel(p, ti, Int1{}, std::false_type{});
        else if (wv == 0) panel(p, p, Int0{}, std::false_type{});
        if (p > 0 && wv >= 2) {
            const int h = wv - 2, q = p - 1;
            fresh();
            hand_out(q, h);
            // panel q applied to the tiles (i, j), j > p, and the next rows of
            // the block inverse (columns j of its tiles: wave 3 - j % 2); in
            // step 1 wave 2 has a tile of the panel and wave 3 does both
            int x = 0;
            for (int i = p + 1; i < npan; ++i)
                for (int j = p + 1; j <= i; ++j, ++x) {
                    if (p == 1 ? h == 0 : (x & 1) == h) continue;
                    const acc_t acc = outer(i, j, q);
#pragma unroll
                    for (int v = 0; v < 4; ++v) A[16 * i + M::row(lane, v)][16 * j + l16] -= acc[v];
                }
            flag_out(q);
            for (int j = 1 - h; j <= q; j += 2) {
                if (j < q) {
                    inverse_tile(q, j);
                    wave_lds_sync();
                }
                for (int i = p; i < npan; ++i) inverse_sum(i, q, j);
            }
            if (p > 1) store_inverse_rows(p - 2, lane + 64 * h, std::integral_constant<int, 128>{});
        }
        __syncthreads();
    }
    // the last panel: its 16x16 triangle of L, one entry a thread; the last
    // block row of the inverse (waves 0 .. 2), the one before to memory
    fresh();
    const int q = npan - 1;
    {
        const int i = PW * q + (t & 15), k = PW * q + (t >> 4);
        const T v = i == k ? W.dg[i] : A[k][i];
        if (i >= k && i < nb) P[(int64_t)(c0 + k) * m + c0 + i] = v;
    }
    if (wv < q) inverse_tile(q, wv);
    else if (wv == 3 && q > 0) store_inverse_rows(q - 1, lane, std::integral_constant<int, 64>{});
    if (next_full) fill_last_inverse(Vi + nb * nb);
    if (t == 0 && bad >= 0) atomicMin(status, (unsigned long long)(g0 + bad));
    if (BOOST && t == 0 && boosted) atomicAdd(pfl.count, boosted);
    __syncthreads();
    store_inverse_rows(q, t, std::integral_constant<int, 256>{});
}

// ---------------------------------------------------------------------------
// One workgroup's diagonal block (nb <= kNB = 64), from its panel, held in
// LDS (potrf_lds).
// ---------------------------------------------------------------------------
template <typename T>
struct BlockLds {
    T A[kNB][kNB + 1];
    PotrfLds<T> W;
};
template <typename T, bool BOOST>
__device__ __forceinline__ void potrf_body(const PanelTask &tk, BlockLds<T> &L, T *Lx, T *Linv,
                                           unsigned long long *status, const int32_t *status_slot,
                                           PivotFloor<T> pfl) {
    constexpr int NB = kNB;
    const int64_t m = tk.m;
    const int c0 = tk.c0, nb = tk.c1 - tk.c0;
    T *P = Lx + tk.loff;
    const int t = threadIdx.x;
    {
        T ld[NB * NB / 256];
#pragma unroll
        for (int q = 0; q < NB * NB / 256; ++q) {
            const int e = t + 256 * q, i = e % NB, k = e / NB;
            const int ic = min(i, nb - 1), kc = min(k, ic);
            ld[q] = P[(int64_t)(c0 + kc) * m + c0 + ic];
        }
#pragma unroll
        for (int q = 0; q < NB * NB / 256; ++q) {
            const int e = t + 256 * q, i = e % NB, k = e / NB;
            L.A[i][k] = (i < nb && k <= i) ? ld[q] : (i == k ? T(1) : T(0));
        }
    }
    __syncthreads();
    potrf_lds<T, BOOST>(L.A, L.W, nb, P, m, c0, Linv + tk.ioff, status + (status_slot ? status_slot[tk.s] : 0),
                        tk.g0, nullptr, tk.next_full != 0, pfl);
}

// ---------------------------------------------------------------------------
// Tiny supernodes: one wave per supernode with w <= kTinyW and m <= kTinyM (four per
// workgroup, no barriers): lane = row of the panel, the row's w entries in
// registers, values of other rows read from their lanes.
//   1. column Cholesky: l_jj = sqrt(d_j), l_ij = a_ij / l_jj, then
//      a_ik -= l_ij l_kj for the later columns;
//   2. inverse of the diagonal triangle: lane c < w forms column c by
//      forward substitution;
//   3. the update C[i][k] = sum_j l_ij l_kj of the rows below (w <= k <= i)
//      in 16x16 MFMA tiles (L through LDS; tiles transposed, so 16 lanes add
//      to 16 rows of one target column), scatter-added into the ancestors:
//      C[i][k] goes to cbase[k] + rel[crel[k] + i].
// Pivots that are not positive and finite lower the status word.
// Bound by latency in the narrow levels, where a launch is one round trip
// after the other (task, panel, scatter addresses, atomics), and by the
// atomics in the wide ones.  The scatter addresses do not depend on the
// values, so they are loaded before the factorization (the far row tiles'
// after it, together); loading them 8 columns at a time after it took 21 us a
// launch over the levels of a 34^3 grid (FP32) and 45 over those of the 60^3
// grid (FP64), this form 9 and 38.
// ---------------------------------------------------------------------------
// LDS of one wave's tiny supernode: L[c][row] (the stride puts the four k of
// a 16x16x4 operand in different banks), and the scatter addressing of its
// row positions taken as columns.
template <typename T>
struct TinyLds {
    T l[kTinyW][kTinyM + 16];
    int64_t cb[kTinyM], cr[kTinyM];
};

// One wave's tiny supernode (of k_level and of the persistent launch).  COH: the panel is read with device-scope loads, for a launch in
// which other workgroups (on other XCDs) scatter-added into it.
template <typename T, bool COH>
__device__ __forceinline__ void tiny_body(const SmallTask &tk, TinyLds<T> &L, const int64_t *cbase,
                                          const int64_t *crel, const int32_t *rel, T *Lx, T *Linv,
                                          unsigned long long *status, const int32_t *status_slot,
                                          PivotFloor<T> pfl) {
    constexpr int WT = kTinyW, NTM = kTinyM / 16;  // NTM: row tiles below, at most
    static_assert(NTM == 4, "three near tiles, seven far ones");
    using M = Mfma<T>;
    using acc_t = typename M::acc;
    const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    const int m = tk.m, w = tk.w;
    T *P = Lx + tk.loff;
    const int rc = min(lane, m - 1);
    T r[WT];
#pragma unroll
    for (int c = 0; c < WT; ++c) {
        const T *src = &P[(int64_t)min(c, w - 1) * m + rc];
        r[c] = COH ? dev_load(src) : *src;
    }
    // scatter addresses: lane's row i = w + 16 ti + l16 of C, columns
    // k = w + 16 tj + M::row(lane, v)
    const int nt = (m - w + 15) >> 4;
    if (nt > 0) {
        const int64_t kpos = tk.roff + min(max(lane, w), m - 1);
        const int64_t cb = cbase[kpos], cr = crel[kpos];
        L.cb[lane] = cb;
        L.cr[lane] = cr;
        wave_lds_sync();
    }
    auto row_of = [&](int ti) { return w + 16 * ti + l16; };
    auto col_of = [&](int tj, int v) { return w + 16 * tj + M::row(lane, v); };
    // offsets of the row tiles T0 .. T1 - 1, tile (ti, tj) at ti (ti + 1) / 2 +
    // tj less that of (T0, 0); those of the first two are loaded ahead
    auto offsets = [&](auto t0c, auto t1c, auto &rv) {
        constexpr int T0 = decltype(t0c)::value, T1 = decltype(t1c)::value;
        int x = 0;
#pragma unroll
        for (int ti = T0; ti < T1; ++ti)
#pragma unroll
            for (int tj = 0; tj <= ti; ++tj, ++x)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    rv[x][v] = rel[L.cr[min(col_of(tj, v), m - 1)] + min(max(row_of(ti), col_of(tj, v)), m - 1)];
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, NTM>;
    int32_t near[3][4], far[7][4];
    if (nt > 1) offsets(I0{}, I2{}, near);
    else if (nt == 1) offsets(I0{}, I1{}, near);
    // 1. column Cholesky
    int bad = -1, boosted = 0;
    T rdg[WT];
    const T flo = pfl.v ? pfl.v[tk.g0 + min(lane, w - 1)] : T(0);
#pragma unroll
    for (int c = 0; c < WT; ++c) {
        if (c < w) {
            T d = lane_read(r[c], c);
            if (pfl.v) {
                const T fc = lane_read(flo, c);
                if (d < fc) {
                    d = fc;
                    ++boosted;
                }
            }
            if (bad < 0 && !finite_pos(d)) bad = c;
            const T rs = rsqrt_nr(d);
            rdg[c] = rs;
            const T lic = (lane == c) ? d * rs : r[c] * rs;
            r[c] = lic;
#pragma unroll
            for (int c2 = c + 1; c2 < WT; ++c2)
                if (c2 < w) r[c2] -= lic * lane_read(lic, c2);
        }
    }
    if (lane == 0 && bad >= 0)
        atomicMin(status + (status_slot ? status_slot[tk.s] : 0), (unsigned long long)(tk.g0 + bad));
    if (lane == 0 && boosted) atomicAdd(pfl.count, boosted);
    // 3. update of the rows below, scatter-added into the ancestors
    if (nt > 0) {
#pragma unroll
        for (int c = 0; c < WT; ++c) L.l[c][lane] = c < w ? r[c] : T(0);
        wave_lds_sync();
    }
    auto operand = [&](int t, int h) { return L.l[4 * h + lg][row_of(t)]; };  // columns 4 h + lg of row tile t
    auto update = [&](auto t0c, auto t1c, auto &rv) {
        constexpr int T0 = decltype(t0c)::value, T1 = decltype(t1c)::value;
        int x = 0;
#pragma unroll
        for (int ti = T0; ti < T1; ++ti) {
            if (ti >= nt) break;  // (uniform)
            const T b0 = operand(ti, 0), b1 = operand(ti, 1);
#pragma unroll
            for (int tj = 0; tj <= ti; ++tj, ++x) {
                acc_t acc = {0, 0, 0, 0};
                acc = M::run(operand(tj, 0), b0, acc);
                acc = M::run(operand(tj, 1), b1, acc);
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (row_of(ti) < m && col_of(tj, v) <= row_of(ti))
                        atomicAdd(&Lx[L.cb[col_of(tj, v)] + rv[x][v]], -acc[v]);
            }
        }
    };
    if (nt > 2) offsets(I2{}, I4{}, far);
    if (nt > 1) update(I0{}, I2{}, near);
    else if (nt == 1) update(I0{}, I1{}, near);
    if (nt > 2) update(I2{}, I4{}, far);
    if (lane < m)
#pragma unroll
        for (int c = 0; c < WT; ++c)
            if (c < w && c <= lane) P[(int64_t)c * m + lane] = r[c];
    // 2. inverse of the diagonal triangle, column `lane`
    {
        T y[WT];
#pragma unroll
        for (int a = 0; a < WT; ++a) {
            T v = (a == lane) ? T(1) : T(0);
#pragma unroll
            for (int k = 0; k < a; ++k) v -= lane_read(r[k], a) * y[k];
            y[a] = a < w ? v * rdg[a] : T(0);
        }
        T *Vi = Linv + tk.ioff;
        if (lane < w)
#pragma unroll
            for (int a = 0; a < WT; ++a)
                if (a < w) Vi[lane * w + a] = y[a];
    }
}

// ---------------------------------------------------------------------------
// Grouped tiny supernodes (w <= kGroupW, m <= G): G = 16 or 32 lanes per
// supernode, 64 / G of them per wave, the steps of tiny_body inside each
// group; values of other rows come from their lanes by ds_bpermute (every
// lane of the wave takes part in each exchange, so a lane read is always
// active).  Groups past the end of a launch's list (live false) run on an
// identity block and store nothing.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int32_t pull32(int32_t v, int src) {
    return __builtin_amdgcn_ds_bpermute(src << 2, v);
}
__device__ __forceinline__ double lane_pull(double v, int src) {
    const long long b = __double_as_longlong(v);
    const int lo = pull32((int)(b & 0xffffffffll), src), hi = pull32((int)(b >> 32), src);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ float lane_pull(float v, int src) { return __int_as_float(pull32(__float_as_int(v), src)); }
__device__ __forceinline__ int64_t lane_pull(int64_t v, int src) {
    const int lo = pull32((int)(v & 0xffffffffll), src), hi = pull32((int)(v >> 32), src);
    return ((int64_t)hi << 32) | (uint32_t)lo;
}

template <typename T, int G, bool COH>
__device__ __forceinline__ void group_body(const SmallTask &tk, bool live, const int64_t *cbase, const int64_t *crel,
                                           const int32_t *rel, T *Lx, T *Linv, unsigned long long *status,
                                           const int32_t *status_slot, PivotFloor<T> pfl) {
    constexpr int WG = kGroupW;
    static_assert(G == 16 || G == 32, "group of 16 or 32 lanes");
    const int lane = threadIdx.x & 63, gi = lane & (G - 1), gb = lane - gi;
    const int m = live ? tk.m : 1, w = live ? tk.w : 1;
    T *P = Lx + tk.loff;
    const int rc = min(gi, m - 1);
    T r[WG];
#pragma unroll
    for (int c = 0; c < WG; ++c) {
        if (live) {
            const T *src = &P[(int64_t)min(c, w - 1) * m + rc];
            r[c] = COH ? dev_load(src) : *src;
        } else {
            r[c] = gi == c ? T(1) : T(0);
        }
    }
    int64_t my_cb = 0, my_cr = 0;
    if (live) {
        const int64_t kpos = tk.roff + min(max(gi, w), m - 1);
        my_cb = cbase[kpos];
        my_cr = crel[kpos];
    }
    // scatter addresses of the columns k (lane = row), before the
    // factorization as in tiny_body
    auto column_live = [&](int k) { return live && k >= w && k < m; };
    int32_t rv[G];
#pragma unroll
    for (int k = 0; k < G; ++k) {
        if (k == 0) continue;
        const int64_t crk = lane_pull(my_cr, gb + min(k, m - 1));
        rv[k] = rel[column_live(k) ? crk + min(max(gi, k), m - 1) : 0];
    }
    const T flo = (live && pfl.v) ? pfl.v[tk.g0 + min(gi, w - 1)] : T(0);
    // 1. column Cholesky (columns past w are padding: left alone)
    int bad = -1, boosted = 0;
    T rdg[WG];
#pragma unroll
    for (int c = 0; c < WG; ++c) {
        const bool on = c < w;
        T d = lane_pull(r[c], gb + c);
        if (pfl.v) {
            const T fc = lane_pull(flo, gb + c);
            if (on && d < fc) {
                d = fc;
                ++boosted;
            }
        }
        if (on && bad < 0 && !finite_pos(d)) bad = c;
        const T rs = rsqrt_nr(on ? d : T(1));
        rdg[c] = rs;
        const T lic = (gi == c) ? d * rs : r[c] * rs;
        if (on) r[c] = lic;
#pragma unroll
        for (int c2 = c + 1; c2 < WG; ++c2) {
            const T lk = lane_pull(lic, gb + c2);
            if (on) r[c2] -= lic * lk;
        }
    }
    if (live && gi == 0 && bad >= 0)
        atomicMin(status + (status_slot ? status_slot[tk.s] : 0), (unsigned long long)(tk.g0 + bad));
    if (live && gi == 0 && boosted) atomicAdd(pfl.count, boosted);
    if (live && gi < m)
#pragma unroll
        for (int c = 0; c < WG; ++c)
            if (c < w && c <= gi) P[(int64_t)c * m + gi] = r[c];
    // 2. inverse of the diagonal triangle, column gi
    {
        T y[WG];
#pragma unroll
        for (int a = 0; a < WG; ++a) {
            T v = (a == gi) ? T(1) : T(0);
#pragma unroll
            for (int k = 0; k < a; ++k) v -= lane_pull(r[k], gb + a) * y[k];
            y[a] = a < w ? v * rdg[a] : T(0);
        }
        T *Vi = Linv + tk.ioff;
        if (live && gi < w)
#pragma unroll
            for (int a = 0; a < WG; ++a)
                if (a < w) Vi[gi * w + a] = y[a];
    }
    // 3. update of the rows below, scatter-added into the ancestors
#pragma unroll
    for (int k = 1; k < G; ++k) {
        if (!__any(column_live(k))) continue;
        T a = T(0);
#pragma unroll
        for (int j = 0; j < WG; ++j) {
            const T lk = lane_pull(r[j], gb + min(k, m - 1));
            if (j < w) a += r[j] * lk;
        }
        const int64_t cbk = lane_pull(my_cb, gb + min(k, m - 1));
        if (column_live(k) && gi >= k && gi < m) atomicAdd(&Lx[cbk + rv[k]], -a);
    }
}

// Workgroup b of the tiny supernodes of one level: tasks [0, n16) in groups
// of 16 lanes (16 per workgroup), [n16, n32) in groups of 32 (8 per
// workgroup), the rest one wave each (4 per workgroup); the workgroups of
// the three parts follow each other.
template <typename T>
__device__ __forceinline__ void tiny_block(int64_t b, const SmallTask *tasks, int64_t n16, int64_t n32,
                                           int64_t ntasks, TinyLds<T> *L, const int64_t *cbase, const int64_t *crel,
                                           const int32_t *rel, T *Lx, T *Linv, unsigned long long *status,
                                           const int32_t *status_slot, PivotFloor<T> pfl) {
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t b16 = (n16 + 15) / 16, b32 = (n32 - n16 + 7) / 8;
    if (b < b16) {
        const int64_t gi = b * 16 + wv * 4 + (lane >> 4);
        const bool live = gi < n16;
        group_body<T, 16, false>(tasks[live ? gi : 0], live, cbase, crel, rel, Lx, Linv, status, status_slot, pfl);
        return;
    }
    b -= b16;
    if (b < b32) {
        const int64_t gi = n16 + b * 8 + wv * 2 + (lane >> 5);
        const bool live = gi < n32;
        group_body<T, 32, false>(tasks[live ? gi : n16], live, cbase, crel, rel, Lx, Linv, status, status_slot,
                                 pfl);
        return;
    }
    b -= b32;
    const int64_t ti = n32 + b * 4 + wv;
    if (ti >= ntasks) return;  // the whole wave
    tiny_body<T, false>(tasks[ti], L[wv], cbase, crel, rel, Lx, Linv, status, status_slot, pfl);
}

// ---------------------------------------------------------------------------
// Small supernodes: one workgroup each (w <= kSmallW, m <= kSmallM),
// the whole m x w panel in LDS:
//   1. column Cholesky by panels of 16 columns: each wave holds the panel's
//      16 diagonal rows in lanes 0..15 and 48 rows below in the others, 16
//      columns of a row in registers, pivots and multipliers read from their
//      lanes as for the tiny ones (POTRF of the diagonal block and TRSM of the rows
//      below at once); every wave factors the diagonal rows for itself, so
//      the pivot chain crosses no barrier.  Waves 0..2 cover all the rows.
//      The second panel's columns are brought up to date in 16x16 MFMA tiles
//      in between;
//   2. the inverse of the diagonal triangle (kept for the solves) by wave 3:
//      each 16x16 triangle by forward substitution, lane = column, then
//      inv [L11 0; L21 L22] = [X11 0; -X22 L21 X11  X22];
//   3. the update C = P P^T of the rows below the block in 16x16 MFMA tiles,
//      taken by the waves from a counter and scatter-added into the
//      ancestors: C[i][k] goes to cbase[k] + rel[crel[k] + i].  The tile is
//      formed transposed, so 16 lanes add to 16 rows of one target column.
// Pivots that are not positive and finite lower the status word.
// Bound by latency (a chain of w pivots in a launch of few workgroups, or
// the atomics of the scatter in a wide one): a column at a time with
// three barriers each and a division per entry took 55 us a launch over the
// levels of the 64^2 grid (FP64) and 67 us over those of a batch of 32
// systems (FP32), this form 16 and 32 us.
// ---------------------------------------------------------------------------
// LDS of one small supernode: A[c][i] = panel entry (row i, column c), the
// inverse Vt[c][a] = (L^{-1})_ac, and the scatter addresses of its rows.
// (A's row stride puts the four k of a 16x16x4 operand in different banks.)
template <typename T>
struct SmallLds {
    T A[kSmallW][kSmallM + 16];
    T Vt[kSmallW][kSmallW + 1];
    T U[16][17];
    T rdg[kSmallW];
    int64_t cb[kSmallM], cr[kSmallM];
    int tile;
};

// One workgroup's small supernode (of k_level and of the persistent
// launch); COH as in tiny_body.
template <typename T, bool COH>
__device__ __forceinline__ void small_body(const SmallTask &tk, SmallLds<T> &L, const int64_t *cbase,
                                           const int64_t *crel, const int32_t *rel, T *Lx, T *Linv,
                                           unsigned long long *status, const int32_t *status_slot,
                                           PivotFloor<T> pfl) {
    constexpr int MS = kSmallM, PW = 16, RW = 64 - PW;  // RW: rows below per wave
    static_assert(kSmallW == 2 * PW && 3 * RW >= kSmallM, "two panels; three waves cover the rows");
    using M = Mfma<T>;
    using acc_t = typename M::acc;
    auto &A = L.A;
    auto &Vt = L.Vt;
    const int m = tk.m, w = tk.w;
    T *P = Lx + tk.loff;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int npan = w > PW ? 2 : 1;
    // columns in pairs (128 threads a column); columns w.. of a panel are zero
    auto fill = [&](auto count) {
        constexpr int N = decltype(count)::value;
        T ld[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int e = tid + 256 * q, i = e % MS, c = e / MS;
            const T *src = &P[(int64_t)min(c, w - 1) * m + min(i, m - 1)];
            ld[q] = COH ? dev_load(src) : *src;
        }
        if (tid < MS) {
            const int64_t k = tk.roff + min(max(tid, w), m - 1);
            L.cb[tid] = cbase[k];
            L.cr[tid] = crel[k];
        }
        if (tid == 0) L.tile = 0;
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int e = tid + 256 * q, i = e % MS, c = e / MS;
            A[c][i] = (i < m && c < w) ? ld[q] : T(0);
        }
    };
    if (npan == 1) fill(std::integral_constant<int, PW / 2>{});
    else fill(std::integral_constant<int, PW>{});
    __syncthreads();
    // inverse of the diagonal triangle at p0 (wave 3; lane = column): v holds
    // the right-hand side from row k on, shifted up one row a step, so the
    // step's code is the same for every k
    auto invert16 = [&](int p0) {
        const int w1 = min(w, p0 + PW);
        T v[PW];
#pragma unroll
        for (int a = 0; a < PW; ++a) v[a] = a == l16 ? T(1) : T(0);
#pragma unroll 1
        for (int k = p0; k < w1; ++k) {
            const T y = v[0] * L.rdg[k];
            if (lane < PW) Vt[p0 + l16][k] = y;
#pragma unroll
            for (int a = 1; a < PW; ++a) {
                const T l = A[k][k + a];
                v[a - 1] = v[a] - (k + a < w1 ? l : T(0)) * y;
            }
            v[PW - 1] = T(0);
        }
    };
    int bad = -1, boosted = 0;
#pragma unroll 1
    for (int p = 0; p < npan; ++p) {
        const int p0 = PW * p, b0 = min(w, p0 + PW);
        if (p == 1) {
            // the second panel's columns less the first panel's product:
            // rows 16.. in tiles of 16, tile = (columns) x (rows)
            for (int i0 = PW + 16 * wv; i0 < m; i0 += 64) {
                acc_t acc = {0, 0, 0, 0};
#pragma unroll
                for (int kk = 0; kk < PW; kk += 4) acc = M::run(A[kk + lg][PW + l16], A[kk + lg][i0 + l16], acc);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int c = PW + M::row(lane, v);
                    if (c < w) A[c][i0 + l16] -= acc[v];
                }
            }
            __syncthreads();
        }
        // lanes 0..15: the diagonal rows (identity beyond w); the others: rows b0 + RW wv ..
        const bool dg = lane < PW;
        const int i = dg ? p0 + lane : b0 + RW * wv + lane - PW;
        const bool real = dg ? i < w : i < m;
        T r[PW];
#pragma unroll
        for (int c = 0; c < PW; ++c) {
            const T a = A[p0 + c][min(i, m - 1)];
            r[c] = real ? a : (c == lane ? T(1) : T(0));
        }
        // FP32: the hardware's 1/sqrt takes no subnormal number, so a panel
        // with diagonals near them is scaled by powers of two, each column
        // and each diagonal row by its own
        const T dmax = sizeof(T) == 4 && p0 + l16 < w ? A[p0 + l16][p0 + l16] : T(1);
        const bool far = sizeof(T) == 4 && __any(pivot_far(dmax));
        const int se = far ? pivot_exponent(dmax) : 0;
        __syncthreads();  // every wave has read the diagonal rows that wave 0 stores below
        if (wv < 3 && (wv == 0 || b0 + RW * wv < m)) {
            T mine = T(0);
            T flo = pfl.v ? pfl.v[tk.g0 + min(p0 + l16, w - 1)] : T(0);
            if (far) {
                const T sc = pow2(T(), -se);
#pragma unroll
                for (int c = 0; c < PW; ++c) r[c] = r[c] * lane_read(sc, c) * (dg ? sc : T(1));
                flo = flo * sc * sc;
            }
#pragma unroll
            for (int c = 0; c < PW; ++c) {
                if ((c & 3) == 0 && p0 + c >= w) break;
                T d = lane_read(r[c], c);
                if (pfl.v) {
                    const T fc = lane_read(flo, c);
                    if (d < fc && p0 + c < w) {
                        d = fc;
                        ++boosted;
                    }
                }
                if (bad < 0 && p0 + c < w && !finite_pos(d)) bad = p0 + c;
                // l_cc, 1 / l_cc and l_ic with a correction step each, which
                // leaves the rounding of a square root and a division
                const T rs = rsqrt_nr(d);
                T ld = d * rs;
                ld = fma(fma(-ld, ld, d), T(0.5) * rs, ld);
                if (lane == c) mine = fma(fma(-rs, ld, T(1)), rs, rs);
                const T q = r[c] * rs;
                const T lic = (lane == c) ? ld : fma(fma(-q, ld, r[c]), rs, q);
                r[c] = lic;
#pragma unroll
                for (int c2 = c + 1; c2 < PW; ++c2) r[c2] -= lic * lane_read(lic, c2);
            }
            if (far) {
                mine *= pow2(T(), -se);
                if (dg)
#pragma unroll
                    for (int c = 0; c < PW; ++c) r[c] *= pow2(T(), se);
            }
            if (wv == 0 && dg) L.rdg[p0 + lane] = mine;
            if (real && (wv == 0 || !dg))
#pragma unroll
                for (int c = 0; c < PW; ++c) {
                    if (dg && c > lane) continue;
                    A[p0 + c][i] = r[c];
                    if (p0 + c < w) P[(int64_t)(p0 + c) * m + i] = r[c];
                }
        } else if (wv == 3 && p == 1) {
            invert16(0);
        }
        __syncthreads();
    }
    if (tid == 0 && bad >= 0)
        atomicMin(status + (status_slot ? status_slot[tk.s] : 0), (unsigned long long)(tk.g0 + bad));
    if (tid == 0 && boosted) atomicAdd(pfl.count, boosted);
    if (wv == 3) {
        invert16(PW * (npan - 1));
        wave_lds_sync();
        if (npan == 2) {
            acc_t acc = {0, 0, 0, 0};  // L21 X11
#pragma unroll
            for (int kk = 0; kk < PW; kk += 4) {
                const int k = kk + lg;
                acc = M::run(PW + l16 < w ? A[k][PW + l16] : T(0), Vt[l16][k], acc);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) L.U[M::row(lane, v)][l16] = acc[v];
            wave_lds_sync();
            acc = acc_t{0, 0, 0, 0};  // X22 (L21 X11)
#pragma unroll
            for (int kk = 0; kk < PW; kk += 4)
                acc = M::run(PW + kk + lg < w ? Vt[PW + kk + lg][PW + l16] : T(0), L.U[kk + lg][l16], acc);
#pragma unroll
            for (int v = 0; v < 4; ++v) Vt[l16][PW + M::row(lane, v)] = -acc[v];
            wave_lds_sync();
        }
        T *Vi = Linv + tk.ioff;
        for (int e = lane; e < w * w; e += 64) {
            const int c = e / w, a = e % w;
            Vi[e] = a >= c ? Vt[c][a] : T(0);
        }
    }
    // update of the rows below, scatter-added into the ancestors
    const int mb = m - w, nt = (mb + 15) / 16, ntile = nt * (nt + 1) / 2;
    for (;;) {
        int x = 0;
        if (lane == 0) x = atomicAdd(&L.tile, 1);
        x = __builtin_amdgcn_readfirstlane(x);
        if (x >= ntile) break;
        int ti = 0;
        while ((ti + 1) * (ti + 2) / 2 <= x) ++ti;
        const int tj = x - ti * (ti + 1) / 2;
        const int i = w + 16 * ti + l16, ic = min(i, m - 1);  // row of C
        int64_t cbk[4];
        int32_t rv[4];
        bool ok[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = w + 16 * tj + M::row(lane, v), kc = min(k, ic);  // column of C
            ok[v] = i < m && k <= i;
            cbk[v] = L.cb[kc];
            rv[v] = rel[L.cr[kc] + ic];
        }
        acc_t acc = {0, 0, 0, 0};
        for (int kk = 0; kk < w; kk += 4)
            acc = M::run(A[kk + lg][w + 16 * tj + l16], A[kk + lg][w + 16 * ti + l16], acc);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (ok[v]) atomicAdd(&Lx[cbk[v] + rv[v]], -acc[v]);
    }
}

// ---------------------------------------------------------------------------
// k_level: what a level starts with, in one launch: the first diagonal blocks
// of its wide supernodes, then its small supernodes, then its tiny ones,
// one workgroup range after the other (longest first).  They do not depend
// on each other (their scatter goes to later levels only), and in the narrow
// levels each is a chain of latencies on a few workgroups.  With the tiny
// supernodes in a launch of their own the factorizations of the 64^2 grid
// (FP64) and a 34^3 grid (FP32) took 296 and 2062 us, in one launch 257 and
// 1988; with three launches 325 and 2160.  The wide levels of a batch of 160
// systems lose nothing by the lower occupancy (11.2 ms either way): the
// atomics bound them.
// ---------------------------------------------------------------------------
template <typename T>
union LevelLds {
    BlockLds<T> block;
    SmallLds<T> small;
    TinyLds<T> tiny[4];
};
template <typename T, bool BOOST>
__global__ __launch_bounds__(256, 3) void k_level(const PanelTask *potrf, int npotrf, const SmallTask *small,
                                                  int nsmall, const SmallTask *tiny, int64_t n16, int64_t n32,
                                                  int64_t ntiny, const int64_t *cbase, const int64_t *crel,
                                                  const int32_t *rel, T *Lx, T *Linv, unsigned long long *status,
                                                  const int32_t *status_slot, PivotFloor<T> pfl) {
    __shared__ __align__(16) char mem[sizeof(LevelLds<T>)];
    LevelLds<T> &L = *reinterpret_cast<LevelLds<T> *>(mem);
    const int b = blockIdx.x;
    if (b < npotrf)
        potrf_body<T, BOOST>(potrf[b], L.block, Lx, Linv, status, status_slot, pfl);
    else if (b < npotrf + nsmall)
        small_body<T, false>(small[b - npotrf], L.small, cbase, crel, rel, Lx, Linv, status, status_slot, pfl);
    else
        tiny_block<T>(b - npotrf - nsmall, tiny, n16, n32, ntiny, L.tiny, cbase, crel, rel, Lx, Linv, status,
                      status_slot, pfl);
}

// ---------------------------------------------------------------------------
// k_persist_small: every small subtree of the elimination forest (of every
// system of a batch), all its levels, in one launch.  Resident workgroups
// take queue entries from a work counter; the queue is in level order, so
// every supernode an entry waits for belongs to an earlier entry, which a
// running workgroup holds or has finished: no wait can deadlock.  An entry is
// one small supernode (the workgroup, small_body) or up to four tiny ones
// (one wave each, tiny_body).  Before it starts, a supernode waits until
// every source inside the launch has scatter-added its update into it
// (pdep[s] counted down to 0); after its own scatter-adds have completed
// (s_waitcnt), it counts down each of its targets inside the launch.  The
// scatter-adds are device-scope atomics and the panel is read with
// device-scope loads, so the values cross XCDs without cache-wide fences.
// ---------------------------------------------------------------------------
__global__ void k_persist_reset(const int32_t *pdep0, int64_t ns, int32_t *pdep, int32_t *qctr) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ns) pdep[i] = pdep0[i];
    if (i == 0) *qctr = 0;
}

template <typename T>
__global__ __launch_bounds__(256, 3) void k_persist_small(const PersistEntry *queue, const int32_t *chunk, int64_t nc,
                                                       const SmallTask *psmall,
                                                       const SmallTask *ptiny, const int64_t *ptgt_ptr,
                                                       const int32_t *ptgt, int32_t *pdep, int32_t *qctr,
                                                       const int64_t *cbase, const int64_t *crel, const int32_t *rel,
                                                       T *Lx, T *Linv, unsigned long long *status,
                                                       const int32_t *status_slot, PivotFloor<T> pfl, WaitCtl wc) {
    __shared__ SmallLds<T> L;  // also the four waves' TinyLds
    static_assert(4 * sizeof(TinyLds<T>) <= sizeof(L), "the waves' tiny supernodes fit");
    __shared__ int32_t slot;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (;;) {
        if (tid == 0) slot = atomicAdd(qctr, 1);
        __syncthreads();
        const int64_t c = slot;
        __syncthreads();  // every thread has read the slot
        if (c >= nc) return;
        // the chunk's entries in order: an entry waits only on entries before
        // it, earlier in this chunk (done) or in chunks taken before
        for (int32_t q = chunk[c]; q < chunk[c + 1]; ++q) {
        const PersistEntry e = queue[q];
        if (e.kind == 0) {
            const SmallTask tk = psmall[e.first];
            if (tid == 0) wait_value(&pdep[tk.s], 0, wc.err, wc.spin);
            __syncthreads();
            small_body<T, true>(tk, L, cbase, crel, rel, Lx, Linv, status, status_slot, pfl);
            __builtin_amdgcn_s_waitcnt(0);  // this thread's scatter-adds have completed
            __syncthreads();
            for (int64_t k = ptgt_ptr[tk.s] + tid; k < ptgt_ptr[tk.s + 1]; k += 256) atomicSub(&pdep[ptgt[k]], 1);
        } else if (e.kind == 1) {
            if (wv < e.count) {
                const SmallTask tk = ptiny[e.first + wv];
                if (lane == 0) wait_value(&pdep[tk.s], 0, wc.err, wc.spin);
                __asm__ volatile("" ::: "memory");
                tiny_body<T, true>(tk, reinterpret_cast<TinyLds<T> *>(&L)[wv], cbase, crel, rel, Lx, Linv, status, status_slot, pfl);
                __builtin_amdgcn_s_waitcnt(0);
                for (int64_t k = ptgt_ptr[tk.s] + lane; k < ptgt_ptr[tk.s + 1]; k += 64)
                    atomicSub(&pdep[ptgt[k]], 1);
            }
        } else {
            // kind 2 (3): up to 16 (8) tiny supernodes in groups of 16 (32)
            // lanes; each group's first lane waits for its own supernode
            const int G = e.kind == 2 ? 16 : 32;
            const int gi = wv * (64 / G) + lane / G, gl = lane & (G - 1);
            const bool live = gi < e.count;
            const SmallTask tk = ptiny[e.first + (live ? gi : 0)];
            if (live && gl == 0) wait_value(&pdep[tk.s], 0, wc.err, wc.spin);
            __asm__ volatile("" ::: "memory");
            if (e.kind == 2)
                group_body<T, 16, true>(tk, live, cbase, crel, rel, Lx, Linv, status, status_slot, pfl);
            else
                group_body<T, 32, true>(tk, live, cbase, crel, rel, Lx, Linv, status, status_slot, pfl);
            __builtin_amdgcn_s_waitcnt(0);
            if (live)
                for (int64_t k = ptgt_ptr[tk.s] + gl; k < ptgt_ptr[tk.s + 1]; k += G) atomicSub(&pdep[ptgt[k]], 1);
        }
        __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// MFMA tiles.  One workgroup (4 waves) computes a 64x64 tile C = A B^T,
// each wave a 2x2 set of 16x16x4 MFMA blocks; K staged through LDS 16 at a
// time, the next chunk loaded into registers while the current one is used.
//   MODE_TRAILING: A, B = panel rows i0.., j0..; P[i][j] -= C for i >= j,
//                  j < jmax.  The diagonal tile of the next column block
//                  then factors that block (potrf_lds); a tile below it
//                  with a flag then solves X L^T = P - C for its rows,
//                  following the block's panels as they are handed out,
//                  and stores X instead.  The block's factorization is
//                  claimed by whichever of these workgroups comes first.
//   MODE_SCATTER:  A, B = panel rows i0.., j0..; C (i >= j) scatter-added
//                  atomically into the ancestors: C[i][j] goes to
//                  cbase[j] + rel[crel[j] + i].
//   MODE_TRSM:     B = inverse of block blk (at aux), stored as
//                  Q[k' * nb + c] = (L^{-1})_{c k'}; P[i][k0 + c] = C
//                  (rows times the transposed inverse: X = B L^{-T}).
// ---------------------------------------------------------------------------
enum { MODE_TRAILING = 0, MODE_SCATTER = 1, MODE_TRSM = 2 };

template <typename T, int MODE, bool BF = false>
__global__ __launch_bounds__(256, 3) void k_tiles(const TileTask *tasks, const int64_t *cbase, const int64_t *crel,
                                               const int32_t *rel, T *Linv, T *Lx, unsigned long long *status,
                                               const int32_t *status_slot, int32_t *hflags, WaitCtl wctl,
                                               PivotFloor<T> pfl) {
    constexpr int TM = kTile, KB = 16, CPT = 16;
    using acc_t = typename Mfma<T>::acc;
    __shared__ T ABs[2][KB][TM + 4];  // A and B chunks, one buffer
    __shared__ T Cs[TM][TM + 1];
    __shared__ int64_t cb[TM], cr[TM];
    __shared__ int claimed;
    T(*As)[TM + 4] = ABs[0];
    T(*Bs)[TM + 4] = ABs[1];
    const TileTask own = tasks[blockIdx.x];
    if (MODE == MODE_TRAILING && own.s < 0) return;  // a no-op entry of the launch layout
    // the claim of the next block's factorization (see below): thread 0 of
    // the diagonal tile's workgroup takes it at its start and reads the
    // outcome only before factoring, so the atomic's round trip overlaps the
    // tile's update
    int32_t *const claim = (MODE == MODE_TRAILING && own.flag >= 0) ? hflags + kFlagsPerBlock * own.flag + 4 : nullptr;
    int32_t ticket = 0;
    // one tile task (the whole body; its returns end that task); defer: the
    // diagonal tile's own task, which factors the block only if its ticket
    // won the claim
    auto body = [&](const TileTask tk, bool defer) {
    const int64_t m = tk.m;
    T *P = Lx + tk.loff;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
    acc_t acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = acc_t{0, 0, 0, 0};

    const int lr = tid & 63, lk = tid >> 6;
    const int kw = tk.k1 - tk.k0;
    const bool row_ok = tk.i0 + lr < m;
    const bool col_ok = (MODE == MODE_TRSM) ? lr < kw : tk.j0 + lr < tk.jmax;
    const T *pa = P + min<int64_t>(tk.i0 + lr, m - 1);
    const T *pb = (MODE == MODE_TRSM) ? Linv + tk.aux + min(lr, kw - 1) : P + min(tk.j0 + lr, tk.jmax - 1);
    const int64_t ldb = (MODE == MODE_TRSM) ? kw : m;
    const int kofs = (MODE == MODE_TRSM) ? tk.k0 : 0;
    if (MODE == MODE_SCATTER && tid < TM) {
        const int64_t k = tk.aux + min(tk.j0 + tid, tk.jmax - 1);
        cb[tid] = cbase[k];
        cr[tid] = crel[k];
    }
    // the next K chunk is loaded into registers while the current one is used
    T ra[KB / 4], rb[KB / 4];
    auto load = [&](int kb) {
#pragma unroll
        for (int e = 0; e < KB / 4; ++e) {
            const int k = min(kb + lk + 4 * e, tk.k1 - 1);
            ra[e] = pa[(int64_t)k * m];
            rb[e] = pb[(int64_t)(k - kofs) * ldb];
        }
    };
    const int r = tid & 63, cg = tid >> 6;
    const int64_t gi = tk.i0 + r;
    T old[CPT];  // trailing tiles: the tile's values before the update
    auto load_old = [&] {
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) {
            const int64_t gj = min(tk.j0 + cg * CPT + cc, tk.jmax - 1);
            old[cc] = P[gj * m + min<int64_t>(gi, m - 1)];
        }
    };
    if (MODE == MODE_TRAILING && tk.blk >= 0 && tk.i0 == tk.j0) {
        // the diagonal tile of the next block heads the step's critical
        // path: the tile and its panel rows (A = B) are loaded with one
        // round trip, TM columns of K at a time, staged in Cs
        load_old();
        for (int kb = tk.k0; kb < tk.k1; kb += TM) {
            T xv[TM / 4];
#pragma unroll
            for (int e = 0; e < TM / 4; ++e) xv[e] = pa[(int64_t)min(kb + lk + 4 * e, tk.k1 - 1) * m];
            if (kb > tk.k0) __syncthreads();
#pragma unroll
            for (int e = 0; e < TM / 4; ++e)
                Cs[lk + 4 * e][lr] = (kb + lk + 4 * e < tk.k1 && row_ok) ? xv[e] : T(0);
            __syncthreads();
#pragma unroll
            for (int kk = 0; kk < TM; kk += 4) {
                T af[2], bf[2];
#pragma unroll
                for (int a = 0; a < 2; ++a) af[a] = Cs[kk + (lane >> 4)][wr + a * 16 + (lane & 15)];
#pragma unroll
                for (int b = 0; b < 2; ++b) bf[b] = Cs[kk + (lane >> 4)][wc + b * 16 + (lane & 15)];
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc[a][b] = Mfma<T>::run(af[a], bf[b], acc[a][b]);
            }
        }
        __syncthreads();
    } else if constexpr (BF) {
        // BF16 operands, FP32 accumulation, K staged 32 at a time: thread
        // (row lr, quarter lk) loads k = 8 lk .. 8 lk + 7 of its row of A
        // and of B, rounds them to BF16 and writes each as 16 bytes of an
        // LDS row (k contiguous), which a lane then reads with one load
        static_assert(sizeof(T) == 4, "BF16 updates are for FP32 panels");
        constexpr int KBB = 32, RS = KBB + 8;  // row stride in bf16 (16 bytes of padding)
        // staged in Cs, which the epilogue needs only after the last chunk
        __bf16 *Ab = reinterpret_cast<__bf16 *>(&Cs[0][0]);
        __bf16 *Bb = Ab + TM * RS;
        static_assert(2 * TM * RS * sizeof(__bf16) <= sizeof(Cs), "bf16 staging fits the output tile buffer");
        float fa[8], fb[8];
        auto loadb = [&](int kb) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = min(kb + 8 * lk + e, tk.k1 - 1);
                fa[e] = pa[(int64_t)k * m];
                fb[e] = pb[(int64_t)k * m];
            }
        };
        loadb(tk.k0);
        for (int kb = tk.k0; kb < tk.k1; kb += KBB) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool kin = kb + 8 * lk + e < tk.k1;
                fa[e] = (kin && row_ok) ? fa[e] : 0.0f;
                fb[e] = (kin && col_ok) ? fb[e] : 0.0f;
            }
            *reinterpret_cast<bf16x8 *>(Ab + lr * RS + 8 * lk) = to_bf16x8(fa);
            *reinterpret_cast<bf16x8 *>(Bb + lr * RS + 8 * lk) = to_bf16x8(fb);
            __syncthreads();
            if (kb + KBB < tk.k1) loadb(kb + KBB);
            bf16x8 af[2], bf[2];
#pragma unroll
            for (int a = 0; a < 2; ++a)
                af[a] = *reinterpret_cast<const bf16x8 *>(Ab + (wr + a * 16 + (lane & 15)) * RS + 8 * (lane >> 4));
#pragma unroll
            for (int b = 0; b < 2; ++b)
                bf[b] = *reinterpret_cast<const bf16x8 *>(Bb + (wc + b * 16 + (lane & 15)) * RS + 8 * (lane >> 4));
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = mfma_bf16(af[a], bf[b], acc[a][b]);
            __syncthreads();
        }
        if (MODE == MODE_TRAILING) load_old();
    } else {
        load(tk.k0);
        for (int kb = tk.k0; kb < tk.k1; kb += KB) {
#pragma unroll
            for (int e = 0; e < KB / 4; ++e) {
                const int kk = lk + 4 * e;
                const bool kin = kb + kk < tk.k1;
                As[kk][lr] = (kin && row_ok) ? ra[e] : T(0);
                Bs[kk][lr] = (kin && col_ok) ? rb[e] : T(0);
            }
            __syncthreads();
            if (kb + KB < tk.k1) load(kb + KB);
#pragma unroll
            for (int kk = 0; kk < KB; kk += 4) {
                T af[2], bf[2];
#pragma unroll
                for (int a = 0; a < 2; ++a) af[a] = As[kk + (lane >> 4)][wr + a * 16 + (lane & 15)];
#pragma unroll
                for (int b = 0; b < 2; ++b) bf[b] = Bs[kk + (lane >> 4)][wc + b * 16 + (lane & 15)];
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc[a][b] = Mfma<T>::run(af[a], bf[b], acc[a][b]);
            }
            __syncthreads();
        }
        // epilogue: thread = row r, columns cg*16 .. cg*16+15
        if (MODE == MODE_TRAILING) load_old();
    }
    int32_t rv[CPT];
    if (MODE == MODE_SCATTER) {
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) {
            const int c = cg * CPT + cc;
            const int64_t gj = min(tk.j0 + c, tk.jmax - 1);
            rv[cc] = rel[cr[c] + max(min<int64_t>(gi, m - 1), gj)];
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int rr = wr + a * 16 + Mfma<T>::row(lane, v);
                const int c = wc + b * 16 + (lane & 15);
                Cs[c][rr] = acc[a][b][v];
            }
    __syncthreads();
    if (MODE == MODE_TRAILING && tk.blk >= 0 && tk.i0 == tk.j0) {
        // diagonal tile of the next column block: its rows r < nb2 form the
        // block, final after this update; factor it here (rows below it are
        // stored as in any other tile)
        const int nb2 = min(TM, tk.jmax - tk.j0);
        T nv[CPT];
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) nv[cc] = old[cc] - Cs[cg * CPT + cc][r];
        if (r >= nb2 && gi < m)
#pragma unroll
            for (int cc = 0; cc < CPT; ++cc) {
                const int64_t gj = tk.j0 + cg * CPT + cc;
                if (gj < tk.jmax) P[gj * m + gi] = nv[cc];
            }
        if (defer) {
            if (tid == 0) claimed = ticket == 0;
            __syncthreads();
            if (!claimed) return;  // a tile below took the factorization
        }
        __syncthreads();
        // LDS for the factorization: the tile buffers, free now (cb and cr
        // hold no scatter addresses in this mode)
        T(*A)[TM + 1] = Cs;
        static_assert(sizeof(PotrfLds<T>) <= sizeof(ABs), "the factorization's scratch fits the chunk buffers");
        PotrfLds<T> &W = *reinterpret_cast<PotrfLds<T> *>(&ABs[0][0][0]);
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) {
            const int c = cg * CPT + cc;
            A[r][c] = (r < nb2 && c <= r) ? nv[cc] : (r == c ? T(1) : T(0));
        }
        __syncthreads();
        // with a flag, each panel goes to the tiles below as it comes out
        // (also after a failed pivot, which the status word reports, so
        // that no tile waits in vain)
        potrf_lds<T, BF>(A, W, nb2, P, m, tk.j0, Linv + tk.aux, status + (status_slot ? status_slot[tk.s] : 0),
                         tk.blk, tk.flag >= 0 ? hflags + kFlagsPerBlock * tk.flag : nullptr,
                         tk.j0 + 2 * kNB <= tk.jmax, pfl);
        return;
    }
    if (MODE == MODE_TRAILING && tk.flag >= 0) {
        // below the diagonal tile of a block factored in this launch: the
        // block's TRSM on this tile, X L^T = C (C the updated tile), 16
        // columns at a time as the block's panels come out: X_p = C_p
        // L_pp^{-T}, then C_q -= X_p L_qp^T for the later panels q.  Each
        // wave owns 16 rows of the tile, so the waves never wait for each
        // other, only for the panel flags (kPanelParts once a panel is out).
        static_assert(TM == kNB && TM == 64, "four 16-column panels per block");
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) Cs[cg * CPT + cc][r] = old[cc] - Cs[cg * CPT + cc][r];
        __syncthreads();
        const T *Vi = Linv + tk.aux;                        // (L^{-1})_{jk} at Vi[k * TM + j]
        const T *Lb = P + (int64_t)tk.j0 * m + tk.j0;       // block-local L[i][k] at Lb[k * m + i]
        int32_t *pf = hflags + kFlagsPerBlock * tk.flag;
        const int w16 = wave * 16, l16 = lane & 15, lk4 = lane >> 4;
        bool ok = true;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            // B operands: the inverse of the panel's diagonal triangle,
            // B[k][j] = (L^{-1})_{16p+j,16p+k}, and L below it, B[k][j] =
            // L[16q+j][16p+k], once the panel is out: its flag (every lane
            // reads the same word: one load), or for the last one its values
            T bi[4] = {T(0), T(0), T(0), T(0)}, bl[3][4];
            auto load_inverse = [&] {
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) bi[kk] = dev_load(Vi + (16 * p + 4 * kk + lk4) * TM + 16 * p + l16);
            };
            bool ready = false;
            for (int it = 0; ok && it < wctl.spin; ++it) {
                if (p < 3) {
                    ready = __builtin_amdgcn_readfirstlane(dev_load(pf + p)) >= kPanelParts;
                } else {
                    load_inverse();
                    ready = !__any(is_unset(bi[0]) || is_unset(bi[1]) || is_unset(bi[2]) || is_unset(bi[3]));
                }
                if (ready) break;
                __builtin_amdgcn_s_sleep(1);
            }
            ok = ok && ready;
            __asm__ volatile("" ::: "memory");
            if (p < 3) load_inverse();
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                const int k = 16 * p + 4 * kk + lk4;
#pragma unroll
                for (int q = p + 1; q < 4; ++q) bl[q - p - 1][kk] = dev_load(Lb + (int64_t)k * m + 16 * q + l16);
            }
            // X_p for this wave's rows, staged over C_p in Cs
            acc_t x = {0, 0, 0, 0};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) x = Mfma<T>::run(Cs[16 * p + 4 * kk + lk4][w16 + l16], bi[kk], x);
#pragma unroll
            for (int v = 0; v < 4; ++v) Cs[16 * p + l16][w16 + Mfma<T>::row(lane, v)] = x[v];
            wave_lds_sync();
#pragma unroll
            for (int q = p + 1; q < 4; ++q) {
                acc_t u = {0, 0, 0, 0};
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    u = Mfma<T>::run(Cs[16 * p + 4 * kk + lk4][w16 + l16], bl[q - p - 1][kk], u);
#pragma unroll
                for (int v = 0; v < 4; ++v) Cs[16 * q + l16][w16 + Mfma<T>::row(lane, v)] -= u[v];
            }
            wave_lds_sync();
        }
        if (!ok && lane == 0) flag_device_error(wctl.err);
        __syncthreads();
        if (gi < m)
#pragma unroll
            for (int cc = 0; cc < CPT; ++cc) P[(tk.j0 + cg * CPT + cc) * m + gi] = Cs[cg * CPT + cc][r];
        return;
    }
    if (gi >= m) return;
#pragma unroll
    for (int cc = 0; cc < CPT; ++cc) {
        const int c = cg * CPT + cc;
        const int64_t gj = tk.j0 + c;
        if (gj >= tk.jmax) continue;
        const T v = Cs[c][r];
        if (MODE == MODE_TRSM) {
            P[gj * m + gi] = v;
        } else if (MODE == MODE_TRAILING) {
            if (gj <= gi) P[gj * m + gi] = old[cc] - v;
        } else {
            if (gj <= gi) atomicAdd(&Lx[cb[c] + rv[cc]], -v);
        }
    }
    };
    if (MODE == MODE_TRAILING && own.flag >= 0) {
        // The factorization of the next block (its diagonal tile's update,
        // POTRF and the panels handed out) is one job that the first
        // workgroup of the hand-over to arrive claims: the diagonal tile's,
        // or, if that one has not started yet, a tile below it, which does
        // the job before its own work.  A tile that waits for the panels
        // thus always waits for a workgroup that is running and never waits
        // itself, whatever the dispatch order, the XCDs or other launches.
        // The claim word is cleared with the factorization's status.  The
        // diagonal tile starts at once and looks at its ticket before it
        // factors; a tile below first reads the word and takes a ticket
        // only while nobody has (the diagonal tile, first in the launch,
        // nearly always has).
        if (own.i0 == own.j0) {
            if (threadIdx.x == 0) ticket = __hip_atomic_fetch_add(claim, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            body(own, true);
            return;
        }
        if (threadIdx.x == 0)
            claimed = dev_load(claim) == 0 &&
                      __hip_atomic_fetch_add(claim, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
        __syncthreads();
        const bool mine = claimed;
        __syncthreads();
        if (mine) {
            TileTask d = own;
            d.i0 = d.j0;
            body(d, false);
            __syncthreads();
        }
    }
    body(own, false);
}

// ---------------------------------------------------------------------------
// k_tiles128: the scatter update on 128x128 tiles for the large supernodes
// (same operation as k_tiles in MODE_SCATTER), or, with TRAIL, the bulk
// trailing update inside a wide supernode (as MODE_TRAILING without the
// next block's factorization: P[i][j] -= C for i >= j, j < jmax, in place).
// 8 waves in a 2x4 grid of 64x32 sub-tiles, each a 4x2 set of 16x16x4 MFMA
// blocks, so two waves share each SIMD and hide each other's MFMA latency; K
// staged through LDS 16 at a time with the next chunk in registers while the
// current one is consumed.  The epilogue goes through LDS in four passes of
// 32 columns.
// ---------------------------------------------------------------------------
template <typename T, bool BF = false, bool TRAIL = false>
__global__ __launch_bounds__(512) void k_tiles128(const TileTask *tasks, const int64_t *cbase, const int64_t *crel,
                                                  const int32_t *rel, T *Lx) {
    constexpr int TM = 128, KB = 16, PADA = 4, CPT = 8, NT = 512;
    constexpr int KBB = 32, RS = KBB + 8;  // BF16: K per chunk, LDS row stride (bf16)
    using acc_t = typename Mfma<T>::acc;
    constexpr int kSmem = BF ? (2 * TM * RS * 2 + sizeof(T) - 1) / sizeof(T) : 2 * KB * (TM + PADA);
    __shared__ T smem[kSmem];
    __shared__ int64_t cb[TM], cr[TM];
    T(*As)[TM + PADA] = reinterpret_cast<T(*)[TM + PADA]>(smem);
    T(*Bs)[TM + PADA] = reinterpret_cast<T(*)[TM + PADA]>(smem + KB * (TM + PADA));
    const TileTask tk = tasks[blockIdx.x];
    const int64_t m = tk.m;
    T *P = Lx + tk.loff;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = (wave >> 2) * 64, wc = (wave & 3) * 32;
    acc_t acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = acc_t{0, 0, 0, 0};
    // loader: thread covers row lr (0..127) and k-rows lk, lk+4, lk+8, lk+12
    const int lr = tid & 127, lk = tid >> 7;
    const bool row_ok = tk.i0 + lr < m;
    const bool col_ok = tk.j0 + lr < tk.jmax;
    const T *pa = P + min<int64_t>(tk.i0 + lr, m - 1);
    const T *pb = P + min(tk.j0 + lr, tk.jmax - 1);
    if (!TRAIL && tid < TM) {
        const int64_t k = tk.aux + min(tk.j0 + tid, tk.jmax - 1);
        cb[tid] = cbase[k];
        cr[tid] = crel[k];
    }
    if constexpr (BF) {
        // BF16 operands, FP32 accumulation (as in k_tiles): thread (row lr,
        // quarter lk) stages k = 8 lk .. 8 lk + 7 of its rows of A and B
        static_assert(sizeof(T) == 4, "BF16 updates are for FP32 panels");
        __bf16 *Ab = reinterpret_cast<__bf16 *>(smem);
        __bf16 *Bb = Ab + TM * RS;
        float fa[8], fb[8];
        auto loadb = [&](int kb) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int64_t k = min(kb + 8 * lk + e, tk.k1 - 1);
                fa[e] = pa[k * m];
                fb[e] = pb[k * m];
            }
        };
        loadb(tk.k0);
        for (int kb = tk.k0; kb < tk.k1; kb += KBB) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool kin = kb + 8 * lk + e < tk.k1;
                fa[e] = (kin && row_ok) ? fa[e] : 0.0f;
                fb[e] = (kin && col_ok) ? fb[e] : 0.0f;
            }
            *reinterpret_cast<bf16x8 *>(Ab + lr * RS + 8 * lk) = to_bf16x8(fa);
            *reinterpret_cast<bf16x8 *>(Bb + lr * RS + 8 * lk) = to_bf16x8(fb);
            __syncthreads();
            if (kb + KBB < tk.k1) loadb(kb + KBB);
            bf16x8 af[4], bf[2];
#pragma unroll
            for (int a = 0; a < 4; ++a)
                af[a] = *reinterpret_cast<const bf16x8 *>(Ab + (wr + a * 16 + (lane & 15)) * RS + 8 * (lane >> 4));
#pragma unroll
            for (int b = 0; b < 2; ++b)
                bf[b] = *reinterpret_cast<const bf16x8 *>(Bb + (wc + b * 16 + (lane & 15)) * RS + 8 * (lane >> 4));
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = mfma_bf16(af[a], bf[b], acc[a][b]);
            __syncthreads();
        }
    } else {
    T ra[KB / 4], rb[KB / 4];
    auto load = [&](int kb) {
#pragma unroll
        for (int e = 0; e < KB / 4; ++e) {
            const int64_t k = min(kb + lk + 4 * e, tk.k1 - 1);
            ra[e] = pa[k * m];
            rb[e] = pb[k * m];
        }
    };
    load(tk.k0);
    for (int kb = tk.k0; kb < tk.k1; kb += KB) {
#pragma unroll
        for (int e = 0; e < KB / 4; ++e) {
            const bool kin = kb + lk + 4 * e < tk.k1;
            As[lk + 4 * e][lr] = (kin && row_ok) ? ra[e] : T(0);
            Bs[lk + 4 * e][lr] = (kin && col_ok) ? rb[e] : T(0);
        }
        __syncthreads();
        if (kb + KB < tk.k1) load(kb + KB);
#pragma unroll
        for (int kk = 0; kk < KB; kk += 4) {
            T af[4], bf[2];
#pragma unroll
            for (int a = 0; a < 4; ++a) af[a] = As[kk + (lane >> 4)][wr + a * 16 + (lane & 15)];
#pragma unroll
            for (int b = 0; b < 2; ++b) bf[b] = Bs[kk + (lane >> 4)][wc + b * 16 + (lane & 15)];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[a][b] = Mfma<T>::run(af[a], bf[b], acc[a][b]);
        }
        __syncthreads();
    }
    }
    // epilogue: 4 passes of 32 columns staged as Cs[32][128 + 1]; in pass p
    // the two waves with wc = 32 p stage their columns, then thread (row r,
    // quarter cq) adds 8 of them
    static_assert(32 * (TM + 1) <= kSmem, "the epilogue's staging fits");
    T(*Cs)[TM + 1] = reinterpret_cast<T(*)[TM + 1]>(smem);
    const int r = tid & 127, cq = tid >> 7;
    const int64_t gi = tk.i0 + r;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass) {
        int32_t rv[CPT];
        T old[CPT];
#pragma unroll
        for (int cc = 0; cc < CPT; ++cc) {
            const int c = 32 * pass + cq * CPT + cc;
            const int64_t gj = min(tk.j0 + c, tk.jmax - 1);
            if constexpr (TRAIL) {
                old[cc] = P[gj * m + min<int64_t>(gi, m - 1)];
                rv[cc] = 0;
            } else {
                rv[cc] = rel[cr[c] + max(min<int64_t>(gi, m - 1), gj)];
                old[cc] = T(0);
            }
        }
        if (wc == 32 * pass)
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        Cs[b * 16 + (lane & 15)][wr + a * 16 + Mfma<T>::row(lane, v)] = acc[a][b][v];
        __syncthreads();
        if (gi < m) {
#pragma unroll
            for (int cc = 0; cc < CPT; ++cc) {
                const int c = 32 * pass + cq * CPT + cc;
                const int64_t gj = tk.j0 + c;
                if (gj >= tk.jmax || gj > gi) continue;
                if constexpr (TRAIL)
                    P[gj * m + gi] = old[cc] - Cs[c & 31][r];
                else
                    atomicAdd(&Lx[cb[c] + rv[cc]], -Cs[c & 31][r]);
            }
        }
        __syncthreads();
    }
    (void)NT;
}

// ---------------------------------------------------------------------------
// Triangular solves on permuted work vectors (n x nrhs, column-major,
// leading dimension n), one launch per level of the block tree.
// Forward, block q (rows g0.., width nb), tasks = chunks of rows below it:
//   x_q = Linv_q y_q;  the first task stores x_q in X;  every task does
//   Y[rows[r]] -= sum_k P[r][c0+k] x_q[k] for its rows (atomic).
// Backward: each task adds sum_r P[r][c0+k] X[rows[r]] over its rows into
//   Acc; the last task of the block (counter) forms t = X_q - Acc_q and
//   stores x_q = Linv_q^T t.  Rows below belong to ancestors, whose x is
//   final when the block's level runs.
// ---------------------------------------------------------------------------
// What a solve starts with, in one launch: the permuted right-hand sides in Y,
// Acc set (unset pattern or zero), the counters of the persistent sweeps
// (dep <- the forward counts, cnt <- 0, queues <- 0).  The error word is the
// factor's, cleared only by a factorization, so a wait that gave up stays
// reported.
template <typename T>
__global__ void k_solve_init(const int32_t *perm, int64_t n, int nrhs, const double *B, int64_t ldb, T *Y, T *Acc,
                             int persist, const int32_t *fdep, int64_t nblocks, SolveSync sy) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n * nrhs) {
        // (32-bit division where it reaches: the 64-bit one is the most of this kernel)
        const int64_t k = n * nrhs <= UINT_MAX ? (uint32_t)i / (uint32_t)nrhs : i / nrhs;
        const int64_t r = i - k * nrhs;
        Y[i] = (T)B[perm[k] + r * ldb];
        Acc[i] = persist ? __builtin_bit_cast(T, Unset<T>::bits) : T(0);
    }
    if (i < nblocks) {
        sy.dep[i] = fdep[i];
        sy.cnt[i] = 0;
    }
    if (i < 2) sy.queue[i] = 0;
}

template <typename T>
__global__ void k_perm_out(const int32_t *perm, int64_t n, int nrhs, const T *W, double *B, int64_t ldb) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * nrhs) return;
    const int64_t k = n * nrhs <= UINT_MAX ? (uint32_t)i / (uint32_t)nrhs : i / nrhs;
    const int64_t r = i - k * nrhs;
    B[perm[k] + r * ldb] = (double)W[i];
}

constexpr int kMaxRhs = 16;

// Persistent sweeps: instead of one launch per block-tree level, a grid of
// resident workgroups takes tasks from an atomic counter in an order where
// every task's dependencies come first, so a task waits only on tasks that
// running workgroups already hold and the sweep cannot deadlock.  Forward:
// a block's tasks wait until every task updating its rows has counted down
// dep[block]; backward: a task waits for the x of its rows (bounded waits,
// wait_value, wait_handed and fetch_rows).

// Data handed between workgroups of one persistent sweep moves through
// device-scope atomics (loads after a wait, stores before a flag is raised),
// and a workgroup raises a flag after waiting for its own memory operations;
// no cache-wide fences, whose writeback and invalidation cost more than the
// data.
template <typename T>
__device__ __forceinline__ T shared_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void shared_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void release_own() { __builtin_amdgcn_s_waitcnt(0); }
__device__ __forceinline__ void acquire_after_wait() {}

// Bounded wait for a handed-over value (0 once a wait gave up).
template <typename T>
__device__ __forceinline__ T wait_handed(const T *p, int32_t *err, int32_t spin) {
    for (int it = 0; it < spin; ++it) {
        const T v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!is_unset(v)) return v;
        if ((it & 255) == 255 && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return T(0);
        __builtin_amdgcn_s_sleep(1);
    }
    flag_device_error(err);
    return T(0);
}

// Next task of a workgroup: the persistent grid takes it from the work
// counter (through `order` when given), the level-launch grid takes its
// own index once.  Returns -1 when there is none.
template <bool PERSIST>
__device__ __forceinline__ int64_t next_task(int pass, const int32_t *order, int32_t *queue, int64_t ntasks,
                                             int32_t *slot) {
    if (!PERSIST) return pass == 0 ? (int64_t)blockIdx.x : -1;
    if (threadIdx.x == 0) *slot = atomicAdd(queue, 1);
    __syncthreads();
    const int64_t i = *slot;
    if (i >= ntasks) return -1;
    return order ? order[i] : i;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
    v = pair_add<kRor8>(pair_add<kRor4>(pair_add<kXor2>(pair_add<kXor1>(v))));
    return half_add<32>(half_add<16>(v));
}

// ---------------------------------------------------------------------------
// One-wave solves of tiny supernodes (w <= kTinyW, m <= kTinyM), four per
// workgroup, for the wide bottom levels where nearly every supernode is
// tiny: a supernode costs one wave instead of a workgroup sized for a
// 64-column block.  Right-hand sides are interleaved by row (entry (k, q) at
// k * nrhs + q), so the values of one row sit together.
// Forward: x = Linv y for the w diagonal rows, stored in X; then each row
// i >= w below takes
//   Y[rows[i]] -= sum_c L[i][c] x_c      (atomic, as in the block sweep).
// One right-hand side: lane i holds row position i, y_c and x_c are
// broadcast from lane c.  Several: x goes through LDS and the update is the
// product (rows x w)(w x 16) on 16x16x4 MFMA (four row tiles, two steps of
// the contraction), so the 16 lanes of one output row write its 16
// consecutive values.
// Bound by latency (a trip for the task, one for its rows and panel, one for
// the values of the rows) and, in the bottom levels of a batch, by the
// scattered rows.  Everything a wave reads is asked for ahead of its first
// use, the inverse (at most 64 entries) by one load a lane and through LDS.
// wg: the workgroup's place among those of the level's tiny tasks; lds:
// kTinyLds values for each of its waves (several right-hand sides).
// ---------------------------------------------------------------------------
static_assert(kTinyW * kTinyW <= 64);
constexpr int kTinyLds = 2 * kTinyW * (kMaxRhs + 1) + kTinyW * kTinyW;

template <typename T, int NR>
__device__ __forceinline__ void solve_tiny_fwd_body(int64_t wg, const SmallTask *tasks, int64_t ntasks,
                                                    const int32_t *rows, const T *Lx, const T *Linv, T *Y, T *X,
                                                    int nrhs, T *lds) {
    constexpr int WT = kTinyW;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t ti = wg * 4 + wv;
    if constexpr (NR == 1) {
        if (ti >= ntasks) return;  // the whole wave
        const SmallTask tk = tasks[ti];
        const int m = tk.m, w = tk.w;
        const T *P = Lx + tk.loff;
        const T *Q = Linv + tk.ioff;
        const int rc = min(lane, m - 1), dc = min(lane, w - 1);
        T l[WT], vi[WT];
#pragma unroll
        for (int c = 0; c < WT; ++c) l[c] = P[(int64_t)min(c, w - 1) * m + rc];
#pragma unroll
        for (int c = 0; c < WT; ++c) vi[c] = Q[dc + min(c, w - 1) * w];  // (L^{-1})[dc][c]
        const int64_t g = rows[tk.roff + rc];
        const T y = Y[tk.g0 + dc];
        T x = T(0), acc = T(0);
#pragma unroll
        for (int c = 0; c < WT; ++c)
            if (c < w) x += (c <= lane ? vi[c] : T(0)) * lane_read(y, c);
#pragma unroll
        for (int c = 0; c < WT; ++c)
            if (c < w) acc += l[c] * lane_read(x, c);
        if (lane < w) X[tk.g0 + lane] = x;
        else if (lane < m) atomicAdd(&Y[g], -acc);
    } else {
        using acc_t = typename Mfma<T>::acc;
        T(*ys)[kMaxRhs + 1] = (T(*)[kMaxRhs + 1])(lds + wv * kTinyLds);
        T(*xs)[kMaxRhs + 1] = ys + WT;
        T *qs = lds + wv * kTinyLds + 2 * WT * (kMaxRhs + 1);
        const bool active = ti < ntasks;
        const SmallTask tk = tasks[active ? ti : ntasks - 1];  // idle waves mirror a task, store nothing
        const int m = tk.m, w = tk.w;
        const T *P = Lx + tk.loff;
        const T *Q = Linv + tk.ioff;
        const int kq = lane & 15, kr = lane >> 4;
        const int64_t g = rows[tk.roff + min(lane, m - 1)];  // lane = row position
        // A operands: row 16 tt + kq of the panel, columns 4 s + kr
        T a[4][2];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)
                a[tt][s2] = P[(int64_t)min(4 * s2 + kr, w - 1) * m + min(16 * tt + kq, m - 1)];
        // y of the diagonal rows, two (c, q) slots per lane: c = kr + 4 h
        const T ql = Q[min(lane, w * w - 1)];
        T yv[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) yv[h] = Y[(tk.g0 + min(kr + 4 * h, w - 1)) * nrhs + min(kq, nrhs - 1)];
#pragma unroll
        for (int h = 0; h < 2; ++h) ys[kr + 4 * h][kq] = (kr + 4 * h < w && kq < nrhs) ? yv[h] : T(0);
        qs[lane] = ql;
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = kr + 4 * h;
            T xv = T(0);
#pragma unroll
            for (int j = 0; j < WT; ++j) {
                const T vq = qs[min(c, w - 1) + min(j, w - 1) * w];  // (L^{-1})[c][j]
                xv += (j <= c && c < w) ? vq * ys[j][kq] : T(0);
            }
            xs[c][kq] = xv;
            if (active && c < w && kq < nrhs) X[(tk.g0 + c) * nrhs + kq] = xv;
        }
        wave_lds_sync();
        // B operands: x[4 s + kr][kq] (zero beyond w)
        const T b0 = xs[kr][kq], b1 = xs[4 + kr][kq];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            if (16 * tt >= m) break;  // uniform
            acc_t acc = {0, 0, 0, 0};
            acc = Mfma<T>::run(4 * 0 + kr < w ? a[tt][0] : T(0), b0, acc);
            acc = Mfma<T>::run(4 + kr < w ? a[tt][1] : T(0), b1, acc);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = 16 * tt + Mfma<T>::row(lane, v);
                const int64_t gr = __shfl(g, min(r, 63));
                if (active && r >= w && r < m && kq < nrhs) atomicAdd(&Y[gr * nrhs + kq], -acc[v]);
            }
        }
    }
}

// Backward: t_c = X[g0 + c] - sum_{i >= w} L[i][c] X[rows[i]] for the w
// columns c (the rows below are ancestors, final already), then
// x = Linv^T t.  One right-hand side: the sums are wave reductions.
// Several: the sums form the product (L_below^T)(X_rows), w x 16 with up to
// 64 rows of contraction, on 16x16x4 MFMA (A: lane l brings L[k][l%16],
// B: X[rows[k]][l%16], k = 4 s + l/16); t goes through LDS for the final
// small product with the inverse.
template <typename T, int NR>
__device__ __forceinline__ void solve_tiny_bwd_body(int64_t wg, const SmallTask *tasks, int64_t ntasks,
                                                    const int32_t *rows, const T *Lx, const T *Linv, T *X, int nrhs,
                                                    T *lds) {
    constexpr int WT = kTinyW;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t tr = wg * 4 + wv;
    const bool active = tr < ntasks;
    const SmallTask tk = tasks[active ? tr : ntasks - 1];  // idle waves mirror a task, store nothing
    const int m = tk.m, w = tk.w;
    const T *P = Lx + tk.loff;
    const T *Q = Linv + tk.ioff;
    const int rc = min(lane, m - 1), dc = min(lane, w - 1);
    const int64_t g = rows[tk.roff + rc];
    if constexpr (NR == 1) {
        T l[WT], vt[WT];
#pragma unroll
        for (int c = 0; c < WT; ++c) l[c] = P[(int64_t)min(c, w - 1) * m + rc];
#pragma unroll
        for (int i = 0; i < WT; ++i) vt[i] = Q[min(i, w - 1) + dc * w];  // (L^{-1})[i][dc]
        const T xr = (lane >= w && lane < m) ? X[g] : T(0);
        T t = X[tk.g0 + dc];
#pragma unroll
        for (int c = 0; c < WT; ++c)
            if (c < w) {
                const T sc = wave_sum(l[c] * xr);
                if (lane == c) t -= sc;
            }
        T xv = T(0);
#pragma unroll
        for (int i = 0; i < WT; ++i)
            if (i < w) xv += (i >= lane ? vt[i] : T(0)) * lane_read(t, i);
        if (active && lane < w) X[tk.g0 + lane] = xv;
    } else {
        using acc_t = typename Mfma<T>::acc;
        const int kq = lane & 15, kr = lane >> 4;
        T(*ts)[kMaxRhs + 1] = (T(*)[kMaxRhs + 1])(lds + wv * kTinyLds);
        T *qs = lds + wv * kTinyLds + WT * (kMaxRhs + 1);
        T a[16], b[16], xo[4];
        const T ql = Q[min(lane, w * w - 1)];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            xo[v] = X[(tk.g0 + min(Mfma<T>::row(lane, v), w - 1)) * nrhs + min(kq, nrhs - 1)];
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int k = 4 * s + kr, kc = min(k, m - 1);
            const int64_t gk = __shfl(g, kc);
            const bool row_ok = k >= w && k < m;
            const T av = P[(int64_t)min(kq, w - 1) * m + kc];
            const T bv = X[gk * nrhs + min(kq, nrhs - 1)];
            a[s] = (row_ok && kq < w) ? av : T(0);
            b[s] = (row_ok && kq < nrhs) ? bv : T(0);
        }
        acc_t acc = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 16; ++s) acc = Mfma<T>::run(a[s], b[s], acc);
        // element v of this lane: row c of (L_below^T X_rows), column kq
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int c = Mfma<T>::row(lane, v);
            if (c < WT) ts[c][kq] = (c < w && kq < nrhs) ? xo[v] - acc[v] : T(0);
        }
        qs[lane] = ql;
        wave_lds_sync();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = kr + 4 * h;
            T xv = T(0);
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                const T vq = qs[min(i, w - 1) + min(c, w - 1) * w];  // (L^{-1})[i][c]
                xv += (i >= c && i < w) ? vq * ts[i][kq] : T(0);
            }
            if (active && c < w && kq < nrhs) X[(tk.g0 + c) * nrhs + kq] = xv;
        }
    }
}

// Levels whose tiny supernodes are launched by themselves
template <typename T, int NR>
__global__ __launch_bounds__(256) void k_solve_tiny_fwd(const SmallTask *tasks, int64_t ntasks, const int32_t *rows,
                                                        const T *Lx, const T *Linv, T *Y, T *X, int nrhs) {
    __shared__ T lds[NR > 1 ? 4 * kTinyLds : 1];
    solve_tiny_fwd_body<T, NR>(blockIdx.x, tasks, ntasks, rows, Lx, Linv, Y, X, nrhs, lds);
}
template <typename T, int NR>
__global__ __launch_bounds__(256) void k_solve_tiny_bwd(const SmallTask *tasks, int64_t ntasks, const int32_t *rows,
                                                        const T *Lx, const T *Linv, T *X, int nrhs) {
    __shared__ T lds[NR > 1 ? 4 * kTinyLds : 1];
    solve_tiny_bwd_body<T, NR>(blockIdx.x, tasks, ntasks, rows, Lx, Linv, X, nrhs, lds);
}

// Forward, one task = rows r0..r1-1 below block q:
//   x_q = Linv_q y_q (every task; the first task stores it in X), then
//   Y[rows[r]] -= sum_k L[r][c0+k] x_q[k] (atomic).
// One right-hand side: thread = row for the update; for x_q four threads
// share a row of Linv (16 columns each, held in registers) and add up by
// lane shuffles.  Everything a task reads besides y (its panel rows, its
// part of Linv, its target blocks) is loaded before it waits.
// A persistent task's rows fall in at most 256 blocks (one per row), so
// each thread holds at most one target block to count down.
// Persistent sweep, inside a supernode: the first task of block q - 1 puts
// its sums for q's rows into H (as values, not subtracted from Y) instead
// of counting q down, and q's tasks take y_q = Y - H once those values are
// there (hand bits).
template <typename T, bool PERSIST>
__global__ __launch_bounds__(256) void k_solve_fwd(const SolveTask *tasks, int64_t ntasks, const int32_t *rows,
                                                   const T *Lx, const T *Linv, T *Y, T *X, T *H, int64_t n,
                                                   const int64_t *tgt_ptr, const int32_t *tgt, SolveSync sy,
                                                   const SmallTask *tiny, int64_t ntiny) {
    if constexpr (!PERSIST)
        if (blockIdx.x >= ntasks)
            return solve_tiny_fwd_body<T, 1>(blockIdx.x - ntasks, tiny, ntiny, rows, Lx, Linv, Y, X, 1, nullptr);
    constexpr int NB = kNB, QW = NB / 4;
    __shared__ T yq[NB];
    __shared__ T xq[NB];
    __shared__ int32_t slot;
    const int tid = threadIdx.x;
    const int vi = tid >> 2, vp = tid & 3;  // x: row vi of Linv, columns QW vp .. QW vp + QW - 1
    for (int pass = 0;; ++pass) {
        const int64_t t = next_task<PERSIST>(pass, nullptr, sy.queue, ntasks, &slot);
        if (t < 0) return;
        const SolveTask tk = tasks[t];
        const int nb = tk.nb;
        const int64_t m = tk.m;
        const T *P = Lx + tk.loff;
        const T *Q = Linv + tk.ioff;
        const int64_t r = tk.r0 + tid;
        const int64_t rc = min(r, m - 1);
        T qv[QW], pv[NB];
        const int qi = min(vi, nb - 1);
#pragma unroll
        for (int k = 0; k < QW; ++k) qv[k] = Q[qi + (int64_t)min(QW * vp + k, nb - 1) * nb];
        const int64_t gr = rows[tk.roff + rc];
#pragma unroll
        for (int k = 0; k < NB; ++k) pv[k] = P[(int64_t)(tk.c0 + min(k, nb - 1)) * m + rc];
        int32_t my_tgt = -1;
        if (PERSIST) {
            const int64_t tb = tgt_ptr[t], te = tgt_ptr[t + 1];
            if (tid < te - tb) my_tgt = tgt[tb + tid];
            if (tid == 0) wait_value(&sy.dep[tk.blk], 0, sy.err, sy.spin);
            __syncthreads();
            acquire_after_wait();
        }
        if (tid < NB) {
            const T *py = &Y[tk.g0 + min(tid, nb - 1)];
            T yv = PERSIST ? shared_load(py) : *py;
            if (PERSIST && (tk.hand & kHandIn) && tid < nb) yv -= wait_handed(&H[tk.g0 + tid], sy.err, sy.spin);
            yq[tid] = tid < nb ? yv : T(0);
        }
        __syncthreads();
        {
            T a0 = T(0), a1 = T(0);
#pragma unroll
            for (int k = 0; k < QW; k += 2) {
                const int c = QW * vp + k;
                a0 += (c <= vi ? qv[k] : T(0)) * yq[c];
                a1 += (c + 1 <= vi ? qv[k + 1] : T(0)) * yq[c + 1];
            }
            T a = a0 + a1;
            a = pair_add<kXor2>(pair_add<kXor1>(a));
            if (vp == 0) xq[vi] = vi < nb ? a : T(0);
        }
        __syncthreads();
        if (r < tk.r1) {
            // entries of x_q beyond nb are zero, so clamped columns add nothing
            T a0 = T(0), a1 = T(0), a2 = T(0), a3 = T(0);
#pragma unroll
            for (int k = 0; k < NB; k += 4) {
                a0 += pv[k] * xq[k];
                a1 += pv[k + 1] * xq[k + 1];
                a2 += pv[k + 2] * xq[k + 2];
                a3 += pv[k + 3] * xq[k + 3];
            }
            const T v = (a0 + a1) + (a2 + a3);
            if (PERSIST && (tk.hand & kHandOut) && tid < (tk.hand >> 8)) shared_store(&H[gr], v);
            else atomicAdd(&Y[gr], -v);
        }
        if (PERSIST) {
            release_own();
            __syncthreads();
            if (my_tgt >= 0 && !((tk.hand & kHandOut) && my_tgt == tk.blk + 1)) atomicSub(&sy.dep[my_tgt], 1);
        }
        // (off the chain: after what others wait for)
        if (tk.first && tid < nb) X[tk.g0 + tid] = xq[tid];
    }
}

// Several right-hand sides (up to kMaxRhs): the update of the task's rows
// is the product (rows x 64) (64 x 16) on 16x16x4 MFMA blocks, wave w
// taking the 16-row tiles w, w + 4, w + 8 and w + 12 in that order (so the
// first 64 rows, handed over to the next block in the persistent sweep, are
// done first, by all four waves); the A operand comes straight from the
// panel, the B operand (x_q) from LDS.  Two workgroups per CU (the FP64
// form then keeps 256 registers with a spill of two): the persistent sweep
// runs twice as many resident workgroups, so the tasks waiting on a block
// leave room for the ones on the chain.
// Bound by latency from block to block.  A thread's handed-over values polled
// together instead of one after the other, and x stored after what other
// tasks wait for, took the persistent sweep of a 50^3 grid (FP32, 8 right-hand
// sides) from 382 to 312 us, of the 30x29x27 elasticity operator (FP64, 16)
// from 441 to 376.
template <typename T, bool PERSIST>
__global__ __launch_bounds__(256, 2) void k_solve_fwd_multi(const SolveTask *tasks, int64_t ntasks,
                                                         const int32_t *rows, const T *Lx, const T *Linv, T *Y,
                                                         T *X, T *H, int64_t n, int nrhs, const int64_t *tgt_ptr,
                                                         const int32_t *tgt, SolveSync sy,
                                                         const SmallTask *tiny, int64_t ntiny) {
    constexpr int NB = kNB, NR = kMaxRhs, YPT = NB * NR / 256, KS = NB / 4;
    using acc_t = typename Mfma<T>::acc;
    __shared__ T yx[2][NB][NR + 1];
    auto &yq = yx[0], &xq = yx[1];
    if constexpr (!PERSIST) {
        static_assert(4 * kTinyLds <= 2 * NB * (NR + 1));
        if (blockIdx.x >= ntasks)
            return solve_tiny_fwd_body<T, NR>(blockIdx.x - ntasks, tiny, ntiny, rows, Lx, Linv, Y, X, nrhs,
                                              &yx[0][0][0]);
    }
    __shared__ int64_t grs[256];
    __shared__ int32_t slot;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int pass = 0;; ++pass) {
        const int64_t t = next_task<PERSIST>(pass, nullptr, sy.queue, ntasks, &slot);
        if (t < 0) return;
        const SolveTask tk = tasks[t];
        const int nb = tk.nb;
        const int64_t m = tk.m;
        const T *P = Lx + tk.loff;
        const T *Q = Linv + tk.ioff;
        // x = Linv y on MFMA as well: wave w the rows 16 w .. 16 w + 15 of x,
        // lane bringing Linv[16 w + lane % 16][4 s + lane / 16]
        // Level launches: K-steps of 4 columns that reach the block's nb
        // columns, and the row tiles of 16 that reach the task's rows; the
        // clamped operands beyond them only ever meet zeros, so the narrow
        // blocks and short tasks of the bottom levels skip their loads and
        // products (same for every lane of a wave).  The persistent sweep,
        // of mostly full blocks, keeps the unconditional form.
        const int ksn = (nb + 3) >> 2;
        const int64_t nrows = tk.r1 - tk.r0;
        T qv[KS], yv[YPT], av[4][KS];
        if constexpr (PERSIST) {
#pragma unroll
            for (int s2 = 0; s2 < KS; ++s2) {
                const int i = 16 * wave + (lane & 15), c = 4 * s2 + (lane >> 4);
                const T v = Q[min(i, nb - 1) + (int64_t)min(c, nb - 1) * nb];
                qv[s2] = (c <= i && i < nb) ? v : T(0);
            }
        } else {
#pragma unroll
            for (int s2 = 0; s2 < KS; ++s2) {
                const int i = 16 * wave + (lane & 15), c = 4 * s2 + (lane >> 4);
                const T v = s2 < ksn ? Q[min(i, nb - 1) + (int64_t)min(c, nb - 1) * nb] : T(0);
                qv[s2] = (c <= i && i < nb) ? v : T(0);
            }
        }
        grs[tid] = rows[tk.roff + min<int64_t>(tk.r0 + tid, m - 1)];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const int64_t row = min<int64_t>(tk.r0 + 16 * (4 * tt + wave) + (lane & 15), m - 1);
            if constexpr (PERSIST) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    av[tt][ks] = P[(int64_t)(tk.c0 + min(4 * ks + (lane >> 4), nb - 1)) * m + row];
            } else {
                const bool live = 16 * (4 * tt + wave) < nrows;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    av[tt][ks] = live && ks < ksn
                                     ? P[(int64_t)(tk.c0 + min(4 * ks + (lane >> 4), nb - 1)) * m + row]
                                     : T(0);
            }
        }
        int32_t my_tgt = -1;
        if (PERSIST) {
            // at most one target block per row of the task
            const int64_t tb = tgt_ptr[t], te = tgt_ptr[t + 1];
            if (tid < te - tb) my_tgt = tgt[tb + tid];
            if (tid == 0) wait_value(&sy.dep[tk.blk], 0, sy.err, sy.spin);
            __syncthreads();
            acquire_after_wait();
        }
#pragma unroll
        for (int u = 0; u < YPT; ++u) {
            const int e = tid + 256 * u, i = e / NR, q = e % NR;
            const T *py = &Y[(tk.g0 + min(i, nb - 1)) * nrhs + min(q, nrhs - 1)];
            yv[u] = PERSIST ? shared_load(py) : *py;
        }
        if (PERSIST && (tk.hand & kHandIn)) {
            // the previous block's sums for these rows, a thread's values
            // polled together (padding repeats a real entry)
            T hv[YPT];
            bool ready = false;
            for (int it = 0; it < sy.spin; ++it) {
                bool unset = false;
#pragma unroll
                for (int u = 0; u < YPT; ++u) {
                    const int e = tid + 256 * u, i = e / NR, q = e % NR;
                    hv[u] = shared_load(&H[(tk.g0 + min(i, nb - 1)) * nrhs + min(q, nrhs - 1)]);
                }
#pragma unroll
                for (int u = 0; u < YPT; ++u) unset = unset || is_unset(hv[u]);
                if (!__any(unset)) {
                    ready = true;
                    break;
                }
                if ((it & 255) == 255 && __hip_atomic_load(sy.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    break;
                __builtin_amdgcn_s_sleep(1);
            }
            if (!ready && lane == 0) flag_device_error(sy.err);
#pragma unroll
            for (int u = 0; u < YPT; ++u) yv[u] -= ready ? hv[u] : T(0);
        }
#pragma unroll
        for (int u = 0; u < YPT; ++u) {
            const int e = tid + 256 * u, i = e / NR, q = e % NR;
            yq[i][q] = (i < nb && q < nrhs) ? yv[u] : T(0);
        }
        __syncthreads();
        {
            acc_t xa = {0, 0, 0, 0};
#pragma unroll
            for (int s2 = 0; s2 < KS; ++s2)
                if (PERSIST || s2 < ksn) xa = Mfma<T>::run(qv[s2], yq[4 * s2 + (lane >> 4)][lane & 15], xa);
#pragma unroll
            for (int v = 0; v < 4; ++v) xq[16 * wave + Mfma<T>::row(lane, v)][lane & 15] = xa[v];
        }
        __syncthreads();
        // rows of x_q beyond nb are zero, so the clamped columns contribute nothing
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            if constexpr (!PERSIST) {
                if (16 * (4 * tt + wave) >= nrows) continue;  // no row of this tile is the task's
            }
            acc_t acc = {0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                if (PERSIST || ks < ksn) acc = Mfma<T>::run(av[tt][ks], xq[4 * ks + (lane >> 4)][lane & 15], acc);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int rr = 16 * (4 * tt + wave) + Mfma<T>::row(lane, v), q = lane & 15;
                if (tk.r0 + rr < tk.r1 && q < nrhs) {
                    if (PERSIST && (tk.hand & kHandOut) && rr < (tk.hand >> 8))
                        shared_store(&H[grs[rr] * nrhs + q], acc[v]);
                    else
                        atomicAdd(&Y[grs[rr] * nrhs + q], -acc[v]);
                }
            }
        }
        if (PERSIST) {
            release_own();
            __syncthreads();
            if (my_tgt >= 0 && !((tk.hand & kHandOut) && my_tgt == tk.blk + 1)) atomicSub(&sy.dep[my_tgt], 1);
        }
        if (tk.first)
            for (int e = tid; e < nb * nrhs; e += 256) {
                const int i = e / nrhs, q = e % nrhs;
                X[(tk.g0 + i) * nrhs + q] = xq[i][q];
            }
        __syncthreads();
    }
}

// Four consecutive entries from an address aligned to one entry; they may
// reach up to three entries past what the caller uses (the panel and the
// inverse stores are allocated with that slack), and the caller masks them.
template <typename T>
struct Quad {
    T v[4];
};
template <typename T>
__device__ __forceinline__ Quad<T> load_quad(const T *p) {
    Quad<T> q;
    __builtin_memcpy(&q, p, sizeof(q));
    return q;
}

// Persistent sweep: x of this lane's rows of the row tiles u0 .. u0 + NU - 1 of
// a task (row 64 u + row0 + j), all loads together, until every one has been
// put into XB (bounded; 0 once a wait gave up).  Rows beyond the task give 0.
template <typename T, int NU>
__device__ __forceinline__ void fetch_rows(const T *XB, const int32_t *grs, int row0, int u0, int nrows, int nrhs,
                                           int64_t q, const SolveSync &sy, T *xv) {
    bool ready = false;
    for (int it = 0; it < sy.spin; ++it) {
        bool unset = false;
#pragma unroll
        for (int e = 0; e < 4 * NU; ++e)
            xv[e] = shared_load(&XB[(int64_t)grs[64 * (u0 + e / 4) + row0 + e % 4] * nrhs + q]);
#pragma unroll
        for (int e = 0; e < 4 * NU; ++e)
            unset = unset || (64 * (u0 + e / 4) + row0 + e % 4 < nrows && is_unset(xv[e]));
        if (!__any(unset)) {
            ready = true;
            break;
        }
        if ((it & 255) == 255 && __hip_atomic_load(sy.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
        __builtin_amdgcn_s_sleep(1);
    }
    if (!ready && (threadIdx.x & 63) == 0) flag_device_error(sy.err);
#pragma unroll
    for (int e = 0; e < 4 * NU; ++e)
        xv[e] = ready && 64 * (u0 + e / 4) + row0 + e % 4 < nrows ? xv[e] : T(0);
}

// Backward, one task = rows r0..r1-1 below block q:
//   sums S_c = sum_r L[r][c0+c] x[rows[r]],  t = X_q - S,  x_q = Linv_q^T t.
// A block with one task finishes itself; a block split over several tasks
// adds its sums into Acc.  In a level launch the last task to arrive
// (sy.cnt) finishes the block.  In the persistent sweep the block's first
// task does: it holds the rows nearest the block, whose x are final last,
// and it is queued after the block's other tasks, so it collects their sums
// (waiting on sy.cnt) before its own rows are ready, which keeps that
// exchange off the chain of blocks.  Rows below the block belong to
// ancestors, whose x is final before the block's tasks read it: in a level
// launch by the order of the levels; in the persistent sweep every finished
// x goes into XB, set to a pattern no result takes, and the readers poll the
// values themselves.  The rows come from the block's ancestors in order, and
// the x of a nearer ancestor needed those of all the farther ones, so a task
// polls one value of its nearest ancestor's rows and then loads them all;
// the first task of block q - 1 treats q's rows, which come first, apart:
// everything else is done before they arrive.
//
// Persistent sweep, one right-hand side.  Wave w takes the rows 64 u + 16 w ..
// + 15 of the task (u = 0 .. 3) for all 64 columns, lane l four consecutive
// rows 4 (l / 16) .. + 3 of the columns 16 ct + l % 16 with wide loads (16
// columns x 128 bytes an instruction) and x of its rows straight from XB;
// the four lane groups add up by shuffles, the waves through LDS.  Bound by
// latency from block to block.  With a done flag per block (raised after the
// stores had completed, then polled, then x loaded) and a thread per column
// (64 columns x 8 bytes an instruction) the sweep of the 60^3 grid took 513
// us and that of the 32^2 grid 42, this form 444 and 30.  (FP64 at two
// workgroups a CU spills 13 registers: 495 us.)
template <typename T>
__global__ __launch_bounds__(256) void k_solve_bwd(const SolveTask *tasks, int64_t ntasks, const int32_t *order,
                                                   const int32_t *rows, const T *Lx, const T *Linv, T *X, T *Acc,
                                                   T *XB, SolveSync sy) {
    constexpr int NB = kNB, QW = 16, NT = NB / 16;
    __shared__ T Sm[4][NB];    // sums of the 4 waves
    __shared__ T tq[NB];
    __shared__ int32_t grs[256];
    __shared__ int32_t slot;
    const int tid = threadIdx.x, lane = tid & 63, kq = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), row0 = 16 * wave + 4 * kg;
    // x_q = Linv^T t, with (Linv^T)[c][i] = Linv[i][c] nonzero for i >= c:
    // four threads per output c, 16 rows i each, that part of Linv held in
    // registers.
    const int oc = tid >> 2;
    auto inv_row = [&](int s2) { return QW * (tid & 3) + s2; };
    for (int pass = 0;; ++pass) {
        const int64_t t = next_task<true>(pass, order, sy.queue + 1, ntasks, &slot);
        if (t < 0) return;
        const SolveTask tk = tasks[t];
        const int nb = tk.nb, nrows = tk.r1 - tk.r0;
        const int64_t m = tk.m;
        const T *P = Lx + tk.loff;
        const T *Q = Linv + tk.ioff;
        grs[tid] = rows[tk.roff + min<int64_t>(tk.r0 + tid, m - 1)];
        Quad<T> av[4][NT];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t r = min<int64_t>(tk.r0 + 64 * u + row0, m - 1);
#pragma unroll
            for (int ct = 0; ct < NT; ++ct)
                av[u][ct] = load_quad(P + (int64_t)(tk.c0 + min(16 * ct + kq, nb - 1)) * m + r);
        }
        T qv[QW];
#pragma unroll
        for (int s2 = 0; s2 < QW; ++s2) {
            const int i = inv_row(s2);
            const T v = Q[min(i, nb - 1) + (int64_t)min(oc, nb - 1) * nb];
            qv[s2] = (i >= oc && i < nb && oc < nb) ? v : T(0);
        }
        // the block's own forward values: final since the forward sweep, and
        // overwritten only by the task that finishes this block
        T xb = T(0);
        if (tk.first) xb = X[tk.g0 + min(tid, nb - 1)];
        if (tk.first && tk.ntasks > 1) {
            // every other task of the block was dequeued before this one
            if (tid == 0) {
                wait_value(&sy.cnt[tk.blk], tk.ntasks - 1, sy.err, sy.spin);
                sy.cnt[tk.blk] = 0;
            }
            __syncthreads();
            if (tid < nb)
                xb -= __hip_atomic_exchange(&Acc[tk.g0 + tid], T(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const int nhand = (tk.hand & kHandOut) ? tk.hand >> 8 : 0;  // rows of the next block
        __syncthreads();
        if (nrows < 256) {
            // a ragged task: what the wide loads took beyond its rows
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool in = 64 * u + row0 + j < nrows;
#pragma unroll
                    for (int ct = 0; ct < NT; ++ct) av[u][ct].v[j] = in ? av[u][ct].v[j] : T(0);
                }
        }
        T sum[NT];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) sum[ct] = T(0);
        auto add = [&](int u, const T *xv) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int ct = 0; ct < NT; ++ct) sum[ct] += av[u][ct].v[j] * xv[j];
        };
        if (nhand < nrows) (void)wait_handed(&XB[grs[nhand]], sy.err, sy.spin);
        if (nrows > 64) {
            T xf[12];
            fetch_rows<T, 3>(XB, grs, row0, 1, nrows, 1, 0, sy, xf);
#pragma unroll
            for (int u = 3; u >= 1; --u) add(u, xf + 4 * (u - 1));
        }
        if (nrows > 0) {
            T xn[4];
            fetch_rows<T, 1>(XB, grs, row0, 0, nrows, 1, 0, sy, xn);
            add(0, xn);
        }
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            sum[ct] = half_add<32>(half_add<16>(sum[ct]));
            if (kg == 0) Sm[wave][16 * ct + kq] = sum[ct];
        }
        __syncthreads();
        if (tk.first) {
            if (tid < NB) tq[tid] = tid < nb ? xb - ((Sm[0][tid] + Sm[1][tid]) + (Sm[2][tid] + Sm[3][tid])) : T(0);
            __syncthreads();
            // x_q = Linv^T t
            T a0 = T(0), a1 = T(0);
#pragma unroll
            for (int s2 = 0; s2 < QW; s2 += 2) {
                a0 += qv[s2] * tq[inv_row(s2)];
                a1 += qv[s2 + 1] * tq[inv_row(s2 + 1)];
            }
            T a = a0 + a1;
            a = pair_add<kXor2>(pair_add<kXor1>(a));
            if ((tid & 3) == 0 && oc < nb) {
                shared_store(&XB[tk.g0 + oc], a);
                X[tk.g0 + oc] = a;
            }
        } else {
            if (tid < nb)
                atomicAdd(&Acc[tk.g0 + tid], (Sm[0][tid] + Sm[1][tid]) + (Sm[2][tid] + Sm[3][tid]));
            release_own();
            __syncthreads();
            if (tid == 0) atomicAdd(&sy.cnt[tk.blk], 1);
        }
        __syncthreads();
    }
}

// Backward, several right-hand sides (up to kMaxRhs): the steps of
// k_solve_bwd, with both products on 16x16x4 MFMA blocks.
//   sums: S[c][q] = sum_r L[r][c0+c] X[rows[r]][q].  Wave w takes rows
//     64 u + 16 w .. + 15 of the task (u = 0 .. 3) for all 64 columns; lane
//     l brings four consecutive rows 4 (l / 16) .. + 3 of column l % 16 with
//     one wide load, and the x of the same four rows for right-hand side
//     l % 16 straight from X (the order of k inside a product is free as
//     long as both operands use the same).  The rows handed over by the
//     next block (u = 0) are multiplied last and are spread over all four
//     waves, so the chain from block to block sees a quarter of their
//     products; the panel, the inverse and the other rows' products are
//     done before.
//   x_q = Linv^T t: wave w the outputs 16 w .. 16 w + 15, the inverse and t
//     from LDS.
// Bound by latency: the chain of blocks at the top of the tree, one block
// waiting for the x of the next.  Polling a lane's four values together
// (rather than one right-hand side after the other) and wide panel loads (16
// columns x 128 bytes per instruction rather than 64 columns x 8) took the
// 16-column FP64 solve of the 30x29x27 elasticity operator from 3331 to 1118
// us and the refined FP32 8-column re-solve of a 50^3 grid from 5170 to 3235,
// against the vector-FMA form with x in LDS that this replaced for all counts
// (at 4 right-hand sides, FP64: 48^3 elasticity step 65.7 to 65.1 ms).
// Polling the x values of all rows instead of a done flag per block, and the
// inverse in LDS instead of registers, took the persistent sweep of a 50^3
// grid (FP32, 8) from 324 to 280 us, of the 20^3 elasticity operator (FP32,
// 4) from 186 to 151, of a 200^2 grid (FP64, 8) from 109 to 80.
template <typename T, bool PERSIST>
__global__ __launch_bounds__(256, 2) void k_solve_bwd_multi(const SolveTask *tasks, int64_t ntasks,
                                                            const int32_t *order, const int32_t *rows, const T *Lx,
                                                            const T *Linv, T *X, T *Acc, T *XB, int64_t n, int nrhs,
                                                            SolveSync sy, const SmallTask *tiny, int64_t ntiny) {
    constexpr int NB = kNB, NR = kMaxRhs, NT = NB / 16, EPT = NB * NR / 256;
    using M = Mfma<T>;
    using acc_t = typename M::acc;
    __shared__ T Sm[4][NB][NR + 1];  // each wave's sums
    __shared__ T tq[NB][NR + 1];
    __shared__ T Qs[NB][NB + 1];  // Qs[c][i] = the block inverse's (i, c), zero above its diagonal and beyond nb
    __shared__ int32_t grs[256];
    __shared__ int last;
    __shared__ int32_t slot;
    if constexpr (!PERSIST) {
        static_assert(4 * kTinyLds <= 4 * NB * (NR + 1));
        if (blockIdx.x >= ntasks) {
            const int64_t wg = blockIdx.x - ntasks;
            T *lds = &Sm[0][0][0];
            if (nrhs == 1) solve_tiny_bwd_body<T, 1>(wg, tiny, ntiny, rows, Lx, Linv, X, 1, lds);
            else solve_tiny_bwd_body<T, NR>(wg, tiny, ntiny, rows, Lx, Linv, X, nrhs, lds);
            return;
        }
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kq = lane & 15, kg = lane >> 4;
    const int64_t q = min(kq, nrhs - 1);  // columns beyond nrhs repeat the last and are not stored
    for (int pass = 0;; ++pass) {
        const int64_t t = next_task<PERSIST>(pass, order, sy.queue + 1, ntasks, &slot);
        if (t < 0) return;
        const SolveTask tk = tasks[t];
        const int nb = tk.nb;
        const int64_t m = tk.m;
        const T *P = Lx + tk.loff;
        const T *Q = Linv + tk.ioff;
        const int nrows = tk.r1 - tk.r0;
        const int ntile = (nb + 15) >> 4;  // column tiles that hold columns of the block
        // Level launches skip the tiles beyond the block's columns and the
        // task's rows (the same for every lane of a wave); the persistent
        // sweep, of mostly full blocks, keeps the unconditional form.
        auto row_tile = [&](int u) { return PERSIST || 64 * u + 16 * wave < nrows; };
        auto col_tile = [&](int ct) { return PERSIST || ct < ntile; };
        Quad<T> av[4][NT];
        grs[tid] = rows[tk.roff + min<int64_t>(tk.r0 + tid, m - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t r = min<int64_t>(tk.r0 + 64 * u + 16 * wave + 4 * kg, m - 1);
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                if (row_tile(u) && col_tile(ct))
                    av[u][ct] = load_quad(P + (int64_t)(tk.c0 + min(16 * ct + kq, nb - 1)) * m + r);
                else
                    av[u][ct] = Quad<T>{};
            }
        }
        const bool may_finish = !PERSIST || tk.first;
        if (may_finish) {
            T ld[NB * NB / 256];
#pragma unroll
            for (int u = 0; u < NB * NB / 256; ++u) {
                const int e = tid + 256 * u, i = e % NB, k = e / NB;
                ld[u] = Q[(int64_t)min(k, nb - 1) * nb + min(i, nb - 1)];
            }
#pragma unroll
            for (int u = 0; u < NB * NB / 256; ++u) {
                const int e = tid + 256 * u, i = e % NB, k = e / NB;
                Qs[k][i] = i >= k && i < nb && k < nb ? ld[u] : T(0);
            }
        }
        const int c = 16 * wave + kq;  // this lane's column of the inverse
        // the block's own forward values (as in k_solve_bwd); thread's
        // entries (row ei(v), right-hand side kq)
        auto ei = [&](int v) { return (tid >> 4) + 16 * v; };
        T xb[EPT];
        auto load_xb = [&]() {
#pragma unroll
            for (int v = 0; v < EPT; ++v) xb[v] = X[(int64_t)(tk.g0 + min(ei(v), nb - 1)) * nrhs + q];
        };
#pragma unroll
        for (int v = 0; v < EPT; ++v) xb[v] = T(0);
        if (tk.ntasks == 1 || (PERSIST && tk.first)) load_xb();
        const bool finisher = PERSIST && tk.first && tk.ntasks > 1;
        auto take_acc = [&]() {
#pragma unroll
            for (int v = 0; v < EPT; ++v)
                if (ei(v) < nb && kq < nrhs)
                    xb[v] -= __hip_atomic_exchange(&Acc[(int64_t)(tk.g0 + ei(v)) * nrhs + kq], T(0),
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        if (finisher) {
            // every other task of the block was dequeued before this one
            if (tid == 0) wait_value(&sy.cnt[tk.blk], tk.ntasks - 1, sy.err, sy.spin);
            __syncthreads();
            acquire_after_wait();
            take_acc();
        }
        const int nhand = (PERSIST && (tk.hand & kHandOut)) ? tk.hand >> 8 : 0;  // rows of the next block
        __syncthreads();
        if (nrows < 256) {
            // a ragged task: what the wide loads took beyond its rows
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool in = 64 * u + 16 * wave + 4 * kg + j < nrows;
#pragma unroll
                    for (int ct = 0; ct < NT; ++ct) av[u][ct].v[j] = in ? av[u][ct].v[j] : T(0);
                }
        }
        acc_t acc[NT];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) acc[ct] = acc_t{0, 0, 0, 0};
        auto at = [&](int u, int j) { return 64 * u + 16 * wave + 4 * kg + j; };
        auto product = [&](int u, const T *xv) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int ct = 0; ct < NT; ++ct)
                    if (col_tile(ct)) acc[ct] = M::run(av[u][ct].v[j], xv[j], acc[ct]);
        };
        if constexpr (PERSIST) {
            if (nhand < nrows) (void)wait_handed(&XB[(int64_t)grs[nhand] * nrhs], sy.err, sy.spin);
            T xf[12], xn[4];
            if (nrows > 64) {
                fetch_rows<T, 3>(XB, grs, 16 * wave + 4 * kg, 1, nrows, nrhs, q, sy, xf);
#pragma unroll
                for (int u = 3; u >= 1; --u) product(u, xf + 4 * (u - 1));
            }
            if (nrows > 0) {
                fetch_rows<T, 1>(XB, grs, 16 * wave + 4 * kg, 0, nrows, nrhs, q, sy, xn);
                product(0, xn);
            }
        } else {
#pragma unroll
            for (int u = 3; u >= 0; --u) {
                if (!row_tile(u)) continue;
                T xv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const T v = X[(int64_t)grs[at(u, j)] * nrhs + q];
                    xv[j] = at(u, j) < nrows ? v : T(0);
                }
                product(u, xv);
            }
        }
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int v = 0; v < 4; ++v) Sm[wave][16 * ct + M::row(lane, v)][kq] = acc[ct][v];
        __syncthreads();
        T sum[EPT];
#pragma unroll
        for (int v = 0; v < EPT; ++v)
            sum[v] = (Sm[0][ei(v)][kq] + Sm[1][ei(v)][kq]) + (Sm[2][ei(v)][kq] + Sm[3][ei(v)][kq]);
        bool fin = true;
        if (tk.ntasks > 1 && !finisher) {
            // the partial sums are device-scope atomics and the finishing
            // task reads them back with atomic exchanges: each thread only
            // waits for its own atomics to be performed before the count
            // goes up
            if (nrows > 0)
#pragma unroll
                for (int v = 0; v < EPT; ++v)
                    if (ei(v) < nb && kq < nrhs) atomicAdd(&Acc[(int64_t)(tk.g0 + ei(v)) * nrhs + kq], sum[v]);
            release_own();
            __syncthreads();
            if (PERSIST) {
                if (tid == 0) atomicAdd(&sy.cnt[tk.blk], 1);
                fin = false;
            } else {
                if (tid == 0) last = (atomicAdd(&sy.cnt[tk.blk], 1) == tk.ntasks - 1);
                __syncthreads();
                fin = last;
                if (fin) {
                    load_xb();
                    take_acc();
#pragma unroll
                    for (int v = 0; v < EPT; ++v) sum[v] = T(0);
                }
            }
        }
        if (fin) {
            if (tid == 0 && tk.ntasks > 1) sy.cnt[tk.blk] = 0;
#pragma unroll
            for (int v = 0; v < EPT; ++v) tq[ei(v)][kq] = ei(v) < nb ? xb[v] - sum[v] : T(0);
            __syncthreads();
            // x_q = Linv^T t; the inverse is zero above row c
            acc_t xa[2] = {acc_t{0, 0, 0, 0}, acc_t{0, 0, 0, 0}};
#pragma unroll
            for (int s = 0; s < NT; ++s)
                if (s >= wave && col_tile(s))
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int i = 16 * s + 4 * kg + j;
                        xa[j & 1] = M::run(Qs[c][i], tq[i][kq], xa[j & 1]);
                    }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int co = 16 * wave + M::row(lane, v);
                const T xo = xa[0][v] + xa[1][v];
                if (co < nb && kq < nrhs) {
                    const int64_t e = (int64_t)(tk.g0 + co) * nrhs + kq;
                    if (PERSIST) shared_store(&XB[e], xo);
                    X[e] = xo;
                }
            }
        }
        __syncthreads();
    }
}

// Between the persistent sweeps: the backward hand-over buffer (Y, spent)
// unset, the partial sums (Acc, the forward hand-over buffer) zero.
template <typename T>
__global__ void k_solve_turn(T *Y, T *Acc, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    Y[i] = __builtin_bit_cast(T, Unset<T>::bits);
    Acc[i] = T(0);
}

// |v| for the maxima of refinement, with NaN mapped to +Inf: fmax drops a
// NaN operand, and a NaN in a residual or solution must not vanish from
// its norm (the bit patterns of non-negative doubles order as unsigned
// integers, so the maxima run as integer atomicMax on them).
__device__ __forceinline__ double abs_key(double v) { return v != v ? __longlong_as_double(0x7ff0000000000000ll) : fabs(v); }

// ---------------------------------------------------------------------------
// FP64 kernels of iterative refinement.  A is applied in full through a CSR
// of the symmetric pattern whose entries point into the caller's lower-CSC
// values (valmap), so refinement always uses the values given.  Vectors are
// n x nrhs column-major with leading dimension ld.
// ---------------------------------------------------------------------------
// Sums of Q values over the LPR lanes j of a group: while there is more than
// one value a lane gives half of them to lane j ^ OFF and adds what it gets
// of the other half, so Q - 1 exchanges do for the first steps instead of
// Q each.  Leaves Q / min(Q, LPR) values a lane (fold_first: the first's q).
template <int Q, int OFF, int LPR, int N>
__device__ __forceinline__ void fold_lanes(double (&acc)[N], int j) {
    if constexpr (OFF < LPR) {
        if constexpr (Q > 1) {
            const bool up = (j & OFF) != 0;
#pragma unroll
            for (int k = 0; k < Q / 2; ++k) {
                const double keep = up ? acc[k + Q / 2] : acc[k], give = up ? acc[k] : acc[k + Q / 2];
                acc[k] = keep + __shfl_xor(give, OFF);
            }
            fold_lanes<Q / 2, 2 * OFF, LPR>(acc, j);
        } else {
            acc[0] += __shfl_xor(acc[0], OFF);
            fold_lanes<1, 2 * OFF, LPR>(acc, j);
        }
    }
}
template <int Q, int OFF, int LPR>
__device__ __forceinline__ int fold_first(int j) {
    if constexpr (OFF < LPR && Q > 1) return ((j & OFF) ? Q / 2 : 0) + fold_first<Q / 2, 2 * OFF, LPR>(j);
    else return 0;
}

// Y = B - A X (with B) or Y = A X (B == nullptr), also to Y2 if that is
// given; zero[0 .. nzero) is cleared (the maxima that the next launch takes).
// LPR consecutive lanes share a row (LPR a power of two <= 64, so a group
// never straddles a wave): lane j of the group takes entries j, j + LPR, ...
// of the row, so a group's index and value loads are contiguous.  Q >= nrhs
// values a lane, the columns past nrhs those of the last one again: a test
// on each column made every one of an entry's gathers wait for the one
// before.  Bound by the gathers (125000 rows of 7 entries, 8 columns: 50 MB,
// 10 us at the copy rate); with the tests and a shuffle per column and step
// 31.3 us, now 20.2; 32 systems of 10000 rows, 16 columns 137, now 90; 24000
// rows of 81 entries, 4 columns 19.5, now 13.4.
template <int LPR, int Q>
__global__ __launch_bounds__(256) void k_spmv(const int64_t *rowptr, const int32_t *colidx, const int64_t *valmap,
                                              const double *values, const double *X, const double *B, double *Y,
                                              double *Y2, int64_t n, int nrhs, int64_t ld, unsigned long long *zero,
                                              int64_t nzero) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t k = id; k < nzero; k += (int64_t)gridDim.x * blockDim.x) zero[k] = 0;
    const int64_t i = id / LPR;
    const int64_t ic = i < n ? i : n - 1;
    const int j = threadIdx.x % LPR;
    constexpr int F = Q > LPR ? Q / LPR : 1, S = Q > LPR ? LPR : Q;  // values a lane holds at the end, lanes that store
    const int qf = fold_first<Q, 1, LPR>(j);
    const int64_t e1 = rowptr[ic + 1];
    int64_t e = rowptr[ic] + j;
    double b[F];
#pragma unroll
    for (int k = 0; k < F; ++k) b[k] = B ? B[ic + (int64_t)min(qf + k, nrhs - 1) * ld] : 0.0;
    double acc[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[q] = 0.0;
    for (; e < e1; e += LPR) {
        const double a = values[valmap[e]];
        const double *x = X + colidx[e];
        double v[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) v[q] = x[(int64_t)min(q, nrhs - 1) * ld];
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[q] += a * v[q];
    }
    // every lane takes part in the shuffles
    fold_lanes<Q, 1, LPR>(acc, j);
    if (i < n && j < S)
#pragma unroll
        for (int k = 0; k < F; ++k)
            if (qf + k < nrhs) {
                const int64_t o = i + (int64_t)(qf + k) * ld;
                const double y = B ? b[k] - acc[k] : acc[k];
                Y[o] = y;
                if (Y2) Y2[o] = y;
            }
}

// out = max_i sum_j |a_ij| (as the bit pattern of a non-negative double):
// LPR lanes per row as in k_spmv (so a group's loads are contiguous), rows
// taken grid-stride by a capped grid, one atomic per workgroup
template <int LPR>
__global__ __launch_bounds__(256) void k_norm_inf_A(const int64_t *rowptr, const int64_t *valmap,
                                                    const double *values, int64_t n, unsigned long long *out) {
    __shared__ double wmax[4];
    const int j = threadIdx.x % LPR;
    const int64_t stride = (int64_t)gridDim.x * (blockDim.x / LPR);
    double mx = 0.0;
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / LPR;; i += stride) {
        // every lane takes part in the shuffles: the loop ends for a whole
        // wave at once (i advances by the same stride in all its groups)
        if (__builtin_amdgcn_ballot_w64(i < n) == 0) break;
        double sum = 0.0;
        if (i < n)
            for (int64_t e = rowptr[i] + j; e < rowptr[i + 1]; e += LPR) sum += fabs(values[valmap[e]]);
#pragma unroll
        for (int off = LPR / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
        mx = fmax(mx, abs_key(sum));  // NaN as +Inf
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0)
        atomicMax(out, (unsigned long long)__double_as_longlong(fmax(fmax(wmax[0], wmax[1]), fmax(wmax[2], wmax[3]))));
}

// Y[:, q] = a_q X[:, q] + b_q Y[:, q]; a_q = a[q] (device) or a0 when a is
// null, likewise b_q; b_q = 0 does not read Y.
__global__ void k_axpby(const double *a, double a0, const double *X, const double *b, double b0, double *Y,
                        int64_t n, int64_t ld) {
    const int q = blockIdx.y;
    const double aq = a ? a[q] : a0, bq = b ? b[q] : b0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        Y[i + q * ld] = (bq == 0.0) ? aq * X[i + q * ld] : aq * X[i + q * ld] + bq * Y[i + q * ld];
}

// Conjugate-gradient coefficients per (column, system) slot j < K, formed
// on the device so that a step needs no host round trip, from the dot
// products in dots, which are cleared for the next ones.  CG_START: rho[j] =
// dots[j].  CG_BETA: coef[K + j] = dots[j] / rho[j], then rho[j] = dots[j].
// CG_ALPHA: coef[j] = rho[j] / dots[j]; umax[0 .. 2K), the maxima that
// k_cg_update takes, are cleared.  A frozen slot (its column has met the
// tolerance) and a quotient that is not finite give 0, and a frozen slot
// keeps its rho.
__global__ void k_cg_coef(double *dots, double *rho, const double *frozen, double *coef, unsigned long long *umax,
                          int64_t K, int mode) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= K) return;
    const bool fz = frozen[j] != 0.0;
    const double d = dots[j], r = rho[j];
    dots[j] = 0.0;
    if (mode == CG_START) {
        rho[j] = d;
    } else if (mode == CG_BETA) {
        const double bt = (r != 0.0 && isfinite(d / r)) ? d / r : 0.0;
        coef[K + j] = fz ? 0.0 : bt;
        if (!fz) rho[j] = d;
    } else {
        coef[j] = (!fz && d > 0.0 && isfinite(r / d)) ? r / d : 0.0;
        umax[j] = 0;
        umax[K + j] = 0;
    }
}

// copy n x q between leading dimensions
__global__ void k_copy_cols(const double *X, int64_t ldx, double *Y, int64_t ldy, int64_t n) {
    const int q = blockIdx.y;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        Y[i + q * ldy] = X[i + q * ldx];
}

// Batched right-hand sides: system i's n_i x nrhs block (leading dimension
// ld[i]) <-> rows off[i].. of the merged n x nrhs array (leading dimension
// n).  grid.x = systems, grid.y = right-hand sides, grid.z shares a column's
// rows: 32 systems of 10000 rows, 16 columns took 70 us with one workgroup a
// column (a fifth of the copy rate), now 31.
__global__ void k_batch_move(double *const *ptrs, const int64_t *lds, const int64_t *offs, double *M, int64_t n,
                             int to_merged) {
    const int i = blockIdx.x, q = blockIdx.y;
    const int64_t o = offs[i], ni = offs[i + 1] - o, ld = lds[i];
    double *X = ptrs[i];
    for (int64_t r = (int64_t)blockIdx.z * blockDim.x + threadIdx.x; r < ni; r += (int64_t)gridDim.z * blockDim.x) {
        if (to_merged) M[o + r + q * n] = X[r + q * ld];
        else X[r + q * ld] = M[o + r + q * n];
    }
}

// Segmented forms for batches: row i belongs to system seg[i] (the rows of
// a system are contiguous and the ids ascend), and every reduction or
// coefficient is kept per (column q, system) at index q * nseg + seg[i].
// One row per thread: a wave whose rows all lie in one system reduces in
// registers and makes one atomic; a wave across a boundary makes one per
// row.  Lanes past n contribute the identity (0 for max of magnitudes and
// for sums).
__device__ inline bool wave_in_one_segment(int s) { return __shfl(s, 0) == __shfl(s, 63); }

__global__ void k_seg_norm_inf_A(const int64_t *rowptr, const int64_t *valmap, const double *values,
                                 const int32_t *seg, int64_t n, unsigned long long *out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int s = seg[i < n ? i : n - 1];
    double sum = 0.0;
    if (i < n)
        for (int64_t e = rowptr[i]; e < rowptr[i + 1]; ++e) sum += fabs(values[valmap[e]]);
    sum = abs_key(sum);
    if (wave_in_one_segment(s)) {
        for (int off = 32; off > 0; off >>= 1) sum = fmax(sum, __shfl_xor(sum, off));
        if ((threadIdx.x & 63) == 0) atomicMax(&out[s], (unsigned long long)__double_as_longlong(sum));
    } else if (i < n) {
        atomicMax(&out[s], (unsigned long long)__double_as_longlong(sum));
    }
}

// Column reductions, grid.y = q: a workgroup of 256 threads takes kRedRows
// consecutive rows, kRedPer a thread, their loads ahead of the first use.
// One system (SEG false): the chunks of a workgroup follow each other at the
// grid's stride, one atomic per workgroup (atomics on one address serialize
// at L2).  A batch: a system's rows are contiguous, so when the first and
// last row of the chunk belong to one system the whole chunk does: one
// atomic too; a chunk that spans systems makes one per wave (or per row
// where a wave spans systems).
constexpr int kRedPer = 4, kRedRows = 256 * kRedPer;

// MAX: the larger of two magnitudes (out holds their bit patterns), else the sum
template <bool MAX>
__device__ __forceinline__ double red_op(double a, double b) { return MAX ? fmax(a, b) : a + b; }
template <bool MAX>
__device__ __forceinline__ void red_out(double *out, double v) {
    if constexpr (MAX) atomicMax((unsigned long long *)out, (unsigned long long)__double_as_longlong(v));
    else atomicAdd(out, v);
}
template <bool MAX>
__device__ __forceinline__ double red_wave(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = red_op<MAX>(v, __shfl_xor(v, off));
    return v;
}
template <bool MAX>
__device__ __forceinline__ void red_workgroup(double v, double *out, double *w4) {
    v = red_wave<MAX>(v);
    if ((threadIdx.x & 63) == 0) w4[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) red_out<MAX>(out, red_op<MAX>(red_op<MAX>(w4[0], w4[1]), red_op<MAX>(w4[2], w4[3])));
}
// the workgroup's chunk lies in one system (the same answer for every thread)
__device__ __forceinline__ bool chunk_in_one_segment(const int32_t *seg, int64_t n) {
    const int64_t base = (int64_t)blockIdx.x * kRedRows;
    return seg[base] == seg[(base + kRedRows < n ? base + kRedRows : n) - 1];
}
// a chunk that spans systems; v: this thread's rows (0 past n), out: the column's slots
template <bool MAX>
__device__ __forceinline__ void red_mixed(const double (&v)[kRedPer], const int32_t *seg, int64_t n, double *out) {
#pragma unroll
    for (int r = 0; r < kRedPer; ++r) {
        const int64_t i = (int64_t)blockIdx.x * kRedRows + r * 256 + threadIdx.x;
        const int s = seg[i < n ? i : n - 1];
        if (wave_in_one_segment(s)) {
            const double w = red_wave<MAX>(v[r]);
            if ((threadIdx.x & 63) == 0) red_out<MAX>(out + s, w);
        } else if (i < n) {
            red_out<MAX>(out + s, v[r]);
        }
    }
}

// out[z K + q nseg + s] = max |V_z[i, q]| over system s (bit patterns; NaN as
// +Inf), V0 for grid.z = 0 and V1 for 1
template <bool SEG>
__global__ __launch_bounds__(256) void k_colmax(const double *V0, const double *V1, const int32_t *seg, int64_t n,
                                                int64_t ld, int nseg, double *out, int64_t K) {
    __shared__ double w4[4];
    const double *V = (blockIdx.z ? V1 : V0) + blockIdx.y * ld;
    out += blockIdx.z * K + (int64_t)blockIdx.y * nseg;
    double v[kRedPer], mx = 0.0;
    for (int64_t base = (int64_t)blockIdx.x * kRedRows; base < n; base += (int64_t)gridDim.x * kRedRows) {
        // (past n the last row again, which is the same chunk's)
#pragma unroll
        for (int r = 0; r < kRedPer; ++r) v[r] = V[min(base + r * 256 + threadIdx.x, n - 1)];
#pragma unroll
        for (int r = 0; r < kRedPer; ++r) v[r] = abs_key(v[r]);
#pragma unroll
        for (int r = 0; r < kRedPer; ++r) mx = fmax(mx, v[r]);
    }
    if constexpr (SEG) {
        if (!chunk_in_one_segment(seg, n)) return red_mixed<true>(v, seg, n, out);
        out += seg[(int64_t)blockIdx.x * kRedRows];
    }
    red_workgroup<true>(mx, out, w4);
}

// out[q nseg + s] += sum U[i, q] V[i, q] over system s
template <bool SEG>
__global__ __launch_bounds__(256) void k_coldot(const double *U, const double *V, const int32_t *seg, int64_t n,
                                                int64_t ld, int nseg, double *out) {
    __shared__ double w4[4];
    U += blockIdx.y * ld;
    V += blockIdx.y * ld;
    out += (int64_t)blockIdx.y * nseg;
    double v[kRedPer], acc = 0.0;
    for (int64_t base = (int64_t)blockIdx.x * kRedRows; base < n; base += (int64_t)gridDim.x * kRedRows) {
        double u[kRedPer];
#pragma unroll
        for (int r = 0; r < kRedPer; ++r) {
            const int64_t i = min(base + r * 256 + threadIdx.x, n - 1);
            u[r] = U[i];
            v[r] = V[i];
        }
#pragma unroll
        for (int r = 0; r < kRedPer; ++r) {
            v[r] = base + r * 256 + threadIdx.x < n ? u[r] * v[r] : 0.0;
            acc += v[r];
        }
    }
    if constexpr (SEG) {
        if (!chunk_in_one_segment(seg, n)) return red_mixed<false>(v, seg, n, out);
        out += seg[(int64_t)blockIdx.x * kRedRows];
    }
    red_workgroup<false>(acc, out, w4);
}

// What a refined solve starts with: b into Bw and Xw (leading dimension n),
// out[q nseg + s] = max |b|
template <bool SEG>
__global__ __launch_bounds__(256) void k_refine_start(const double *B, int64_t ldb, double *Bw, double *Xw,
                                                      const int32_t *seg, int64_t n, int nseg, double *out) {
    __shared__ double w4[4];
    B += blockIdx.y * ldb;
    Bw += blockIdx.y * n;
    Xw += blockIdx.y * n;
    out += (int64_t)blockIdx.y * nseg;
    double v[kRedPer], mx = 0.0;
    for (int64_t base = (int64_t)blockIdx.x * kRedRows; base < n; base += (int64_t)gridDim.x * kRedRows) {
#pragma unroll
        for (int r = 0; r < kRedPer; ++r) v[r] = B[min(base + r * 256 + threadIdx.x, n - 1)];
#pragma unroll
        for (int r = 0; r < kRedPer; ++r) {
            const int64_t i = base + r * 256 + threadIdx.x;
            if (i < n) {
                Bw[i] = v[r];
                Xw[i] = v[r];
            }
            v[r] = abs_key(v[r]);
            mx = fmax(mx, v[r]);
        }
    }
    if constexpr (SEG) {
        if (!chunk_in_one_segment(seg, n)) return red_mixed<true>(v, seg, n, out);
        out += seg[(int64_t)blockIdx.x * kRedRows];
    }
    red_workgroup<true>(mx, out, w4);
}

// The end of a conjugate-gradient step in one pass: x += alpha p, r -= alpha
// q, z = r (what the next preconditioner solve starts from), and the maxima
// of r and x per slot (out, out + K; cleared by k_cg_coef).  As launches of
// their own these were two updates, a copy, a clear and two reductions, 29 us
// and five gaps on 24000 rows x 4 columns; now 5.1 us.
template <bool SEG>
__global__ __launch_bounds__(256) void k_cg_update(const double *alpha, const double *Pv, const double *Qv, double *X,
                                                   double *R, double *Z, const int32_t *seg, int64_t n, int nseg,
                                                   double *out, int64_t K) {
    __shared__ double w4[8];
    const int64_t o = blockIdx.y * n, slot = (int64_t)blockIdx.y * nseg;
    double xv[kRedPer], rv[kRedPer], xm = 0.0, rm = 0.0;
    for (int64_t base = (int64_t)blockIdx.x * kRedRows; base < n; base += (int64_t)gridDim.x * kRedRows) {
        double pv[kRedPer], qv[kRedPer], a[kRedPer];
#pragma unroll
        for (int r = 0; r < kRedPer; ++r) {
            const int64_t i = min(base + r * 256 + threadIdx.x, n - 1);
            a[r] = alpha[slot + (SEG ? seg[i] : 0)];
            xv[r] = X[o + i];
            rv[r] = R[o + i];
            pv[r] = Pv[o + i];
            qv[r] = Qv[o + i];
        }
#pragma unroll
        for (int r = 0; r < kRedPer; ++r) {
            const int64_t i = base + r * 256 + threadIdx.x;
            xv[r] += a[r] * pv[r];
            rv[r] -= a[r] * qv[r];
            if (i < n) {
                X[o + i] = xv[r];
                R[o + i] = rv[r];
                Z[o + i] = rv[r];
            }
            // (past n another thread's row, perhaps already updated)
            xv[r] = i < n ? abs_key(xv[r]) : 0.0;
            rv[r] = i < n ? abs_key(rv[r]) : 0.0;
            xm = fmax(xm, xv[r]);
            rm = fmax(rm, rv[r]);
        }
    }
    out += slot;
    if constexpr (SEG) {
        if (!chunk_in_one_segment(seg, n)) {
            red_mixed<true>(rv, seg, n, out);
            red_mixed<true>(xv, seg, n, out + K);
            return;
        }
        out += seg[(int64_t)blockIdx.x * kRedRows];
    }
    red_workgroup<true>(rm, out, w4);
    red_workgroup<true>(xm, out + K, w4 + 4);
}

// Y[:, q] = a X[:, q] + b Y[:, q] with a = a[q * nseg + seg[i]] (or a0 when
// a is null), likewise b; b = 0 does not read Y.
__global__ void k_seg_axpby(const double *a, double a0, const double *X, const double *b, double b0, double *Y,
                            const int32_t *seg, int64_t n, int64_t ld, int nseg) {
    const int q = blockIdx.y;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t k = (int64_t)q * nseg + seg[i];
    const double aq = a ? a[k] : a0, bq = b ? b[k] : b0;
    Y[i + q * ld] = (bq == 0.0) ? aq * X[i + q * ld] : aq * X[i + q * ld] + bq * Y[i + q * ld];
}

inline unsigned grid1(int64_t count, int block) {
    int64_t g = (count + block - 1) / block;
    return (unsigned)(g > 0 ? g : 1);
}

}  // namespace

void launch_status_reset(unsigned long long *status, int count, int32_t *deverr, int32_t *flags, int nflags,
                         hipStream_t st) {
    const int n = count > nflags ? count : nflags;
    if (n <= 0) return;
    hipLaunchKernelGGL(k_status_reset, dim3((n + 255) / 256), dim3(256), 0, st, status, count, deverr, flags, nflags);
}

template <typename T>
void launch_zero(T *x, int64_t count, hipStream_t st) {
    if (count <= 0) return;
    int64_t g = (count + 255) / 256;
    if (g > 65536) g = 65536;
    hipLaunchKernelGGL(k_zero<T>, dim3((unsigned)g), dim3(256), 0, st, x, count);
}

template <typename T>
void launch_assemble(const DevPlan &P, int64_t nnz, const double *values, T *Lx, hipStream_t st) {
    if (nnz <= 0) return;
    hipLaunchKernelGGL(k_assemble<T>, dim3(grid1(nnz, 256)), dim3(256), 0, st, P.amap, nnz, values, Lx);
}

template <typename T>
void launch_pivot_floor(const DevPlan &P, int64_t n, const double *values, double theta, T *floor, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_pivot_floor<T>, dim3(grid1(n, 256)), dim3(256), 0, st, P.dsrc, n, values, theta, floor);
}

static int64_t tiny_blocks(const TinyRange &t) {
    const int64_t n16 = t.e16 - t.t0, n32 = t.e32 - t.t0, nt = t.t1 - t.t0;
    return (n16 + 15) / 16 + (n32 - n16 + 7) / 8 + (nt - n32 + 3) / 4;
}

template <typename T>
void launch_level(const DevPlan &P, int64_t p0, int64_t p1, int64_t s0, int64_t s1, TinyRange t, T *Lx, T *Linv,
                  unsigned long long *status, PivotFloor<T> pfl, hipStream_t st) {
    const int64_t blocks = (p1 - p0) + (s1 - s0) + tiny_blocks(t);
    if (blocks <= 0) return;
    const auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, st, P.potrf_tasks + p0, (int)(p1 - p0),
                           P.small_tasks + s0, (int)(s1 - s0), P.tiny_tasks + t.t0, t.e16 - t.t0, t.e32 - t.t0,
                           t.t1 - t.t0, P.cbase, P.crel, P.rel, Lx, Linv, status, P.status_slot, pfl);
    };
    if (pfl.v) launch(k_level<T, true>);
    else launch(k_level<T, false>);
}

template <typename T>
void launch_tiles(const DevPlan &P, int mode, int64_t t0, int64_t t1, T *Lx, T *Linv, unsigned long long *status,
                  int32_t *hflags, WaitCtl wc, bool bf16, PivotFloor<T> pfl, hipStream_t st) {
    if (t1 <= t0) return;
    const dim3 g((unsigned)(t1 - t0)), b(256);
    if constexpr (std::is_same<T, float>::value) {
        if (bf16 && mode == kTilesTrailing) {
            hipLaunchKernelGGL((k_tiles<T, MODE_TRAILING, true>), g, b, 0, st, P.int_tiles + t0, P.cbase, P.crel,
                               P.rel, Linv, Lx, status, P.status_slot, hflags, wc, pfl);
            return;
        }
        if (bf16 && mode == kTilesScatter) {
            hipLaunchKernelGGL((k_tiles<T, MODE_SCATTER, true>), g, b, 0, st, P.ext_tiles + t0, P.cbase, P.crel,
                               P.rel, Linv, Lx, status, P.status_slot, (int32_t *)nullptr, wc, pfl);
            return;
        }
    }
    if (mode == kTilesTrailing)
        hipLaunchKernelGGL((k_tiles<T, MODE_TRAILING>), g, b, 0, st, P.int_tiles + t0, P.cbase, P.crel, P.rel,
                           Linv, Lx, status, P.status_slot, hflags, wc, PivotFloor<T>{});
    else if (mode == kTilesScatter)
        hipLaunchKernelGGL((k_tiles<T, MODE_SCATTER>), g, b, 0, st, P.ext_tiles + t0, P.cbase, P.crel, P.rel,
                           Linv, Lx, status, P.status_slot, (int32_t *)nullptr, wc, PivotFloor<T>{});
    else
        hipLaunchKernelGGL((k_tiles<T, MODE_TRSM>), g, b, 0, st, P.trsm_tiles + t0, P.cbase, P.crel, P.rel,
                           Linv, Lx, status, P.status_slot, (int32_t *)nullptr, wc, PivotFloor<T>{});
}

template <typename T>
void launch_tiles128(const DevPlan &P, int64_t t0, int64_t t1, T *Lx, bool bf16, hipStream_t st) {
    if (t1 <= t0) return;
    if constexpr (std::is_same<T, float>::value) {
        if (bf16) {
            hipLaunchKernelGGL((k_tiles128<T, true>), dim3((unsigned)(t1 - t0)), dim3(512), 0, st,
                               P.ext_tiles_big + t0, P.cbase, P.crel, P.rel, Lx);
            return;
        }
    }
    hipLaunchKernelGGL((k_tiles128<T, false>), dim3((unsigned)(t1 - t0)), dim3(512), 0, st,
                       P.ext_tiles_big + t0, P.cbase, P.crel, P.rel, Lx);
}

template <typename T>
void launch_trail128(const DevPlan &P, int64_t t0, int64_t t1, T *Lx, bool bf16, hipStream_t st) {
    if (t1 <= t0) return;
    if constexpr (std::is_same<T, float>::value) {
        if (bf16) {
            hipLaunchKernelGGL((k_tiles128<T, true, true>), dim3((unsigned)(t1 - t0)), dim3(512), 0, st,
                               P.trail_big + t0, P.cbase, P.crel, P.rel, Lx);
            return;
        }
    }
    hipLaunchKernelGGL((k_tiles128<T, false, true>), dim3((unsigned)(t1 - t0)), dim3(512), 0, st,
                       P.trail_big + t0, P.cbase, P.crel, P.rel, Lx);
}

template <typename T>
void launch_persist_small(const DevPlan &P, int64_t nchunks, int64_t nsuper, int32_t *pdep, int32_t *qctr, T *Lx,
                          T *Linv, unsigned long long *status, PivotFloor<T> pfl, WaitCtl wc, hipStream_t st) {
    if (nchunks <= 0) return;
    hipLaunchKernelGGL(k_persist_reset, dim3(grid1(std::max<int64_t>(nsuper, 1), 256)), dim3(256), 0, st, P.pdep0,
                       nsuper, pdep, qctr);
    // as many workgroups as can be resident at once (the kernel's occupancy
    // times the CUs), measured once per precision: the entries are short and
    // latency-bound, so every resident slot counts
    static int resident[2] = {0, 0};
    int &r = resident[sizeof(T) == 8 ? 1 : 0];
    if (r == 0) {
        int per_cu = 0, dev = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_persist_small<T>, 256, 0) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per_cu < 1 ||
            cus < 1)
            r = 768;
        else
            r = per_cu * cus;
    }
    const unsigned g = (unsigned)std::min<int64_t>(nchunks, r);
    hipLaunchKernelGGL(k_persist_small<T>, dim3(g), dim3(256), 0, st, P.pqueue, P.pchunk, nchunks, P.psmall, P.ptiny,
                       P.ptgt_ptr,
                       P.ptgt, pdep, qctr, P.cbase, P.crel, P.rel, Lx, Linv, status, P.status_slot, pfl, wc);
}

template <typename T>
void launch_solve_init(const DevPlan &P, int64_t n, int nrhs, const double *B, int64_t ldb, T *Y, T *Acc,
                       bool persist, int64_t nblocks, SolveSync sy, hipStream_t st) {
    const int64_t count = std::max<int64_t>(std::max<int64_t>(n * nrhs, nblocks), 2);
    hipLaunchKernelGGL(k_solve_init<T>, dim3(grid1(count, 256)), dim3(256), 0, st, P.perm, n, nrhs, B, ldb, Y, Acc,
                       persist ? 1 : 0, P.fdep, nblocks, sy);
}

template <typename T>
void launch_solve_turn(T *Y, T *Acc, int64_t count, hipStream_t st) {
    if (count <= 0) return;
    hipLaunchKernelGGL(k_solve_turn<T>, dim3(grid1(count, 256)), dim3(256), 0, st, Y, Acc, count);
}

template <typename T>
void launch_perm_out(const DevPlan &P, int64_t n, int nrhs, const T *W, double *B, int64_t ldb,
                     hipStream_t st) {
    if (n * nrhs <= 0) return;
    hipLaunchKernelGGL(k_perm_out<T>, dim3(grid1(n * nrhs, 256)), dim3(256), 0, st, P.perm, n, nrhs, W,
                       B, ldb);
}

inline unsigned persist_grid(int64_t ntasks) {
    // two resident workgroups per CU on 256 CUs; more only queue behind them
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(ntasks, 512));
}

// The persistent sweeps over the tasks t0 .. t1
template <typename T>
void launch_solve_fwd(const DevPlan &P, int64_t t0, int64_t t1, const T *Lx, const T *Linv, T *Y, T *X, T *H,
                      int64_t n, int nrhs, SolveSync sy, hipStream_t st) {
    if (t1 <= t0) return;
    const int64_t nt = t1 - t0;
    const dim3 g(persist_grid(nt)), b(256);
    const SolveTask *tk = P.stasks + t0;
    const int64_t *tp = P.stgt_ptr + t0;
    if (nrhs == 1)
        hipLaunchKernelGGL((k_solve_fwd<T, true>), g, b, 0, st, tk, nt, P.rows, Lx, Linv, Y, X, H, n, tp, P.stgt, sy,
                           nullptr, 0);
    else
        hipLaunchKernelGGL((k_solve_fwd_multi<T, true>), g, b, 0, st, tk, nt, P.rows, Lx, Linv, Y, X, H, n, nrhs, tp,
                           P.stgt, sy, nullptr, 0);
}

template <typename T>
void launch_solve_bwd(const DevPlan &P, int64_t t0, int64_t t1, const T *Lx, const T *Linv, T *X, T *Acc, T *XB,
                      int64_t n, int nrhs, SolveSync sy, hipStream_t st) {
    if (t1 <= t0) return;
    const int64_t nt = t1 - t0;
    const dim3 g(persist_grid(nt)), b(256);
    // (tasks by their global indices, in the order of bwd_order)
    if (nrhs == 1)
        hipLaunchKernelGGL((k_solve_bwd<T>), g, b, 0, st, P.stasks, nt, P.bwd_order, P.rows, Lx, Linv, X, Acc, XB, sy);
    else
        hipLaunchKernelGGL((k_solve_bwd_multi<T, true>), g, b, 0, st, P.stasks, nt, P.bwd_order, P.rows, Lx, Linv, X,
                           Acc, XB, n, nrhs, sy, nullptr, 0);
}

// One level: its block tasks t0 .. t1 and its tiny supernodes s0 .. s1, in one
// launch.  A launch of either takes 5 to 8 us at the levels below the sweeps,
// most of it start and end: a 50^3 refined re-solve (FP32, 8 columns) 2734 us
// with two launches a level, 2641 with one where the tiny supernodes fill at
// most 512 workgroups, 2593 at most 4096, 2601 always; 32 systems 21^3 (16
// columns) 8443, 8200, 8102, 8118; 34^3 FP32 step 3242, 3208, 3216, 3236.
// Beyond that the tiny ones' own kernel, with fewer registers and less LDS,
// holds more of them in flight.
constexpr int64_t kSolveMergeTiny = 4096;

template <typename T>
void launch_solve_level_fwd(const DevPlan &P, int64_t t0, int64_t t1, int64_t s0, int64_t s1, const T *Lx,
                            const T *Linv, T *Y, T *X, int64_t n, int nrhs, SolveSync sy, hipStream_t st) {
    const int64_t nt = t1 - t0, wgs = (s1 - s0 + 3) / 4;
    const bool merge = nt > 0 && wgs <= kSolveMergeTiny;
    const dim3 b(256);
    const SmallTask *tiny = P.stiny + s0;
    if (wgs > 0 && !merge) {
        if (nrhs == 1)
            hipLaunchKernelGGL((k_solve_tiny_fwd<T, 1>), dim3((unsigned)wgs), b, 0, st, tiny, s1 - s0, P.rows, Lx,
                               Linv, Y, X, nrhs);
        else
            hipLaunchKernelGGL((k_solve_tiny_fwd<T, kMaxRhs>), dim3((unsigned)wgs), b, 0, st, tiny, s1 - s0, P.rows,
                               Lx, Linv, Y, X, nrhs);
    }
    if (nt <= 0) return;
    const dim3 g((unsigned)(nt + (merge ? wgs : 0)));
    const SolveTask *tk = P.stasks + t0;
    const int64_t *tp = P.stgt_ptr + t0;
    if (nrhs == 1)
        hipLaunchKernelGGL((k_solve_fwd<T, false>), g, b, 0, st, tk, nt, P.rows, Lx, Linv, Y, X, (T *)nullptr, n, tp,
                           P.stgt, sy, tiny, s1 - s0);
    else
        hipLaunchKernelGGL((k_solve_fwd_multi<T, false>), g, b, 0, st, tk, nt, P.rows, Lx, Linv, Y, X, (T *)nullptr, n,
                           nrhs, tp, P.stgt, sy, tiny, s1 - s0);
}

// (the blocks take the MFMA form for one right-hand side too: their tasks wait
// for nothing and only move the panel, 47 against 28 us a launch on the 60^3
// grid; in the persistent sweep its longer path from block to block costs
// more, 657 against 444 us)
template <typename T>
void launch_solve_level_bwd(const DevPlan &P, int64_t t0, int64_t t1, int64_t s0, int64_t s1, const T *Lx,
                            const T *Linv, T *X, T *Acc, int64_t n, int nrhs, SolveSync sy, hipStream_t st) {
    const int64_t nt = t1 - t0, wgs = (s1 - s0 + 3) / 4;
    const bool merge = nt > 0 && wgs <= kSolveMergeTiny;
    const dim3 b(256);
    const SmallTask *tiny = P.stiny + s0;
    if (wgs > 0 && !merge) {
        if (nrhs == 1)
            hipLaunchKernelGGL((k_solve_tiny_bwd<T, 1>), dim3((unsigned)wgs), b, 0, st, tiny, s1 - s0, P.rows, Lx,
                               Linv, X, nrhs);
        else
            hipLaunchKernelGGL((k_solve_tiny_bwd<T, kMaxRhs>), dim3((unsigned)wgs), b, 0, st, tiny, s1 - s0, P.rows,
                               Lx, Linv, X, nrhs);
    }
    if (nt <= 0) return;
    hipLaunchKernelGGL((k_solve_bwd_multi<T, false>), dim3((unsigned)(nt + (merge ? wgs : 0))), b, 0, st,
                       P.stasks + t0, nt, (const int32_t *)nullptr, P.rows, Lx, Linv, X, Acc, (T *)nullptr, n, nrhs,
                       sy, tiny, s1 - s0);
}

template <int LPR>
static void launch_spmv_lanes(const int64_t *rowptr, const int32_t *colidx, const int64_t *valmap,
                              const double *values, const double *X, const double *B, double *Y, double *Y2,
                              int64_t n, int nrhs, int64_t ld, unsigned long long *zero, int64_t nzero,
                              hipStream_t st) {
    const dim3 g(grid1(n * LPR, 256)), b(256);
    const int64_t nz = zero ? nzero : 0;
    auto go = [&](auto qc) {
        hipLaunchKernelGGL((k_spmv<LPR, decltype(qc)::value>), g, b, 0, st, rowptr, colidx, valmap, values, X, B, Y,
                           Y2, n, nrhs, ld, zero, nz);
    };
    if (nrhs <= 1) go(std::integral_constant<int, 1>{});
    else if (nrhs <= 2) go(std::integral_constant<int, 2>{});
    else if (nrhs <= 4) go(std::integral_constant<int, 4>{});
    else if (nrhs <= 8) go(std::integral_constant<int, 8>{});
    else go(std::integral_constant<int, kMaxRhs>{});
}
void launch_spmv(const int64_t *rowptr, const int32_t *colidx, const int64_t *valmap, const double *values,
                 const double *X, const double *B, double *Y, double *Y2, int64_t n, int64_t nnz, int nrhs,
                 int64_t ld, unsigned long long *zero, int64_t nzero, hipStream_t st) {
    if (n <= 0 || nrhs <= 0) return;
    // lanes per row: the power of two (4..32) at or above the mean row length
    const int64_t avg = (nnz + n - 1) / n;
    auto lanes = avg <= 4 ? launch_spmv_lanes<4>
                 : avg <= 8 ? launch_spmv_lanes<8>
                 : avg <= 16 ? launch_spmv_lanes<16> : launch_spmv_lanes<32>;
    lanes(rowptr, colidx, valmap, values, X, B, Y, Y2, n, nrhs, ld, zero, nzero, st);
}
void launch_norm_inf_A(const int64_t *rowptr, const int64_t *valmap, const double *values, int64_t n, int64_t nnz,
                       unsigned long long *out, hipStream_t st) {
    if (n <= 0) return;
    const int64_t avg = (nnz + n - 1) / n;
    // (one atomic a workgroup, all on one word: 125000 rows of 7 entries 16.5
    // us with 1024 workgroups, 13.3 with 512)
    const unsigned g4 = (unsigned)std::min<int64_t>(grid1(n * 4, 256), 512);
    const unsigned g32 = (unsigned)std::min<int64_t>(grid1(n * 32, 256), 1024);
    if (avg <= 8)
        hipLaunchKernelGGL(k_norm_inf_A<4>, dim3(g4), dim3(256), 0, st, rowptr, valmap, values, n, out);
    else
        hipLaunchKernelGGL(k_norm_inf_A<32>, dim3(g32), dim3(256), 0, st, rowptr, valmap, values, n, out);
}
static unsigned red_grid(int64_t n) {
    int64_t g = (n + 255) / 256;
    return (unsigned)(g < 1 ? 1 : (g > 1024 ? 1024 : g));
}
// Workgroups a column of a reduction: every chunk its own in a batch; else 512
// over the launch's columns, two a CU.  Each ends in an atomic and the slots of
// all columns lie in a line or two, where an atomic takes about 7 ns: 125000
// rows, 8 columns of r and x with one chunk each (1952 of them) 20.1 us, now
// 7.0.  (The maxima of one of the two took 14.2 us with 1024 workgroups.)
static unsigned red_chunks(const int32_t *seg, int64_t n, int columns) {
    const int64_t c = (n + kRedRows - 1) / kRedRows;
    return (unsigned)(seg ? c : std::min<int64_t>(c, std::max(1, 512 / columns)));
}
#define SPC_LAUNCH_SEG(kernel, grid, ...)                                                                   \
    do {                                                                                                    \
        if (seg) hipLaunchKernelGGL(kernel<true>, grid, dim3(256), 0, st, __VA_ARGS__);                     \
        else hipLaunchKernelGGL(kernel<false>, grid, dim3(256), 0, st, __VA_ARGS__);                        \
    } while (0)
void launch_colmax(const double *V0, const double *V1, const int32_t *seg, int64_t n, int nrhs, int64_t ld, int nseg,
                   unsigned long long *out, int64_t K, hipStream_t st) {
    if (n <= 0 || nrhs <= 0) return;
    SPC_LAUNCH_SEG(k_colmax, dim3(red_chunks(seg, n, 2 * nrhs), nrhs, 2), V0, V1, seg, n, ld, nseg, (double *)out, K);
}
void launch_coldot(const double *U, const double *V, const int32_t *seg, int64_t n, int nrhs, int64_t ld, int nseg,
                   double *out, hipStream_t st) {
    if (n <= 0 || nrhs <= 0) return;
    SPC_LAUNCH_SEG(k_coldot, dim3(red_chunks(seg, n, nrhs), nrhs), U, V, seg, n, ld, nseg, out);
}
void launch_refine_start(const double *B, int64_t ldb, double *Bw, double *Xw, const int32_t *seg, int64_t n,
                         int nrhs, int nseg, unsigned long long *out, hipStream_t st) {
    if (n <= 0 || nrhs <= 0) return;
    SPC_LAUNCH_SEG(k_refine_start, dim3(red_chunks(seg, n, nrhs), nrhs), B, ldb, Bw, Xw, seg, n, nseg, (double *)out);
}
void launch_cg_update(const double *alpha, const double *Pv, const double *Qv, double *X, double *R, double *Z,
                      const int32_t *seg, int64_t n, int nrhs, int nseg, unsigned long long *out, int64_t K,
                      hipStream_t st) {
    if (n <= 0 || nrhs <= 0) return;
    SPC_LAUNCH_SEG(k_cg_update, dim3(red_chunks(seg, n, 2 * nrhs), nrhs), alpha, Pv, Qv, X, R, Z, seg, n, nseg, (double *)out,
                   K);
}
#undef SPC_LAUNCH_SEG
void launch_cg_coef(double *dots, double *rho, const double *frozen, double *coef, unsigned long long *umax, int64_t K,
                    CgCoef mode, hipStream_t st) {
    if (K <= 0) return;
    hipLaunchKernelGGL(k_cg_coef, dim3(grid1(K, 256)), dim3(256), 0, st, dots, rho, frozen, coef, umax, K, (int)mode);
}
void launch_axpby(const double *a, double a0, const double *X, const double *b, double b0, double *Y, int64_t n,
                  int nrhs, int64_t ld, hipStream_t st) {
    if (n <= 0 || nrhs <= 0) return;
    hipLaunchKernelGGL(k_axpby, dim3(red_grid(n), nrhs), dim3(256), 0, st, a, a0, X, b, b0, Y, n, ld);
}
void launch_seg_norm_inf_A(const int64_t *rowptr, const int64_t *valmap, const double *values, const int32_t *seg,
                           int64_t n, unsigned long long *out, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_seg_norm_inf_A, dim3(grid1(n, 256)), dim3(256), 0, st, rowptr, valmap, values, seg, n,
                       out);
}
void launch_seg_axpby(const double *a, double a0, const double *X, const double *b, double b0, double *Y,
                      const int32_t *seg, int64_t n, int nrhs, int64_t ld, int nseg, hipStream_t st) {
    if (n <= 0 || nrhs <= 0) return;
    hipLaunchKernelGGL(k_seg_axpby, dim3(grid1(n, 256), nrhs), dim3(256), 0, st, a, a0, X, b, b0, Y, seg, n, ld,
                       nseg);
}
void launch_batch_move(double *const *ptrs, const int64_t *lds, const int64_t *offs, double *M, int64_t n,
                       int count, int nrhs, bool to_merged, hipStream_t st) {
    if (count <= 0 || nrhs <= 0) return;
    // (by the mean size: a larger system's workgroups go on at the grid's stride)
    const unsigned z = (unsigned)std::min<int64_t>(std::max<int64_t>(n / count / 512, 1), 64);
    hipLaunchKernelGGL(k_batch_move, dim3(count, nrhs, z), dim3(256), 0, st, ptrs, lds, offs, M, n,
                       to_merged ? 1 : 0);
}
void launch_copy_cols(const double *X, int64_t ldx, double *Y, int64_t ldy, int64_t n, int nrhs, hipStream_t st) {
    if (n <= 0 || nrhs <= 0) return;
    hipLaunchKernelGGL(k_copy_cols, dim3(red_grid(n), nrhs), dim3(256), 0, st, X, ldx, Y, ldy, n);
}
template void launch_zero<int32_t>(int32_t *, int64_t, hipStream_t);
template void launch_zero<unsigned long long>(unsigned long long *, int64_t, hipStream_t);

#define SPC_INSTANTIATE(T)                                                                                  \
    template void launch_zero<T>(T *, int64_t, hipStream_t);                                                \
    template void launch_assemble<T>(const DevPlan &, int64_t, const double *, T *, hipStream_t);           \
    template void launch_level<T>(const DevPlan &, int64_t, int64_t, int64_t, int64_t, TinyRange, T *, T *,  \
                                  unsigned long long *, PivotFloor<T>, hipStream_t);                        \
    template void launch_pivot_floor<T>(const DevPlan &, int64_t, const double *, double, T *, hipStream_t); \
    template void launch_tiles<T>(const DevPlan &, int, int64_t, int64_t, T *, T *, unsigned long long *,    \
                                  int32_t *, WaitCtl, bool, PivotFloor<T>, hipStream_t);                    \
    template void launch_tiles128<T>(const DevPlan &, int64_t, int64_t, T *, bool, hipStream_t);            \
    template void launch_trail128<T>(const DevPlan &, int64_t, int64_t, T *, bool, hipStream_t);            \
    template void launch_persist_small<T>(const DevPlan &, int64_t, int64_t, int32_t *, int32_t *, T *, T *, \
                                          unsigned long long *, PivotFloor<T>, WaitCtl, hipStream_t);       \
    template void launch_solve_init<T>(const DevPlan &, int64_t, int, const double *, int64_t, T *, T *,     \
                                       bool, int64_t, SolveSync, hipStream_t);                              \
    template void launch_solve_turn<T>(T *, T *, int64_t, hipStream_t);                                     \
    template void launch_perm_out<T>(const DevPlan &, int64_t, int, const T *, double *, int64_t,           \
                                     hipStream_t);                                                          \
    template void launch_solve_fwd<T>(const DevPlan &, int64_t, int64_t, const T *, const T *, T *, T *, T *, \
                                      int64_t, int, SolveSync, hipStream_t);                                \
    template void launch_solve_bwd<T>(const DevPlan &, int64_t, int64_t, const T *, const T *, T *, T *, T *, \
                                      int64_t, int, SolveSync, hipStream_t);                                \
    template void launch_solve_level_fwd<T>(const DevPlan &, int64_t, int64_t, int64_t, int64_t, const T *, \
                                            const T *, T *, T *, int64_t, int, SolveSync, hipStream_t);     \
    template void launch_solve_level_bwd<T>(const DevPlan &, int64_t, int64_t, int64_t, int64_t, const T *, \
                                            const T *, T *, T *, int64_t, int, SolveSync, hipStream_t);
SPC_INSTANTIATE(double)
SPC_INSTANTIATE(float)

// ---------------------------------------------------------------------------
// Scratch for callers that cannot allocate (spc_solve_noalloc): a fixed
// array in device memory, one copy per device, held until the process ends.
// Every call on a device shares it.
// ---------------------------------------------------------------------------
}  // namespace spc

static __device__ __align__(256) unsigned char scratch[spc::kScratchBytes];

namespace spc {

int scratch_address(int device, void **out) {
    static std::mutex mu;
    static void *addr[64] = {};
    if (device < 0 || device >= 64) return -5;  // SPC_DEVICE_ERROR
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[device]) {
        int cur = -1;
        if (hipGetDevice(&cur) != hipSuccess) return -5;
        if (cur != device && hipSetDevice(device) != hipSuccess) return -5;
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess || !p) return -5;
        addr[device] = p;
    }
    *out = addr[device];
    return 0;
}

}  // namespace spc
