// LDS tile helpers shared by the dense kernels: the bank swizzle, the lane
// order of a digit pair's sweep, barriers, reductions, and the gate maps on a
// 16-register block of two digits.
#pragma once

#include "pp_device.h"

namespace pp {

// Bank swizzle for 8-byte LDS words.  The LDS has 64 four-byte banks and
// serves a 64-bit read or write per half-wave, so a half-wave is free of
// conflicts when its 32 slot indices are distinct modulo 32.  With h the
// index bits from bit 5 up, the swizzle XORs bits 0-4 with h << 3, h and
// h >> 2: it is linear over GF(2) and keeps every 32-slot block's set of
// high bits.  With the lane order group_sweep picks per digit pair, every
// digit pair of 5-, 6- and 7-digit tiles is swept without conflicts, and in
// 6-digit tiles so is every pair of digits 0-4 with the lanes drawn from the
// three other digits below 5 alone.
__host__ __device__ constexpr int sw(int i) {
    const int h = i >> 5;
    return i ^ (((h << 3) ^ h ^ (h >> 2)) & 31);
}

// sw(base ^ off) = sw(base) ^ sw(off): slot offsets of an op's letters are
// the same for every lane, so each address costs one XOR with a uniform.

// Workgroup barrier for LDS data: the fences are scoped to LDS, so global
// loads still in flight (a prefetched next tile) are not waited for, which a
// full __syncthreads() would do.  Every barrier in this file orders LDS
// accesses only (threads never exchange data through global memory).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ long long morton_slot(uint64_t x, uint64_t z, int n) {
    long long s = 0;
    for (int q = 0; q < n; ++q)
        s |= (long long)(((x >> q) & 1ull) | (((z >> q) & 1ull) << 1)) << (2 * q);
    return s;
}

// slot of the j-th string made of I and Z only (z word = j)
__device__ __forceinline__ long long zonly_slot(long long j, int n) {
    long long s = 0;
    for (int q = 0; q < n; ++q) s |= ((j >> q) & 1ll) << (2 * q + 1);
    return s;
}

template <int BLOCK>
__device__ double block_sum_d(double v, double *red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int w = threadIdx.x >> 6;
    lds_barrier();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    lds_barrier();
    double tot = 0.0;
    for (int i = 0; i < BLOCK / 64; ++i) tot += red[i];
    return tot;
}

template <int BLOCK>
__device__ long long block_sum_i(long long v, long long *red) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const int w = threadIdx.x >> 6;
    lds_barrier();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    lds_barrier();
    long long tot = 0;
    for (int i = 0; i < BLOCK / 64; ++i) tot += red[i];
    return tot;
}

// One row of a U1 map, m0 cx + m1 cy + m2 cz, with its rounding points fixed:
// a product, then two fused multiply-adds.  Every kernel applies maps through
// it, so all of them round alike whatever the surrounding code would let the
// compiler contract (a negation folded in from a CX, say).
__device__ __forceinline__ double map_row(double m0, double m1, double m2, double cx, double cy, double cz) {
    return __builtin_fma(m2, cz, __builtin_fma(m1, cy, m0 * cx));
}

// The six signed swaps of CX as (control digit, target digit) pairs, derived
// at compile time from the rule above; in the paper's letters they are
// (I,Z)<->(Z,Z), (I,Y)<->(Z,Y), (X,I)<->(X,X), (X,Z)<->-(Y,Y), (X,Y)<->(Y,Z),
// (Y,I)<->(Y,X) (digit values I=0 X=1 Z=2 Y=3).
struct CxPairC { int dc1, dt1, dc2, dt2, neg; };
constexpr CxPairC cx_pair_c(int p) {
    int found = 0;
    for (int dc = 0; dc < 4; ++dc)
        for (int dt = 0; dt < 4; ++dt) {
            const int xc = dc & 1, zc = dc >> 1, xt = dt & 1, zt = dt >> 1;
            const int dc2 = xc | ((zc ^ zt) << 1), dt2 = (xt ^ xc) | (zt << 1);
            if (dc2 * 4 + dt2 > dc * 4 + dt) {
                if (found == p) return CxPairC{dc, dt, dc2, dt2, xc & zt & ((xt ^ zc) ^ 1)};
                ++found;
            }
        }
    return CxPairC{0, 0, 0, 0, 0};
}
static_assert(cx_pair_c(3).dc1 == 1 && cx_pair_c(3).dt1 == 2 && cx_pair_c(3).dc2 == 3 && cx_pair_c(3).dt2 == 3 &&
                  cx_pair_c(3).neg == 1,
              "XZ <-> -YY");

template <bool CTRL_LO, int P>
__device__ __forceinline__ void cx_swap(double *v) {
    constexpr CxPairC pr = cx_pair_c(P);
    constexpr int e1 = CTRL_LO ? pr.dc1 + 4 * pr.dt1 : pr.dt1 + 4 * pr.dc1;
    constexpr int e2 = CTRL_LO ? pr.dc2 + 4 * pr.dt2 : pr.dt2 + 4 * pr.dc2;
    const double t1 = v[e1], t2 = v[e2];
    v[e1] = pr.neg ? -t2 : t2;
    v[e2] = pr.neg ? -t1 : t1;
}

// CX on a 16-register block v[dlo + 4 * dhi] of two digits; CTRL_LO: the
// control is the lower digit of the pair.
template <bool CTRL_LO>
__device__ __forceinline__ void cx_regs(double *v) {
    cx_swap<CTRL_LO, 0>(v);
    cx_swap<CTRL_LO, 1>(v);
    cx_swap<CTRL_LO, 2>(v);
    cx_swap<CTRL_LO, 3>(v);
    cx_swap<CTRL_LO, 4>(v);
    cx_swap<CTRL_LO, 5>(v);
}

template <bool LO, int Q>
__device__ __forceinline__ void u1_quad(double *v, const double (&m)[9]) {
    constexpr int iX = LO ? 1 + 4 * Q : Q + 4, iZ = LO ? 2 + 4 * Q : Q + 8, iY = LO ? 3 + 4 * Q : Q + 12;
    const double cx = v[iX], cy = v[iY], cz = v[iZ];
    v[iX] = map_row(m[0], m[1], m[2], cx, cy, cz);
    v[iY] = map_row(m[3], m[4], m[5], cx, cy, cz);
    v[iZ] = map_row(m[6], m[7], m[8], cx, cy, cz);
}

// U1 (3x3 map M over X, Y, Z) on one digit of a 16-register block; LO: the
// lower digit of the pair.
template <bool LO>
__device__ __forceinline__ void u1_regs_m(double *v, const double (&m)[9]) {
    u1_quad<LO, 0>(v, m);
    u1_quad<LO, 1>(v, m);
    u1_quad<LO, 2>(v, m);
    u1_quad<LO, 3>(v, m);
}

// Lane order of a group sweep on digits (A, B) of a 4^K-slot tile: thread u
// owns the 16-slot block whose other digits are u's bits deposited at
// pos[0..2(K-2)).  The first five positions are the first five free index
// bits (in lexicographic order of their positions) whose images under sw
// are independent modulo 32, so the 32 lanes of a half-wave hit 32
// distinct bank pairs; the other free bits follow in ascending order.  In a
// 6-digit tile a pair of digits below 5 draws the lanes from the other
// digits below 5 only, so u's bits 6 and 7 (the wave of a 256-thread sweep)
// are digit 5: each wave then reads and writes only the quarter of the tile
// whose digit 5 is its index.
struct LaneOrder {
    int pos[14];
    bool conflict_free;  // the first five positions were found
};
constexpr int gf2_rank(int *v, int n) {
    int r = 0;
    for (int bit = 0; bit < 5; ++bit) {
        int piv = -1;
        for (int i = r; i < n; ++i)
            if ((v[i] >> bit) & 1) {
                piv = i;
                break;
            }
        if (piv < 0) continue;
        const int t = v[r];
        v[r] = v[piv];
        v[piv] = t;
        for (int i = 0; i < n; ++i)
            if (i != r && ((v[i] >> bit) & 1)) v[i] ^= v[r];
        ++r;
    }
    return r;
}
template <int K, int A, int B>
constexpr LaneOrder lane_order() {
    int fr[14] = {0};
    int nf = 0;
    for (int d = 0; d < K; ++d)
        if (d != A && d != B) {
            fr[nf++] = 2 * d;
            fr[nf++] = 2 * d + 1;
        }
    LaneOrder o{};
    for (int j = 0; j < nf; ++j) o.pos[j] = fr[j];
    if (nf < 5) return o;
    // digit 5's two bits come last in fr when the pair avoids it
    const int ns = (K == 6 && B < 5) ? nf - 2 : nf;
    for (int i0 = 0; i0 < ns; ++i0)
        for (int i1 = i0 + 1; i1 < ns; ++i1)
            for (int i2 = i1 + 1; i2 < ns; ++i2)
                for (int i3 = i2 + 1; i3 < ns; ++i3)
                    for (int i4 = i3 + 1; i4 < ns; ++i4) {
                        const int idx[5] = {i0, i1, i2, i3, i4};
                        int c[5] = {0};
                        for (int k = 0; k < 5; ++k) c[k] = sw(1 << fr[idx[k]]) & 31;
                        if (gf2_rank(c, 5) < 5) continue;
                        int j = 0;
                        for (int k = 0; k < 5; ++k) o.pos[j++] = fr[idx[k]];
                        for (int f = 0; f < nf; ++f)
                            if (f != i0 && f != i1 && f != i2 && f != i3 && f != i4) o.pos[j++] = fr[f];
                        o.conflict_free = true;
                        return o;
                    }
    return o;
}

// A 64-bit value made wave-uniform.  readfirstlane returns a signed int:
// each half is widened through uint32_t, or a low half with bit 31 set
// would fill the high half with ones.
__device__ __forceinline__ uint64_t uniform_u64(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

// A 3x3 map into SGPRs by scalar loads (the map array is read-only).
typedef const __attribute__((address_space(4))) double *ConstMaps;
__device__ __forceinline__ void load_map(double (&m)[9], ConstMaps src) {
#pragma unroll
    for (int q = 0; q < 9; ++q) m[q] = src[q];
}

// Orders a wave's LDS accesses: the LDS completes a wave's instructions in
// issue order, and the fences keep the compiler from moving them.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

}  // namespace pp
