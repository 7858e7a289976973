// Record chains: sweeps over the digit pairs of a tile in LDS (see ChainOp),
// shared by the LDS-resident kernel and the 7-qubit tile passes.
#pragma once

#include "lds_tile.h"
#include "pp_device.h"

namespace pp {

constexpr int kPairs7 = 21;
template <int K>
constexpr int kNumPairs = K * (K - 1) / 2;

// sw() of the block base of lane l (wave 0) and of wave w's share, per digit
// pair a < b at index b (b - 1) / 2 + a
struct PairTable {
    uint16_t lane[kPairs7][64];
    uint16_t wave[kPairs7][16];
};

template <int K, int A, int B>
constexpr void fill_pair(PairTable &t) {
    constexpr LaneOrder lo = lane_order<K, A, B>();
    constexpr int bits = 2 * (K - 2);
    constexpr int p = B * (B - 1) / 2 + A;
    for (int l = 0; l < 64; ++l) {
        int v = 0;
        for (int q = 0; q < bits && q < 6; ++q) v |= ((l >> q) & 1) << lo.pos[q];
        t.lane[p][l] = (uint16_t)sw(v);
    }
    for (int w = 0; w < 16; ++w) {
        int v = 0;
        for (int q = 6; q < bits; ++q) v |= ((w >> (q - 6)) & 1) << lo.pos[q];
        t.wave[p][w] = (uint16_t)sw(v);
    }
    if constexpr (A + 1 < B) fill_pair<K, A + 1, B>(t);
    else if constexpr (B + 1 < K) fill_pair<K, 0, B + 1>(t);
}
template <int K>
constexpr PairTable pair_table() {
    PairTable t{};
    fill_pair<K, 0, 1>(t);
    return t;
}
template <int K>
static __device__ const PairTable kPairTable = pair_table<K>();

constexpr int kChunk = 32;                  // records staged at a time
constexpr int kChunkDoubles = kChunk * 18;  // their maps, at most two each
constexpr int kMapStride = 10;              // doubles per staged map (16-byte reads)
constexpr int kChunkSlots = kChunk * 2 * kMapStride;

__device__ __forceinline__ double lane_double(double v, int lane) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
    return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
}

template <typename T>
__device__ __forceinline__ double lds_word(unsigned byte) {
    typedef __attribute__((address_space(3))) T LT;
    return (double)*(LT *)(size_t)byte;
}
template <typename T>
__device__ __forceinline__ void lds_put(unsigned byte, double v) {
    typedef __attribute__((address_space(3))) T LT;
    *(LT *)(size_t)byte = (T)v;
}

// The sixteen addresses of a block: base XOR the words of e's bits.
__device__ __forceinline__ void block_addresses(unsigned (&ad)[16], unsigned base, const unsigned (&c)[4]) {
    ad[0] = base;
    ad[1] = ad[0] ^ c[0];
    ad[2] = ad[0] ^ c[1];
    ad[3] = ad[1] ^ c[1];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        ad[4 + e] = ad[e] ^ c[2];
        ad[8 + e] = ad[e] ^ c[3];
        ad[12 + e] = ad[4 + e] ^ c[3];
    }
}

__device__ __forceinline__ double flip(double v, unsigned sign) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    return __builtin_bit_cast(double, u ^ ((unsigned long long)sign << 32));
}

}  // namespace pp
