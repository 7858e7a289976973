// HBM access of the persistent tile-pass kernels: which tile a block number
// means, and buffer loads and stores of its weights.
#pragma once

#include "pp_device.h"

namespace pp {

// Weights are read and written with buffer instructions: one resource per
// tile (base = the tile's first slot), the lane's slot offset in a VGPR and
// the register's in an SGPR, so the 64 accesses of a lane need no address
// registers.  Both offsets are below 2^31 bytes when the tile's qubits are
// all below 14 (the launcher only picks this kernel for n <= 14).  Every
// weight is read once and written once per pass, so both carry the
// non-temporal hint (nt): the streamed array then does not push the op
// lists and maps, which every tile re-reads, out of L2.
// empty: loads give 0 and touch nothing
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(void *p, bool empty = false) {
    return __builtin_amdgcn_make_buffer_rsrc(p, (short)0, empty ? 0 : -1, 0x00020000);
}
// cache-policy operand of the buffer builtins: bit 1 is nt on gfx950
constexpr int kNonTemporal = 2;
template <typename T>
struct BufIO;
template <>
struct BufIO<double> {
    typedef unsigned V __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ double ld(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, kNonTemporal));
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, double v) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, vo, so, kNonTemporal);
    }
};
template <>
struct BufIO<float> {
    static __device__ __forceinline__ float ld(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, kNonTemporal));
    }
    static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, unsigned vo, unsigned so, float v) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, vo, so, kNonTemporal);
    }
};

struct TileBase {
    const TilePassDesc *d;
    long long base;  // first slot of the tile
};

template <int K>
__device__ __forceinline__ TileBase tile_base(const TilePassDesc *__restrict__ descs, const TileGroups &grp, int b) {
    int g = 0;
    while (g + 1 < grp.ngroups && b >= grp.first_block[g + 1]) ++g;
    const int rel = b - grp.first_block[g];
    const TilePassDesc *d = descs + grp.first_desc[g] + (rel >> grp.shift[g]);
    const long long tile = rel & ((1 << grp.shift[g]) - 1);
    const uint64_t qubits = d->qubits;
    const int n = d->n;
    unsigned inmask = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j < K) inmask |= 1u << (unsigned)((qubits >> (8 * j)) & 0xff);
    // the tile index's digits go to the qubits outside the tile, lowest
    // first: one step per outside qubit
    long long base = 0, t = tile;
    unsigned out = ~inmask & ((1u << n) - 1u);
    while (out) {
        const int q = __builtin_ctz(out);
        out &= out - 1u;
        base |= (t & 3ll) << (2 * q);
        t >>= 2;
    }
    return TileBase{d, base};
}

}  // namespace pp
