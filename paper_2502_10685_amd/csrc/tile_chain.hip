// Passes over 7- and 6-qubit tiles (untracked, n <= 14): persistent workgroups,
// one thread per 16 weights of a tile of 4^k weights in LDS (1,024 threads and
// 128 KiB at k = 7, 256 and 32 KiB at k = 6; doubles in FP32 circuits too, which
// are rounded once per pass), run the pass's record chain.
//
// What bounds it at k = 7: a tile's HBM traffic (256 KiB in FP64, 12.8 us of a
// CU's share of the bandwidth) and its LDS sweeps (16 waves, 1.4 us each, bound
// by the LDS pipe and the VALU in turn) take about the same time, so the two
// must overlap and both must be few.  A 7-qubit pass holds 1.5 to 1.8 times the
// gates of a 6-qubit one for the same bytes per weight.
//   - The first record is applied to the weights as they arrive from HBM (the
//     registers then hold its blocks) and the last as they leave, so two of a
//     pass's sweeps need no LDS round trip of their own.
//   - A tile's results go out, and the next tile's weights come in, in
//     quarters spread over the records of the tile between.  Stored at once,
//     every CU's 128 KiB hit the memory at the same moment and nothing else
//     ran: 9 records took 19.0 us per tile against 16.6 (13.6 without any
//     traffic).
//   - A sweep's 16 waves share four SIMDs, so its VALU instructions count:
//     maps come by scalar loads, a record ahead, as the FMAs' scalar operands.
// Random n = 12 circuits of 20,000 gates take 32.4 ms (42.8 over 6-qubit
// tiles): 67.8 us for a pass of 269 MB, 0.78 of a copy's rate, of which some 13
// are the first loads and last stores of all CUs at once.  Its waves wait 42 %
// of their cycles and issue 23 %.  One workgroup per CU leaves 128 VGPRs per
// thread: 32 for a block, 32 for the traffic, 32 for the results, 16 for
// addresses.
//
// At k = 6 four workgroups share a CU and small circuits have fewer tiles than
// that: a lone workgroup's chain of records counts (5,000 random gates at n = 8
// 0.67 ms, 0.73 when each op of a pass was decoded and swept by itself; n = 9
// 0.77, 0.85).  In large launches sweeps and traffic weigh about the same: 64
// parameter sets of 9 qubits take 103 us for the 537 MB of a pass, a copy's
// rate, and 110 for a first one, which only writes.
#include <algorithm>
#include <type_traits>

#include "chain.h"
#include "lds_tile.h"
#include "pp_device.h"
#include "tile_io.h"

namespace pp {

namespace {

template <typename T, int K>
struct TileChain {
    static constexpr int BLOCK = 1 << (2 * (K - 2));  // one thread per 16-weight block of a sweep
    static constexpr int PAIRS = kNumPairs<K>;
    static constexpr size_t OFF_LANE = (size_t)8 << (2 * K);
    static constexpr size_t OFF_WAVE = OFF_LANE + (size_t)PAIRS * 64 * 2;
    static constexpr size_t LDS = OFF_WAVE + (size_t)PAIRS * 16 * 2;
};

typedef unsigned U4 __attribute__((ext_vector_type(4)));
typedef unsigned U2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) double *GMap;

// uniform offsets of a block's letters: XOR of the words of e's bits
__device__ __forceinline__ unsigned letter_offset(const uint32_t (&c)[4], int e) {
    return ((e & 1) ? c[0] : 0u) ^ ((e & 2) ? c[1] : 0u) ^ ((e & 4) ? c[2] : 0u) ^ ((e & 8) ? c[3] : 0u);
}

// calls body with the record's kind as a constant
template <typename F>
__device__ __forceinline__ void by_kind(unsigned w, F body) {
    const unsigned kind = (w >> kChainKindShift) & 3u;
    if (kind == 3) body(std::integral_constant<int, 3>{});
    else if (kind == 1) body(std::integral_constant<int, 1>{});
    else if (kind == 2) body(std::integral_constant<int, 2>{});
    else body(std::integral_constant<int, 0>{});
}

// the words a record's block is read with, from those it is written with: the
// letters' images under its CX
__device__ __forceinline__ void read_words(unsigned (&r)[4], const unsigned (&c)[4], unsigned w) {
    const unsigned t1 = c[0] ^ c[2], t2 = c[1] ^ c[3];
    const bool lo = w & (kChainFlip6 >> 1), hi = w & kChainFlip6;  // the control
    r[0] = lo ? t1 : c[0];
    r[1] = hi ? t2 : c[1];
    r[2] = hi ? t1 : c[2];
    r[3] = lo ? t2 : c[3];
}

// START: first passes begin their weights (a template, since its code costs the
// others registers); without it they are read like any other's.
template <typename T, int K, bool START>
__global__ __launch_bounds__((TileChain<T, K>::BLOCK), 4)
void tile_chain_kernel(const TilePassDesc *__restrict__ descs, TileGroups grp) {
    using S = TileChain<T, K>;
    constexpr int SH = 3;                            // bytes of a weight in LDS
    constexpr int HSH = sizeof(T) == 8 ? 3 : 2;      // in HBM
    extern __shared__ __align__(256) unsigned char smem[];
    uint16_t *lanetab = reinterpret_cast<uint16_t *>(smem + S::OFF_LANE);
    uint16_t *wavetab = reinterpret_cast<uint16_t *>(smem + S::OFF_WAVE);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    typedef __attribute__((address_space(3))) unsigned char LB;
    const unsigned tile0 = (unsigned)(size_t)(LB *)smem;
    const int total = grp.first_block[grp.ngroups];
    int blk = blockIdx.x;
    if (blk >= total) return;
    for (int i = tid; i < S::PAIRS * 64; i += S::BLOCK) lanetab[i] = (&kPairTable<K>.lane[0][0])[i];
    for (int i = tid; i < S::PAIRS * 16; i += S::BLOCK) wavetab[i] = (&kPairTable<K>.wave[0][0])[i];

    auto word = [](unsigned v, int i) { return (unsigned)__builtin_amdgcn_readlane((int)v, i); };
    // swizzled slot of this thread's block of pair p
    auto block_slot = [&](unsigned p) -> unsigned { return lanetab[p * 64 + lane] ^ wavetab[p * 16 + wave]; };
    // byte offset in HBM of this thread's block of pair p
    auto block_voff = [&](unsigned p, uint64_t qubits) {
        const unsigned i = (unsigned)sw((int)block_slot(p));  // sw is its own inverse
        unsigned v = 0;
#pragma unroll
        for (int j = 0; j < K; ++j)
            v |= ((i >> (2 * j)) & 3u) << (2u * (unsigned)((qubits >> (8 * j)) & 0xff));
        return v * (unsigned)sizeof(T);
    };
    // the records of a pass, one per lane (at most kTileRecords): word and map
    // in R0, write words in R1
    U2 R0;
    U4 R1;
    auto load_records = [&](const TilePassDesc *d) {
        const int l = lane < d->nrec ? lane : 0;
        const unsigned __attribute__((address_space(1))) *g = (const unsigned __attribute__((address_space(1))) *)d->chain + 12 * l;
        R0 = *(const U2 __attribute__((address_space(1))) *)g;
        R1 = *(const U4 __attribute__((address_space(1))) *)(g + 8);
    };
    // a record's first map; one without maps gets any (behind the last map
    // there is nothing to read)
    auto first_map = [](double (&m)[9], const TilePassDesc *d, unsigned map) {
        const unsigned last = d->nmaps > 0 ? d->nmaps - 1 : 0;
        load_map(m, (ConstMaps)d->maps + 9ull * (map < last ? map : last));
    };
    // the signs of a record's CX and its maps on its block, for kind KIND: m1
    // the first map, the second (kind 3) at m2
    auto apply = [](auto kind_c, double (&v)[16], unsigned w, const double (&m1)[9], ConstMaps m2) {
        constexpr int KIND = decltype(kind_c)::value;
        v[6] = flip(v[6], w & kChainFlip6);
        v[9] = flip(v[9], (w << 1) & kChainFlip6);
        v[15] = flip(v[15], (w << 2) & kChainFlip6);
        if constexpr (KIND & 1) u1_regs_m<true>(v, m1);
        if constexpr (KIND == 2) u1_regs_m<false>(v, m1);
        if constexpr (KIND == 3) {
            double m[9];
            load_map(m, m2);
            u1_regs_m<false>(v, m);
        }
    };

    // the same with a branch per map, for the records next to HBM: their loads
    // and stores stay outside the branches (see arrived)
    auto apply_branched = [&](double (&v)[16], unsigned w, const double (&m1)[9], ConstMaps m2) {
        const unsigned kind = (w >> kChainKindShift) & 3u;
        v[6] = flip(v[6], w & kChainFlip6);
        v[9] = flip(v[9], (w << 1) & kChainFlip6);
        v[15] = flip(v[15], (w << 2) & kChainFlip6);
        if (kind & 1u) u1_regs_m<true>(v, m1);
        if (kind & 2u) {
            double m[9];
            load_map(m, kind == 2 ? m2 - 9 : m2);
            u1_regs_m<false>(v, m);
        }
    };

    TileBase cur = tile_base<K>(descs, grp, blk);
    load_records(cur.d);
    lds_barrier();
    // io holds, in turn, a tile's weights as they come from HBM, the results
    // of the tile before on their way out, and the next tile's weights
    T io[16];
    {
        const __amdgpu_buffer_rsrc_t rs =
            tile_rsrc(reinterpret_cast<T *>(cur.d->coef) + cur.base, START && cur.d->start != nullptr);
        const unsigned vo = block_voff(word(R0.x, 0) & 0xffu, cur.d->qubits);
        const uint32_t c[4] = {cur.d->in[0], cur.d->in[1], cur.d->in[2], cur.d->in[3]};
#pragma unroll
        for (int e = 0; e < 16; ++e) io[e] = BufIO<T>::ld(rs, vo, letter_offset(c, e));
    }
    double m1[9];
    first_map(m1, cur.d, word(R0.y, 0));
    // Waits for a tile's records and weights are placed here and at the end of
    // the loop, in straight-line code: behind the kinds' branches the compiler
    // would put them into the record loop too.
    auto arrived = [&] {
        __asm__ volatile("" : "+v"(R0), "+v"(R1));
#pragma unroll
        for (int e = 0; e < 16; ++e) __asm__ volatile("" : "+v"(io[e]));
    };
    arrived();
    T res[16];              // results of the tile before
    T *pbase = nullptr;     // its first slot in HBM
    unsigned pvo = 0;       // this thread's byte offset there
    uint32_t po[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < 16; ++e) res[e] = (T)0;
    // The weights of a tile of a half's first pass, whose loads gave 0: the
    // state's, or the observable's strings in input order.  Filled and
    // scattered by kernels before it and read back they cost 7 us at n = 8, two
    // passes over both arrays in large sweeps (300 sets at n = 9 6.28 ms, 6.04
    // without), and 5,000 gates at n = 10 took 1.25 ms, 1.18 without.
    auto begin = [&](const TileStart *st) {
        const unsigned vs = block_voff(word(R0.x, 0) & 0xffu, cur.d->qubits) >> HSH;  // slots, not bytes
        const uint32_t c[4] = {cur.d->in[0] >> HSH, cur.d->in[1] >> HSH, cur.d->in[2] >> HSH, cur.d->in[3] >> HSH};
        const unsigned xbits = 0x55555555u;
        if (cur.d->forward) {
            const bool z = (((unsigned)cur.base | vs) & xbits) == 0;
#pragma unroll
            for (int e = 0; e < 16; ++e) io[e] = z && (letter_offset(c, e) & xbits) == 0 ? (T)1 : (T)0;
            return;
        }
        unsigned inside = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) inside |= 3u << (2u * (unsigned)((cur.d->qubits >> (8 * j)) & 0xff));
        const int l = lane < st->nterms ? lane : 0;
        const unsigned slot = (unsigned)morton_slot(st->obs_x[l], st->obs_z[l], cur.d->n);
        const double coef = st->obs_c[l];
        uint64_t here = __ballot(lane < st->nterms && (slot & ~inside) == (unsigned)cur.base);
        while (here) {
            const int t = __builtin_ctzll(here);
            here &= here - 1;
            const unsigned at = word(slot, t) & inside;
            const double v = lane_double(coef, t);
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if ((vs ^ letter_offset(c, e)) == at) io[e] = (T)((double)io[e] + v);
        }
    };
    for (;;) {
        const int nrec = cur.d->nrec;
        const ConstMaps gmaps = (ConstMaps)cur.d->maps;
        if constexpr (START)
            if (cur.d->start) begin(cur.d->start);
        // ---- the first record, on the weights from HBM
        {
            const unsigned w = word(R0.x, 0), map = word(R0.y, 0);
            const unsigned at = tile0 + (block_slot(w & 0xffu) << SH);
            double v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = (double)io[e];
            apply_branched(v, w, m1, gmaps + 9ull * (map + 1));
            first_map(m1, cur.d, word(R0.y, 1));
            unsigned ad[16];
            const unsigned c[4] = {word(R1.x, 0), word(R1.y, 0), word(R1.z, 0), word(R1.w, 0)};
            block_addresses(ad, at, c);
#pragma unroll
            for (int e = 0; e < 16; ++e) lds_put<double>(ad[e], v[e]);
        }
        // ---- the tile before goes out and the next one comes in, a quarter
        // at a time through the same registers, spread over the records
        const int nblk = blk + gridDim.x;
        const bool has_next = nblk < total, has_prev = pbase != nullptr;
        TileBase nxt = cur;
        unsigned nmap = 0;   // the next tile's first map
        double touch = 0.0;  // brings its maps into L2 ahead of the scalar loads
        T *nbase = nullptr;
        bool nstart = false;
        unsigned nvo = 0;
        uint32_t ni[4] = {0u, 0u, 0u, 0u};
        if (has_next) {
            nxt = tile_base<K>(descs, grp, nblk);
            typedef const __attribute__((address_space(4))) uint32_t *CW;
            const CW first = (CW)nxt.d->chain;  // word and map of its first record
            nbase = reinterpret_cast<T *>(nxt.d->coef) + nxt.base;
            nstart = START && nxt.d->start != nullptr;
            nvo = block_voff(first[0] & 0xffu, nxt.d->qubits);
#pragma unroll
            for (int q = 0; q < 4; ++q) ni[q] = nxt.d->in[q];
            nmap = first[1];
            if (9 * (int)nmap + tid < 9 * (int)nxt.d->nmaps)
                touch = ((GMap)nxt.d->maps)[9 * (int)nmap + tid];
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) io[e] = res[e];
        auto io_out = [&](auto q_c) {
            constexpr int q = 4 * decltype(q_c)::value;
            if (!has_prev) return;
            const __amdgpu_buffer_rsrc_t rs = tile_rsrc(pbase);
#pragma unroll
            for (int e = q; e < q + 4; ++e) BufIO<T>::st(rs, pvo, letter_offset(po, e), io[e]);
        };
        auto io_in = [&](auto q_c) {
            constexpr int q = 4 * decltype(q_c)::value;
            if (!has_next) return;
            const __amdgpu_buffer_rsrc_t rs = tile_rsrc(nbase, nstart);
#pragma unroll
            for (int e = q; e < q + 4; ++e) io[e] = BufIO<T>::ld(rs, nvo, letter_offset(ni, e));
        };
        // ---- the records between, in LDS
        lds_barrier();
        unsigned w = word(R0.x, 1), slot = block_slot(w & 0xffu);
        int r = 1;
        auto records = [&](int end) {
#pragma unroll 1
            for (; r < end; ++r) {
                const unsigned map = word(R0.y, r), next_map = word(R0.y, r + 1);
                const unsigned c[4] = {word(R1.x, r), word(R1.y, r), word(R1.z, r), word(R1.w, r)};
                by_kind(w, [&](auto kind) {
                    double v[16];
                    {
                        unsigned ra[16], rc[4];
                        read_words(rc, c, w);
                        block_addresses(ra, tile0 + (slot << SH), rc);
#pragma unroll
                        for (int e = 0; e < 16; ++e) v[e] = lds_word<double>(ra[e]);
                    }
                    apply(kind, v, w, m1, gmaps + 9ull * (map + 1));
                    first_map(m1, cur.d, next_map);
                    unsigned wa[16];
                    block_addresses(wa, tile0 + (slot << SH), c);
#pragma unroll
                    for (int e = 0; e < 16; ++e) lds_put<double>(wa[e], v[e]);
                });
                if (K == 6 && ((w >> kChainNoBarrierBit) & 1u)) wave_lds_order();
                else lds_barrier();
                w = word(R0.x, r + 1);
                slot = block_slot(w & 0xffu);
            }
        };
        using Q0 = std::integral_constant<int, 0>;
        using Q1 = std::integral_constant<int, 1>;
        using Q2 = std::integral_constant<int, 2>;
        using Q3 = std::integral_constant<int, 3>;
        io_out(Q0{});
        io_out(Q1{});
        records(1 + (nrec - 2) / 4);
        io_out(Q2{});
        io_out(Q3{});
        records(1 + (nrec - 2) / 2);
        __asm__ volatile("" ::"v"(touch));
        io_in(Q0{});
        io_in(Q1{});
        records(1 + 3 * (nrec - 2) / 4);
        io_in(Q2{});
        io_in(Q3{});
        records(nrec - 1);
        // ---- the last record, on its way to HBM
        {
            const unsigned c[4] = {word(R1.x, r), word(R1.y, r), word(R1.z, r), word(R1.w, r)};
            const unsigned map = word(R0.y, r);
            pbase = reinterpret_cast<T *>(cur.d->coef) + cur.base;
            pvo = block_voff(w & 0xffu, cur.d->qubits);
#pragma unroll
            for (int q = 0; q < 4; ++q) po[q] = cur.d->out[q];
            double v[16];
            {
                unsigned ra[16], rc[4];
                read_words(rc, c, w);
                block_addresses(ra, tile0 + (slot << SH), rc);
#pragma unroll
                for (int e = 0; e < 16; ++e) v[e] = lds_word<double>(ra[e]);
            }
            apply_branched(v, w, m1, gmaps + 9ull * (map + 1));
            first_map(m1, nxt.d, nmap);
            load_records(nxt.d);
#pragma unroll
            for (int e = 0; e < 16; ++e) res[e] = (T)v[e];
            if (!has_next) break;
            lds_barrier();  // every wave has read this tile
            arrived();
        }
        blk = nblk;
        cur = nxt;
    }
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(pbase);
#pragma unroll
    for (int e = 0; e < 16; ++e) BufIO<T>::st(rs, pvo, letter_offset(po, e), res[e]);
}

template <typename T, int K, bool START>
hipError_t launch_tile_chain_t(const TilePassDesc *d, const TileGroups &grp, hipStream_t s) {
    using S = TileChain<T, K>;
    static_assert(S::LDS <= 160 * 1024, "a tile and the pair tables fit one CU's LDS");
    auto fn = tile_chain_kernel<T, K, START>;
    static int resident = 0;
    if (!resident) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
        if (e != hipSuccess) return e;
        int per_cu = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)fn, S::BLOCK, S::LDS);
        if (e != hipSuccess) return e;
        resident = std::max(per_cu, 1) * num_cus();
    }
    const int nblocks = grp.first_block[grp.ngroups];
    hipLaunchKernelGGL(fn, dim3(std::min(nblocks, resident)), dim3(S::BLOCK), S::LDS, s, d, grp);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_tile_chain_k(const TilePassDesc *d, const TileGroups &grp, int k, hipStream_t s) {
    if (k == 6) return grp.start ? launch_tile_chain_t<T, 6, true>(d, grp, s) : launch_tile_chain_t<T, 6, false>(d, grp, s);
    return grp.start ? launch_tile_chain_t<T, 7, true>(d, grp, s) : launch_tile_chain_t<T, 7, false>(d, grp, s);
}

}  // namespace

hipError_t launch_tile_chain(const TilePassDesc *d_descs, const TileGroups &grp, int k, int dtype_bytes,
                             hipStream_t s) {
    return dtype_bytes == 8 ? launch_tile_chain_k<double>(d_descs, grp, k, s)
                            : launch_tile_chain_k<float>(d_descs, grp, k, s);
}

}  // namespace pp
