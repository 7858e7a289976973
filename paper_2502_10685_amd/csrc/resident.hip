// LDS-resident circuits (n <= 7, untracked): one workgroup holds all 4^n
// weights in LDS and runs a chain of sweeps over digit pairs.  They are doubles
// there for FP32 circuits too, rounded where they leave the chip: a sweep ends
// with every record, and rounding each time left the density matrices of 2
// qubits 1.9 times and random circuits of 3 to 6 qubits 1.05 to 1.13 times as
// far off as whole groups of gates between roundings.
//
// What bounds it: the chain.  A circuit's sweeps depend on each other, one
// circuit occupies one or two CUs, and a lone wave issues at most one
// instruction per four cycles and pays some sixty cycles for each branch it
// takes, so the time of a sweep is its instruction count plus the LDS round
// trip it cannot hide.  Hence:
//   - one code path for every digit pair and CX: the 16 letters of a block
//     are read at a base XOR combinations of four uniform words and written
//     at a base XOR combinations of four others, all eight given by the
//     record.  CX permutes the letters linearly (over GF(2)), so it is only
//     another set of words to read with, and three sign flips;
//   - while a block's reads are in flight the wave computes where to write it
//     and where to read the next one;
//   - records and 3x3 maps are staged a chunk ahead: records in registers
//     (one per lane), maps through a double-buffered LDS copy.  Maps are
//     stored in record order, so a chunk is one contiguous piece.
// A record with a CX and two maps takes 0.50 us at n <= 5, 0.70 at n = 6 and
// 1.6 at n = 7, where 16 waves keep the LDS pipe busy two thirds of the time.
// (Code compiled per digit pair and group shape, whose footprint and branches
// a lone workgroup cannot hide, took 1.4, 0.93 and 1.8 us per group.)
//
// An evaluation runs from both ends: <O> = sum_P c(P) r(P) with c the
// observable's weights taken back to some gate in the middle and r(P) =
// Tr(P rho) the state's Pauli coefficients taken forward to it (the density
// operator as a sum over Pauli strings, eqs. (2)-(3); both run through the
// same orthogonal maps).  The halves are independent until the final product,
// so they run side by side: two waves of one workgroup for n <= 5, two
// workgroups above, where the one that ends last reads the other's vector.
#include <algorithm>
#include <type_traits>

#include "chain.h"
#include "lds_tile.h"
#include "pp_device.h"

namespace pp {

namespace {

template <typename T, int N>
struct ChainShape {
    static constexpr int K = N < 2 ? 2 : N;  // a one-qubit circuit leaves digit 1 at I
    static constexpr int SIZE = 1 << (2 * K);
    static constexpr int NG = 1 << (2 * (K - 2));
    static constexpr int W = NG > 64 ? NG / 64 : 1;  // waves of one direction
    static constexpr bool BOTH = K <= 5;             // both directions in one workgroup
    static constexpr int DIRS = BOTH ? 2 : 1;
    static constexpr int BLOCK = 64 * W * DIRS;
    static constexpr int NP = kNumPairs<K>;
    // dynamic LDS: the tiles first (their addresses are XORed, so they are
    // aligned to their size), then the staged maps, the pair table, reductions
    static constexpr int MAPS = 2 * kChunkSlots + 3 * kMapStride;  // reads of absent maps may run past a chunk
    static constexpr size_t OFF_MAPS = (size_t)DIRS * SIZE * 8 < 256 ? 256 : (size_t)DIRS * SIZE * 8;
    static constexpr size_t OFF_LANE = OFF_MAPS + (size_t)DIRS * MAPS * 8;
    static constexpr size_t OFF_WAVE = OFF_LANE + (size_t)NP * 64 * 2;
    static constexpr size_t OFF_RED = (OFF_WAVE + (size_t)NP * 16 * 2 + 15) & ~(size_t)15;
    static constexpr size_t LDS = OFF_RED + (size_t)(BLOCK / 64 + 2) * 8;
};

// Runs records [0, nrec) on the tile at LDS byte address `tile`.  tid: the
// thread's index among the 64 W threads of its direction, lane = tid & 63.
//
// A record's maps: with up to four waves (n <= 6) broadcast reads behind the
// block's own (the LDS pipe has room, and 26 fewer instructions issue); the
// sixteen waves of n = 7, which fill the pipe, take one read a record ahead
// that puts an element in each lane, then move it to SGPRs.  At n = 6 the
// reads take 0.70 us per record and the moves 0.74.
template <typename T, int N>
__device__ __forceinline__ void run_chain(unsigned tile, double *mapbuf, const uint16_t *lanetab,
                                          const uint16_t *wavetab, const ChainOp *__restrict__ recs, int nrec,
                                          const double *__restrict__ maps, int nmaps, int tid) {
    using S = ChainShape<T, N>;
    constexpr int TPD = 64 * S::W;
    constexpr int SPT = (kChunkDoubles + TPD - 1) / TPD;
    constexpr int SH = 3;
    constexpr bool SCALAR = S::W > 4;
    typedef unsigned U4 __attribute__((ext_vector_type(4)));
    typedef double D2 __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(1))) U4 *GRec;
    typedef const __attribute__((address_space(1))) double *GMap;
    if (nrec <= 0) return;
    const GRec grec = (GRec)recs;
    const GMap gmap = (GMap)maps;
    const int lane = tid & 63, wave = tid >> 6;
    const int mend = 9 * nmaps;
    // element of a record's maps that this lane reads: lanes 0..8 the lower
    // digit's map, lanes 32..40 the higher digit's
    const int moff = (lane & 31) < 9 ? (lane & 31) : 0;
    const int mhi = lane >= 32 ? kMapStride : 0;
    // map element i of a chunk goes to its map's kMapStride-double slot
    auto slot = [](int i) { return i + (kMapStride - 9) * (i / 9); };

    // records of the chunk, kChunk lanes each: word and map in R0; the words
    // to read with in the lower lanes of R1, those to write with in the upper
    static_assert(kChunk == 32, "two groups of lanes");
    const int rl = lane & (kChunk - 1), part = 1 + lane / kChunk;
    U4 R0 = {0u, 0u, 0u, 0u}, R1 = R0;
    double stage[SPT];
    if (rl < nrec) {
        R0 = grec[3 * rl];
        R1 = grec[3 * rl + part];
    }
    auto word = [&](unsigned v, int i) { return (unsigned)__builtin_amdgcn_readlane((int)v, i); };
    int mb = (int)word(R0.y, 0);  // first map of the chunk
#pragma unroll
    for (int j = 0; j < SPT; ++j) {
        const int i = tid + j * TPD;
        stage[j] = (i < kChunkDoubles && 9 * mb + i < mend) ? gmap[9 * mb + i] : 0.0;
    }
    int buf = 1;
    for (int c0 = 0; c0 < nrec; c0 += kChunk) {
        const int cn = nrec - c0 < kChunk ? nrec - c0 : kChunk;
        buf ^= 1;
        double *mbuf = mapbuf + buf * kChunkSlots;
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
            const int i = tid + j * TPD;
            if (i < kChunkDoubles) mbuf[slot(i)] = stage[j];
        }
        if constexpr (S::W > 1) lds_barrier();
        else wave_lds_order();
        const bool more = c0 + cn < nrec;
        U4 N0 = {0u, 0u, 0u, 0u}, N1 = N0;
        int mbn = mb;
        if (more) {
            if (c0 + kChunk + rl < nrec) {
                N0 = grec[3 * (c0 + kChunk + rl)];
                N1 = grec[3 * (c0 + kChunk + rl) + part];
            }
            const unsigned lw = word(R0.x, cn - 1);
            mbn = (int)(word(R0.y, cn - 1) + ((lw >> kChainKindShift) & 1u) + ((lw >> (kChainKindShift + 1)) & 1u));
#pragma unroll
            for (int j = 0; j < SPT; ++j) {
                const int i = tid + j * TPD;
                stage[j] = (i < kChunkDoubles && 9 * mbn + i < mend) ? gmap[9 * mbn + i] : 0.0;
            }
        }
        // block base of record i (from its word), and with SCALAR its maps
        auto pair_base = [&](unsigned w, unsigned &sl, unsigned &sv) {
            const unsigned p = w & 0xffu;
            sl = lanetab[p * 64 + lane];
            sv = 0;
            if constexpr (S::W > 1) sv = wavetab[p * 16 + wave];
        };
        auto lane_maps = [&](int i, unsigned w) {
            const int m0 = (int)word(R0.y, i) - mb;
            return mbuf[kMapStride * m0 + moff + ((w >> kChainKindShift) & 1u ? mhi : 0)];
        };
        auto clamp = [&](int i) { return i < cn ? i : cn - 1; };
        // ra: where record i's block is read; base: its block base; wn, sl,
        // sv: the next record's word and base, one read ahead
        unsigned w = word(R0.x, 0), sl, sv, ra[16];
        pair_base(w, sl, sv);
        unsigned base = tile + ((sl ^ sv) << SH);
        {
            const unsigned c[4] = {word(R1.x, 0), word(R1.y, 0), word(R1.z, 0), word(R1.w, 0)};
            block_addresses(ra, base, c);
        }
        unsigned wn = word(R0.x, clamp(1));
        pair_base(wn, sl, sv);
        double mv = 0.0, mvn = 0.0;
        if constexpr (SCALAR) mv = lane_maps(0, w);
#pragma unroll 1
        for (int i = 0; i < cn; ++i) {
            // One body per kind of record, from the reads to the writes, so
            // that no weight crosses a branch (merged paths copied them).
            auto body = [&](auto kind_c) {
                constexpr int KIND = decltype(kind_c)::value;
                double v[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) v[e] = lds_word<double>(ra[e]);
                // where the next block is; the base of the one behind it
                const unsigned here = base;
                const int n1 = clamp(i + 1);
                base = tile + ((sl ^ sv) << SH);
                const unsigned w2 = word(R0.x, clamp(i + 2));
                pair_base(w2, sl, sv);
                if constexpr (SCALAR) mvn = lane_maps(n1, wn);
                // eight of a map's nine elements in pairs (the ninth alone:
                // the unused half of a fifth pair made the compiler wait
                // before it reused the register)
                D2 ml[4], mh[4];
                double ml8 = 0.0, mh8 = 0.0;
                if constexpr (!SCALAR && KIND != 0) {
                    const double *src = mbuf + kMapStride * ((int)word(R0.y, i) - mb);
                    if constexpr (KIND & 1) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) ml[q] = reinterpret_cast<const D2 *>(src)[q];
                        ml8 = src[8];
                        src += kMapStride;
                    }
                    if constexpr (KIND & 2) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) mh[q] = reinterpret_cast<const D2 *>(src)[q];
                        mh8 = src[8];
                    }
                }
                // every read is on its way before anything is computed (not
                // at n = 7, whose 1,024 threads have 128 registers each)
                if constexpr (!SCALAR) __builtin_amdgcn_sched_barrier(0);
                unsigned wa[16];
                {
                    const int u = i + kChunk;
                    const unsigned c[4] = {word(R1.x, u), word(R1.y, u), word(R1.z, u), word(R1.w, u)};
                    block_addresses(wa, here, c);
                }
                {
                    const unsigned c[4] = {word(R1.x, n1), word(R1.y, n1), word(R1.z, n1), word(R1.w, n1)};
                    block_addresses(ra, base, c);
                }
                if constexpr (!SCALAR) __builtin_amdgcn_sched_barrier(0);
                v[6] = flip(v[6], w & kChainFlip6);
                v[9] = flip(v[9], (w << 1) & kChainFlip6);
                v[15] = flip(v[15], (w << 2) & kChainFlip6);
                if constexpr (KIND & 1) {
                    double m[9];
#pragma unroll
                    for (int q = 0; q < 9; ++q) m[q] = SCALAR ? lane_double(mv, q) : (q < 8 ? ml[q >> 1 & 3][q & 1] : ml8);
                    u1_regs_m<true>(v, m);
                }
                if constexpr (KIND & 2) {
                    double m[9];
#pragma unroll
                    for (int q = 0; q < 9; ++q) m[q] = SCALAR ? lane_double(mv, 32 + q) : (q < 8 ? mh[q >> 1 & 3][q & 1] : mh8);
                    u1_regs_m<false>(v, m);
                }
                // every read of this record is taken before its writes go
                // out, so that nothing waits for the writes
                __asm__ volatile("" : "+v"(sl), "+v"(sv));
                if constexpr (SCALAR) {
                    mv = mvn;
                    __asm__ volatile("" : "+v"(mv));
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) lds_put<double>(wa[e], v[e]);
                wn = w2;
            };
            const unsigned wi = w;
            const unsigned kind = (w >> kChainKindShift) & 3u;
            const unsigned wnext = wn;
            if (__builtin_expect(kind == 3, 1)) body(std::integral_constant<int, 3>{});
            else if (kind == 1) body(std::integral_constant<int, 1>{});
            else if (kind == 2) body(std::integral_constant<int, 2>{});
            else body(std::integral_constant<int, 0>{});
            w = wnext;
            if (S::W == 1 || ((wi >> kChainNoBarrierBit) & 1u)) wave_lds_order();
            else lds_barrier();
        }
        R0 = N0;
        R1 = N1;
        mb = mbn;
    }
}

// meet: both directions and the product; otherwise the observable's records
// alone (the plan then has no others), with the readout of the I/Z strings
// and the final weights on request.  out: the one circuit's result, or
// nullptr (each descriptor's own).
template <typename T, int N>
__global__ __launch_bounds__((ChainShape<T, N>::BLOCK))
void chain_kernel(const ResidentDesc *__restrict__ descs, int meet, double *out) {
    using S = ChainShape<T, N>;
    constexpr int TPD = 64 * S::W;
    extern __shared__ __align__(256) unsigned char smem[];
    const int split = !S::BOTH && meet;  // two workgroups per circuit
    const ResidentDesc &d = descs[split ? blockIdx.x >> 1 : blockIdx.x];
    const int tid = threadIdx.x;
    const int dir = S::BOTH ? __builtin_amdgcn_readfirstlane(tid / TPD) : (split ? (int)(blockIdx.x & 1) : 0);
    const int slot = S::BOTH ? dir : 0;
    const int t = S::BOTH ? tid % TPD : tid;
    double *lc = reinterpret_cast<double *>(smem) + slot * S::SIZE;
    double *mapbuf = reinterpret_cast<double *>(smem + S::OFF_MAPS) + slot * S::MAPS;
    uint16_t *lanetab = reinterpret_cast<uint16_t *>(smem + S::OFF_LANE);
    uint16_t *wavetab = reinterpret_cast<uint16_t *>(smem + S::OFF_WAVE);
    double *red = reinterpret_cast<double *>(smem + S::OFF_RED);

    for (int i = tid; i < S::NP * 64; i += S::BLOCK) lanetab[i] = (&kPairTable<S::K>.lane[0][0])[i];
    for (int i = tid; i < S::NP * 16; i += S::BLOCK) wavetab[i] = (&kPairTable<S::K>.wave[0][0])[i];
    for (int i = t; i < S::SIZE; i += TPD) lc[i] = 0.0;
    lds_barrier();
    if (dir == 1) {  // |0...0>: Tr(P rho) = 1 for the strings of I and Z
        for (int j = t; j < (1 << N); j += TPD) lc[sw((int)zonly_slot(j, N))] = 1.0;
    } else if (d.coef_in) {
        const T *in = reinterpret_cast<const T *>(d.coef_in);
        for (int i = t; i < (1 << (2 * N)); i += TPD) lc[sw(i)] = in[i];
    } else if (d.distinct || t == 0) {
        // repeated strings are summed in input order by one thread
        for (int k = t; k < d.nterms; k += d.distinct ? TPD : 1) {
            const int s = sw((int)morton_slot(d.obs_x[k], d.obs_z[k], N));
            lc[s] += d.obs_c[k];
        }
    }
    lds_barrier();
    const int nrec = dir == 0 ? d.nchain : (meet ? d.nchain_fwd : 0);
    typedef __attribute__((address_space(3))) double LT;
    run_chain<T, N>((unsigned)(size_t)(LT *)lc, mapbuf, lanetab, wavetab, d.chain + (dir == 0 ? 0 : d.nchain), nrec,
                    d.maps, d.nmaps, t);
    lds_barrier();

    double *res = out ? out : d.expval_out;
    double part = 0.0;
    if (!meet) {
        if (dir == 0) {
            for (int j = t; j < (1 << N); j += TPD) part += lc[sw((int)zonly_slot(j, N))];
            if (d.coef_out) {
                T *o = reinterpret_cast<T *>(d.coef_out);
                for (int i = t; i < (1 << (2 * N)); i += TPD) o[i] = (T)lc[sw(i)];
            }
        }
    } else if constexpr (S::BOTH) {
        const double *c = reinterpret_cast<const double *>(smem), *r = c + S::SIZE;
        for (int i = tid; i < S::SIZE; i += S::BLOCK) part += c[i] * r[i];
    } else {
        // each workgroup publishes its vector; the one that arrives second
        // multiplies the two (the product and its order do not depend on
        // which one that is).  Agent-scope stores and loads pass the L2 by,
        // so nothing has to be written back: with a __threadfence() of every
        // wave instead, each a write-back of the whole L2, 46 parameter sets
        // of 7 qubits and 7 layers in FP32 took 108 us, not 55.
        // The order rests on the kind of these accesses, not on the language's
        // rules: a relaxed agent-scope store is written through (sc1) and
        // acknowledged where every XCD sees it, which s_waitcnt vmcnt(0) waits
        // for before the ticket is taken, and the loads behind the ticket look
        // there.  A plain store of something else to be read by the other
        // workgroup would not be covered and needs a release.  The plain
        // reset of the ticket is ordered by the end of the kernel.
        T *mine = reinterpret_cast<T *>(d.xbuf) + dir * S::SIZE;
        const T *theirs = reinterpret_cast<const T *>(d.xbuf) + (1 - dir) * S::SIZE;
        for (int i = tid; i < S::SIZE; i += S::BLOCK)
            __hip_atomic_store(mine + i, (T)lc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's stores are at the agent's point of coherence
        __syncthreads();
        unsigned *flag = reinterpret_cast<unsigned *>(red + S::BLOCK / 64 + 1);
        if (tid == 0) *flag = __hip_atomic_fetch_add(d.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (*flag == 0u) return;
        constexpr int PER = S::SIZE / S::BLOCK;
        T v[PER];  // all in flight at once
#pragma unroll
        for (int j = 0; j < PER; ++j)
            v[j] = __hip_atomic_load(theirs + tid + j * S::BLOCK, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < PER; ++j) part += (double)(T)lc[tid + j * S::BLOCK] * (double)v[j];
        if (tid == 0) *d.ticket = 0u;  // for the next launch
    }
    const double total = block_sum_d<S::BLOCK>(part, red);
    if (tid == 0) *res = total;
}

template <typename T, int N>
hipError_t launch_chain_t(const ResidentDesc *d, int nd, bool meet, double *out, hipStream_t s) {
    using S = ChainShape<T, N>;
    static_assert(S::LDS <= 160 * 1024, "the tiles and the staged maps share one CU's LDS");
    auto fn = chain_kernel<T, N>;
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
        if (e != hipSuccess) return e;
        attr = true;
    }
    const int grid = (!S::BOTH && meet) ? 2 * nd : nd;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(S::BLOCK), S::LDS, s, d, (int)meet, out);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_chain_n(const ResidentDesc *d, int nd, int n, bool meet, double *out, hipStream_t s) {
    switch (n) {
    case 1: return launch_chain_t<T, 1>(d, nd, meet, out, s);
    case 2: return launch_chain_t<T, 2>(d, nd, meet, out, s);
    case 3: return launch_chain_t<T, 3>(d, nd, meet, out, s);
    case 4: return launch_chain_t<T, 4>(d, nd, meet, out, s);
    case 5: return launch_chain_t<T, 5>(d, nd, meet, out, s);
    case 6: return launch_chain_t<T, 6>(d, nd, meet, out, s);
    default: return launch_chain_t<T, 7>(d, nd, meet, out, s);
    }
}

}  // namespace

hipError_t launch_chain(const ResidentDesc *d_descs, int ndescs, int n, int dtype_bytes, bool meet, double *out,
                        hipStream_t s) {
    if (ndescs <= 0) return hipSuccess;
    if (n < 1 || n > 7 || (out && ndescs != 1)) return hipErrorInvalidValue;
    return dtype_bytes == 8 ? launch_chain_n<double>(d_descs, ndescs, n, meet, out, s)
                            : launch_chain_n<float>(d_descs, ndescs, n, meet, out, s);
}

size_t chain_exchange_bytes(int n, int dtype_bytes) {
    return n >= 6 ? 2 * ((size_t)1 << (2 * n)) * (size_t)dtype_bytes : 0;
}

}  // namespace pp
