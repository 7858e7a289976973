// Adjoint gradient: the forward sweep of the observable's weights c and the
// state's coefficients r, and the derivative of every rotation from it.
//
// <O> = c . r just before any gate.  For a rotation about sigma its derivative
// is c^T A r with A the generator of the forward rotation on a digit's (X, Y,
// Z): RX: c_Z r_Y - c_Y r_Z, RY: c_X r_Z - c_Z r_X, RZ: c_Y r_X - c_X r_Y,
// summed over the other digits, so minus the sigma component of v = sum c x r.
// A one-qubit gate acts on (X, Y, Z) as a proper rotation F, and F c x F r =
// F (c x r): v moves through a run of gates on one qubit as a vector.  So the
// sweep takes whole runs as one map each (see ChainOp), sums v once per run,
// before its map, and grad_runs_kernel walks the run's gates with v alone.
#include "chain.h"

namespace pp {
namespace {

// Tiles of K digits, c and r in LDS side by side.  One sweep per record: a
// thread takes its block of both vectors through the CX, adds its share of v,
// applies the maps and writes back.  What bounds it is the LDS, 128 KiB per
// record at K = 6, and, where few tiles leave most CUs idle, the time of a
// lone workgroup: 12.5 us per pass of 3.5 records (n = 8, 16 tiles, HEA of 40
// layers).  One sweep per rotation and another for its v, each with a
// workgroup reduction, took 40.6 us for the same pass (12 rotations).
template <int K_>
struct AdjointShape {
    static constexpr int K = K_;
    static constexpr int SIZE = 1 << (2 * K);
    static constexpr int NG = 1 << (2 * (K - 2));
    static constexpr int W = NG > 64 ? NG / 64 : 1;
    static constexpr int BLOCK = 64 * W;
    static constexpr int NP = kNumPairs<K>;
    static constexpr int CHUNK = 16;  // records staged at a time
    static constexpr int MAPS = CHUNK * 2 * kMapStride;
    static constexpr int ROWS = 4 * W;  // a record's partial sums: one per 16 lanes
    // the tiles first: their addresses are XORed
    static constexpr size_t OFF_MAPS = 2 * (size_t)SIZE * 8;
    static constexpr size_t OFF_RED = OFF_MAPS + (size_t)MAPS * 8;
    static constexpr size_t OFF_LANE = OFF_RED + (size_t)CHUNK * ROWS * 3 * 8;
    static constexpr size_t OFF_WAVE = OFF_LANE + (size_t)NP * 64 * 2;
    static constexpr size_t LDS = (OFF_WAVE + (size_t)NP * 16 * 2 + 15) & ~(size_t)15;
};

template <int CTRL>
__device__ __forceinline__ double row_add(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
}

// sum over each row of 16 lanes, in every lane of it
__device__ __forceinline__ double row_sum(double v) {
    v = row_add<0xB1>(v);   // lane ^ 1
    v = row_add<0x4E>(v);   // lane ^ 2
    v = row_add<0x141>(v);  // lane ^ 7 (the halves of 8)
    return row_add<0x140>(v);  // lane ^ 15
}

// c x r of one digit of a block, summed over the other digit
template <bool LO>
__device__ __forceinline__ void cross(const double (&c)[16], const double (&r)[16], double (&v)[3]) {
    v[0] = v[1] = v[2] = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int iX = LO ? 1 + 4 * q : q + 4, iZ = LO ? 2 + 4 * q : q + 8, iY = LO ? 3 + 4 * q : q + 12;
        v[0] += c[iY] * r[iZ] - c[iZ] * r[iY];
        v[1] += c[iZ] * r[iX] - c[iX] * r[iZ];
        v[2] += c[iX] * r[iY] - c[iY] * r[iX];
    }
}

template <int K>
__global__ __launch_bounds__((AdjointShape<K>::BLOCK)) void adjoint_kernel(const GradPassDesc *__restrict__ desc) {
    using S = AdjointShape<K>;
    extern __shared__ __align__(256) unsigned char smem[];
    typedef __attribute__((address_space(3))) double LT;
    typedef const __attribute__((address_space(4))) uint32_t *ConstWords;
    const GradPassDesc d = *desc;
    double *lc = reinterpret_cast<double *>(smem), *lr = lc + S::SIZE;
    double *mbuf = reinterpret_cast<double *>(smem + S::OFF_MAPS);
    double *red = reinterpret_cast<double *>(smem + S::OFF_RED);
    uint16_t *lanetab = reinterpret_cast<uint16_t *>(smem + S::OFF_LANE);
    uint16_t *wavetab = reinterpret_cast<uint16_t *>(smem + S::OFF_WAVE);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned tile = (unsigned)(size_t)(LT *)lc;
    const ConstWords recs = (ConstWords)d.chain;

    // the tile's first slot, and where local index i lies behind it
    long long base = 0;
    {
        unsigned inmask = 0;
        for (int j = 0; j < d.k; ++j) inmask |= 1u << (unsigned)((d.qubits >> (8 * j)) & 0xff);
        long long t = blockIdx.x;
        unsigned out = ~inmask & ((1u << d.n) - 1u);
        while (out) {
            const int q = __builtin_ctz(out);
            out &= out - 1u;
            base |= (t & 3ll) << (2 * q);
            t >>= 2;
        }
    }
    auto deposit = [&](int i) {
        long long o = 0;
#pragma unroll
        for (int j = 0; j < K; ++j) o |= (long long)((i >> (2 * j)) & 3) << (2 * (int)((d.qubits >> (8 * j)) & 0xff));
        return o;
    };
    const int size = 1 << (2 * d.k);  // 4 in a tile of two digits for n = 1
    // local index tid + BLOCK j: the parts below and above BLOCK do not overlap
    constexpr int PER = S::SIZE / S::BLOCK > 0 ? S::SIZE / S::BLOCK : 1;
    const long long off = base + deposit(tid);
    if (size >= S::BLOCK) {
        const double *gc = d.c + off, *gr = d.r + off;
#pragma unroll
        for (int j0 = 0; j0 < PER; j0 += 8) {
            double vc[8], vr[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const long long o = deposit(S::BLOCK * (j0 + j));
                if (j0 + j < PER) {
                    vc[j] = gc[o];
                    vr[j] = gr[o];
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j0 + j < PER) {
                    lc[sw(tid + S::BLOCK * (j0 + j))] = vc[j];
                    lr[sw(tid + S::BLOCK * (j0 + j))] = vr[j];
                }
        }
    } else {
        for (int i = tid; i < S::SIZE; i += S::BLOCK) {
            lc[sw(i)] = i < size ? d.c[off] : 0.0;
            lr[sw(i)] = i < size ? d.r[off] : 0.0;
        }
    }
    for (int i = tid; i < S::NP * 64; i += S::BLOCK) lanetab[i] = (&kPairTable<K>.lane[0][0])[i];
    for (int i = tid; i < S::NP * 16; i += S::BLOCK) wavetab[i] = (&kPairTable<K>.wave[0][0])[i];
    for (int c0 = 0; c0 < d.nrec; c0 += S::CHUNK) {
        const int cn = d.nrec - c0 < S::CHUNK ? d.nrec - c0 : S::CHUNK;
        const int mb = (int)recs[12 * c0 + 1];
        for (int i = tid; i < S::CHUNK * 18; i += S::BLOCK)
            mbuf[i + (kMapStride - 9) * (i / 9)] = mb + i / 9 < d.nmaps ? d.maps[9ll * mb + i] : 0.0;
        lds_barrier();
#pragma unroll 1
        for (int i = 0; i < cn; ++i) {
            const ConstWords rec = recs + 12 * (c0 + i);
            const unsigned w = rec[0];
            const double *src = mbuf + kMapStride * ((int)rec[1] - mb);
            const unsigned p = w & 0xffu;
            unsigned at = lanetab[p * 64 + lane];
            if constexpr (S::W > 1) at ^= wavetab[p * 16 + wave];
            at = tile + (at << 3);
            auto body = [&](auto kind_c) {
                constexpr int KIND = decltype(kind_c)::value;
                double c[16], r[16];
                unsigned ad[16];
                {
                    const unsigned x[4] = {rec[4], rec[5], rec[6], rec[7]};
                    block_addresses(ad, at, x);
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    c[e] = lds_word<double>(ad[e]);
                    r[e] = lds_word<double>(ad[e] + S::SIZE * 8);
                }
                {
                    const unsigned x[4] = {rec[8], rec[9], rec[10], rec[11]};
                    block_addresses(ad, at, x);
                }
                c[6] = flip(c[6], w & kChainFlip6);
                r[6] = flip(r[6], w & kChainFlip6);
                c[9] = flip(c[9], (w << 1) & kChainFlip6);
                r[9] = flip(r[9], (w << 1) & kChainFlip6);
                c[15] = flip(c[15], (w << 2) & kChainFlip6);
                r[15] = flip(r[15], (w << 2) & kChainFlip6);
                double vl[3] = {}, vh[3] = {};
                if constexpr (KIND & 1) {
                    cross<true>(c, r, vl);
                    double m[9];
#pragma unroll
                    for (int q = 0; q < 9; ++q) m[q] = src[q];
                    u1_regs_m<true>(c, m);
                    u1_regs_m<true>(r, m);
                }
                if constexpr (KIND & 2) {
                    cross<false>(c, r, vh);
                    double m[9];
#pragma unroll
                    for (int q = 0; q < 9; ++q) m[q] = src[(KIND & 1 ? kMapStride : 0) + q];
                    u1_regs_m<false>(c, m);
                    u1_regs_m<false>(r, m);
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    lds_put<double>(ad[e], c[e]);
                    lds_put<double>(ad[e] + S::SIZE * 8, r[e]);
                }
                // with maps on both digits the lower half of the wave sums
                // the lower digit's v and the upper half the higher digit's
                if constexpr (KIND != 0) {
                    double *out = red + ((size_t)i * S::ROWS + 4 * wave + (lane >> 4)) * 3;
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        double v;
                        if (S::NG < 64 && lane >= S::NG) vl[t] = vh[t] = 0.0;  // repeats another lane's block
                        if constexpr (KIND == 3) {
                            const double give = lane < 32 ? vh[t] : vl[t], keep = lane < 32 ? vl[t] : vh[t];
                            v = keep + __shfl_xor(give, 32, 64);
                        } else {
                            v = KIND == 1 ? vl[t] : vh[t];
                        }
                        v = row_sum(v);
                        if ((lane & 15) == 0) out[t] = v;
                    }
                }
            };
            const unsigned kind = (w >> kChainKindShift) & 3u;
            if (kind == 3) body(std::integral_constant<int, 3>{});
            else if (kind == 1) body(std::integral_constant<int, 1>{});
            else if (kind == 2) body(std::integral_constant<int, 2>{});
            else body(std::integral_constant<int, 0>{});
            if (S::W == 1 || ((w >> kChainNoBarrierBit) & 1u)) wave_lds_order();
            else lds_barrier();
        }
        lds_barrier();
        // the chunk's sums, rows in order
        for (int t = tid; t < cn * 6; t += S::BLOCK) {
            const int i = t / 6, high = (t % 6) / 3, x = t % 3;
            const uint32_t *rec = reinterpret_cast<const uint32_t *>(d.chain) + 12 * (c0 + i);
            const unsigned kind = (rec[0] >> kChainKindShift) & 3u;
            if (!((kind >> high) & 1u)) continue;
            double v = 0.0;
            for (int row = 0; row < S::ROWS; ++row)
                if (kind != 3 || ((row >> 1) & 1) == high) v += red[((size_t)i * S::ROWS + row) * 3 + x];
            const long long m = (long long)rec[1] + (high & (int)(kind & 1u)) - d.map_base;
            d.partials[(3 * m + x) * d.ntiles + blockIdx.x] = v;
        }
        lds_barrier();
    }
    lds_barrier();
    if (size >= S::BLOCK) {
        double *gc = d.c + off, *gr = d.r + off;
#pragma unroll 8
        for (int j = 0; j < PER; ++j) {
            const long long o = deposit(S::BLOCK * j);
            gc[o] = lc[sw(tid + S::BLOCK * j)];
            gr[o] = lr[sw(tid + S::BLOCK * j)];
        }
    } else if (tid < size) {
        d.c[off] = lc[sw(tid)];
        d.r[off] = lr[sw(tid)];
    }
}

// One wave per map: its v summed over the tiles (lanes, then a tree: a fixed
// order), then its run of gates.
__global__ __launch_bounds__(256) void grad_runs_kernel(GradRunsDesc d, int m0, int m1, int ntiles) {
    const int m = m0 + (int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6), lane = threadIdx.x & 63;
    if (m >= m1) return;
    double v[3];
    for (int t = 0; t < 3; ++t) {
        const double *p = d.partials + (3ll * (m - m0) + t) * ntiles;
        double s = 0.0;
        for (int i = lane; i < ntiles; i += 64) s += p[i];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        v[t] = s;
    }
    if (lane != 0) return;
    for (int r = d.roff[m]; r < d.roff[m + 1]; ++r) {
        const int op = d.rop[r];
        if (op >= 3) d.rot_grad[d.rslot[r]] = -(op == 3 ? v[0] : (op == 4 ? v[1] : v[2]));
        // the forward rotation about axis 0, 1 or 2 takes the next two axes
        // (a, b) to (c a - s b, s a + c b); S is RZ(pi / 2), H (z, -y, x)
        double sn = 1.0, cs = 0.0;
        if (op >= 3) sincos(d.theta[d.rparam[r]], &sn, &cs);
        const bool rx = op == 3, ry = op == 4, h = op == 0;
        const double a = rx ? v[1] : (ry ? v[2] : v[0]), b = rx ? v[2] : (ry ? v[0] : v[1]);
        const double a2 = cs * a - sn * b, b2 = sn * a + cs * b;
        const double x = rx ? v[0] : (ry ? b2 : a2), y = rx ? a2 : (ry ? v[1] : b2), z = rx ? b2 : (ry ? a2 : v[2]);
        const double hx = v[2], hy = -v[1], hz = v[0];
        v[0] = h ? hx : x;
        v[1] = h ? hy : y;
        v[2] = h ? hz : z;
    }
}

// r of |0...0><0...0|: Tr(P rho) = 1 for strings of I and Z only, else 0
__global__ void grad_init_state_kernel(double *r, int n, long long size) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < size;
         i += (long long)gridDim.x * blockDim.x) {
        bool zonly = true;
        for (int q = 0; q < n; ++q) zonly = zonly && !((i >> (2 * q)) & 1);
        r[i] = zonly ? 1.0 : 0.0;
    }
}

// Gates that share a parameter are summed in gate order.
__global__ void grad_accumulate_kernel(const double *__restrict__ rot_grad, const int32_t *__restrict__ off,
                                       const int32_t *__restrict__ slots, double *__restrict__ grad, int nparams) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= nparams) return;
    double g = 0.0;
    for (int i = off[p]; i < off[p + 1]; ++i) g += rot_grad[slots[i]];
    grad[p] = g;
}

template <int K>
hipError_t launch_adjoint_t(const GradPassDesc *d, int ntiles, hipStream_t s) {
    using S = AdjointShape<K>;
    static_assert(S::LDS <= 80 * 1024, "two workgroups per CU");
    auto fn = adjoint_kernel<K>;
    static bool attr = false;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
        if (e != hipSuccess) return e;
        attr = true;
    }
    hipLaunchKernelGGL(fn, dim3(ntiles), dim3(S::BLOCK), S::LDS, s, d);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_grad_pass(const GradPassDesc *d_desc, int ntiles, int k, hipStream_t s) {
    switch (k) {
    case 1:
    case 2: return launch_adjoint_t<2>(d_desc, ntiles, s);
    case 3: return launch_adjoint_t<3>(d_desc, ntiles, s);
    case 4: return launch_adjoint_t<4>(d_desc, ntiles, s);
    case 5: return launch_adjoint_t<5>(d_desc, ntiles, s);
    case 6: return launch_adjoint_t<6>(d_desc, ntiles, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_grad_runs(const GradRunsDesc &d, int m0, int m1, int ntiles, hipStream_t s) {
    if (m1 <= m0) return hipSuccess;
    hipLaunchKernelGGL(grad_runs_kernel, dim3((m1 - m0 + 3) / 4), dim3(256), 0, s, d, m0, m1, ntiles);
    return hipGetLastError();
}

hipError_t launch_grad_init_state(double *r, int n, hipStream_t s) {
    const long long size = 1ll << (2 * n);
    const int grid = (int)((size + 255) / 256 < 4096 ? (size + 255) / 256 : 4096);
    hipLaunchKernelGGL(grad_init_state_kernel, dim3(grid), dim3(256), 0, s, r, n, size);
    return hipGetLastError();
}

hipError_t launch_grad_accumulate(const double *rot_grad, const int32_t *off, const int32_t *slots, double *grad,
                                  int nparams, hipStream_t s) {
    hipLaunchKernelGGL(grad_accumulate_kernel, dim3((nparams + 255) / 256), dim3(256), 0, s, rot_grad, off, slots,
                       grad, nparams);
    return hipGetLastError();
}

}  // namespace pp
