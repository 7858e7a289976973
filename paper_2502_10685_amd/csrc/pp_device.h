// Internal structures shared by the HIP kernels and the host runtime of
// libpauliprop.  Not part of the public C ABI (include/pauliprop.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pp {

// ---------------------------------------------------------------- dense ops
// Dense layout: the weight of string P(x, z) lives at slot
//   idx = sum_q (x_q << 2q) | (z_q << (2q + 1)),
// i.e. qubit q owns the base-4 digit q (digit value x + 2z: I=0 X=1 Z=2 Y=3).
// This is the paper's index space 0 ... 4^n - 1 (Sec. III-B) with a digit
// order that makes a qubit's four letters one digit of the slot index.
enum : uint8_t { DOP_U1 = 0, DOP_CX = 1, DOP_GROUP = 2, DOP_SEG = 3 };

// One device operation on an LDS tile.  U1: a composed single-qubit map on
// local digit a (a real 3x3 matrix over the X, Y, Z weights, I is fixed).
// CX: control digit a, target digit b.  GROUP: header of the next ngates ops,
// which act only on digits a and b; a thread applies all of them to each
// 16-slot block of those two digits in registers.  SEG: header of the next
// ngates entries (GROUP headers included), whose ops act only on the digit
// triple a < b < smask; the register-tile kernel holds those three digits in
// registers for the whole segment, the LDS kernels skip the header.  16
// bytes, read uniformly.
struct DOp {
    uint8_t kind;
    uint8_t a, b;
    uint8_t ngates;   // gates folded into this op (term-update counting)
    uint16_t smask;   // U1: structural 3x3 pattern, bit (3*row + col)
    uint16_t perm;    // U1: 1 if the map is a signed permutation
    uint32_t map;     // U1: index into the 3x3 map array (9 doubles each)
    uint32_t reserved;
};
static_assert(sizeof(DOp) == 16, "DOp must stay 16 bytes");
// Bit of DOp::perm (any op but SEG): the next op of the pass stays inside
// one wave's quarter of a 6-digit tile as this one does, so 256-thread
// sweeps skip the workgroup barrier between them.
constexpr unsigned kSkipBarrier = 0x8000u;

// One record of an LDS-resident chain: an optional CX, then an optional 3x3
// map on each digit of one digit pair a < b.  word: pair index b (b - 1) / 2 +
// a in bits 0-7; 1 for a map on the lower digit + 2 for one on the higher in
// bits 8-9; kChainNoBarrierBit; the sign flips of the CX in bits 29-31 (bit 29:
// there is a CX; bit 30: its control is the lower digit; bit 31: the higher).
// map: the first of its maps (lower digit first); a chain's maps are stored in
// record order.
// The 16 letters of a block, e = letter of a + 4 letter of b, are read at the
// block's base XOR the words read[k] of e's set bits k and written at it XOR
// write[k]: swizzled byte offsets, those of read being the letters' images
// under the CX.
struct ChainOp {
    uint32_t word, map, reserved[2];
    uint32_t read[4], write[4];
};
static_assert(sizeof(ChainOp) == 48, "records are read as three 16-byte words");
constexpr unsigned kChainKindShift = 8;
// no workgroup barrier behind it: it and the next record avoid digit 5 of a
// six-qubit circuit, so each wave stays in its quarter of the tile
constexpr unsigned kChainNoBarrierBit = 12;
// letter pairs whose sign the CX flips: e = 6 in bit 31, e = 9 in bit 30, e =
// 15 in bit 29
constexpr unsigned kChainFlip6 = 0x80000000u;

// A whole circuit run inside one workgroup's LDS (n <= 7).  Tracked runs read
// ops; untracked ones the chain, whose first nchain records take the
// observable back and whose next nchain_fwd take the state forward.
struct ResidentDesc {
    const void *coef_in;       // start weights (4^n, slot order) or nullptr = the observable
    void *coef_out;            // final weights (4^n, slot order) or nullptr
    uint8_t *pres_out;         // final presence bytes or nullptr
    const DOp *ops;
    const double *maps;
    const uint64_t *obs_x, *obs_z;
    const double *obs_c;
    double *expval_out;
    unsigned long long *counters;  // [0] term updates, [1] final strings
    int32_t nops;
    int32_t n;
    int32_t nterms;
    int32_t distinct;  // 1: no string is repeated among the nterms
    const ChainOp *chain;
    int32_t nchain, nchain_fwd;
    int32_t nmaps;
    int32_t reserved;
    void *xbuf;        // n >= 6: where the two directions exchange their vectors
    unsigned *ticket;  // n >= 6: 0 between launches
};

// Where an evaluation's first pass over 6- or 7-qubit tiles begins: the
// observable of at most kStartTerms strings (the forward half begins with
// |0...0>).
constexpr int kStartTerms = 64;
struct TileStart {
    const uint64_t *obs_x, *obs_z;
    const double *obs_c;
    int32_t nterms;
};

// One pass of one circuit over its 4^(n-k) tiles of 4^k slots.
struct TilePassDesc {
    void *coef;                    // 4^n weights of the circuit
    uint8_t *pres;                 // presence bytes (tracked runs) or nullptr
    const DOp *ops;
    const double *maps;
    unsigned long long *counters;  // [0] term updates (tracked runs)
    int32_t n, k;
    int32_t op_begin, op_end;
    int32_t tile_begin;            // first block of this desc in the launch
    int32_t ntiles;
    uint64_t qubits;               // byte j = global qubit of local digit j (ascending)
    uint32_t forward;              // 1: a pass of the forward half (coef holds the state's coefficients)
    uint32_t reg_entry;            // register-tile kernel: digit triple (bit mask) to load into registers
    uint32_t nmaps;                // maps of the schedule (chained passes)
    // chained passes: the pass's records; its first is applied to the weights
    // as they come from HBM and its last as they go there, so these are byte
    // offsets in the 4^n array of the letters of their digit pairs, as in
    // ChainOp (in: read words of the first, out: write words of the last)
    const ChainOp *chain;
    int32_t nrec;
    uint32_t in[4], out[4];
    const TileStart *start;        // the first pass of a half: coef is not read but begun here (or nullptr)
};

// One pass of the adjoint sweep over tiles of 4^k slots (k = n: one tile).
// c: the observable's weights, r: the Pauli coefficients Tr(P rho) of the
// state, both FP64, both propagated forward through the pass's records.
struct GradPassDesc {
    double *c;
    double *r;
    const ChainOp *chain;
    const double *maps;   // forward maps
    double *partials;     // [3 (map - map_base) + letter][tile]: sums of c x r before the map
    int32_t n, k;
    int32_t nrec, nmaps;
    int32_t ntiles, map_base;
    uint64_t qubits;
};
// Maps [m0, m1): their sums over the tiles, then the derivative of every
// rotation in their recipes.
struct GradRunsDesc {
    const int32_t *roff, *rparam, *rslot;
    const uint8_t *rop;
    const double *theta;
    const double *partials;
    double *rot_grad;
};

// Block -> descriptor mapping of one tile-pass launch.  Descriptors are
// grouped by tile count (a power of 4); group g covers blocks
// [first_block[g], first_block[g+1]) and block b of it handles tile
// (b - first_block[g]) & ((1 << shift[g]) - 1) of descriptor
// first_desc[g] + ((b - first_block[g]) >> shift[g]).
constexpr int kMaxTileGroups = 8;
struct TileGroups {
    int32_t ngroups;
    int32_t chain;  // every descriptor holds its pass as records too
    int32_t start;  // some may hold first passes, whose weights were not filled in (chain kernel only)
    int32_t first_block[kMaxTileGroups + 1];
    int32_t first_desc[kMaxTileGroups];
    int32_t shift[kMaxTileGroups];
};

// Start weights and readout of one tiled circuit of a batch: the observable
// is scattered into its 4^n weights, and <O> read out into *out.
struct DenseIODesc {
    void *coef;
    const uint64_t *obs_x, *obs_z;
    const double *obs_c;
    double *out;
    int32_t n, nterms;
    int32_t distinct;  // 1: no string is repeated among the nterms
    int32_t reserved;
    void *state;       // the state's coefficients of a circuit run from both ends, or nullptr
    double *part;      // and kMeetDoubles for the product of the two
};

// Where the product c . r of a circuit run from both ends is summed up: one
// sum per block (at most kMeetBlocks), then the blocks' ticket (0 between
// launches).
constexpr int kMeetBlocks = 256;
constexpr int kMeetDoubles = kMeetBlocks + 8;

// Per-circuit composition job: maps[i] = product of the gate matrices of
// recipe entries [roff[i], roff[i+1]) in Heisenberg order.
struct ComposeDesc {
    const int32_t *roff;
    const uint8_t *rop;
    const int32_t *rparam;
    const double *theta;
    double *maps;
    int32_t nmaps;
    int32_t fwd_from;  // maps from this one on are forward maps (each gate's Heisenberg matrix transposed)
};

// --------------------------------------------------------------- sparse ops
// A sparse pass: a run of Clifford gates then (optionally) one rotation.
// Clifford gate code: op | q0 << 8 | q1 << 16 (op in {H, S, CX}).
struct SparsePassDesc {
    int32_t g_begin, g_end;  // range in the Clifford code array
    int32_t rot_op;          // 3..5 for RX/RY/RZ, -1 for none
    int32_t rot_q;
    int32_t rot_param;
    int32_t ngates;          // Cliffords + rotation (term-update counting)
};

// Clifford-frame sparse engine (n <= 31, exact propagation).  The Clifford
// gates are never applied to the strings: the host keeps the accumulated
// Clifford D (processed gates, Heisenberg order) and the stored set S stands
// for D^dag S D.  A rotation exp(-i t sigma/2) on qubit q is then a rotation
// about P = D sigma D^dag in the stored frame (a multi-qubit Pauli with a
// sign), whose child of an anticommuting S is i sin(t) P S.  Keys are packed
// as (z << n) | x.
struct FramePassDesc {
    uint64_t pmask;     // packed key of P's Pauli string
    int32_t sign;       // +1 or -1: P = sign * (the Hermitian Pauli of pmask)
    int32_t a;          // popcount(x & z) of P, mod 4
    int32_t rot_param;  // -1: no rotation (Clifford gates only)
    int32_t ngates;     // gates of the pass (term-update counting)
};

struct FrameBuffers {
    uint64_t *keys;            // list of stored strings: packed keys
    void *coef;                // their weights (FP64 or FP32)
    uint32_t *index;           // hash index: list positions (kFrameEmpty when free)
    unsigned long long *cnt;   // pass p reads the list length L and child
                               // count D of pass p - 1 from slot (p-1) mod 3
                               // ([slot] and [3 + slot]), records its own
                               // length in slot p mod 3 and counts its
                               // children in [3 + p mod 3]; [6] overflow
    unsigned long long *updates;
    unsigned long long *exact; // exact sum of the readout
    int64_t cap;               // list capacity
    int64_t slots;             // index slots (power of two, >= 2 cap)
    int32_t slot_bits;
    int32_t n;
};
constexpr uint32_t kFrameEmpty = ~0u;
constexpr int kFrameMaxN = 31;  // a key's 2n bits in one word

// ------------------------------------------------------------ launchers
// Dense engine (dense.hip)
// max_maps: the largest nmaps of the descriptors (sizes the grid; any value
// gives the same maps)
hipError_t launch_compose(const ComposeDesc *d_descs, int ndescs, hipStream_t s, int max_maps = 1);
hipError_t launch_resident_tracked(const ResidentDesc *d_descs, int ndescs, int n, int dtype_bytes, hipStream_t s);
// Untracked LDS-resident circuits (resident.hip).  meet: run the two
// directions and multiply (an evaluation); otherwise the observable's records
// only, with coef_in / coef_out.  out: result of a single descriptor, or
// nullptr for each descriptor's own expval_out.
hipError_t launch_chain(const ResidentDesc *d_descs, int ndescs, int n, int dtype_bytes, bool meet, double *out,
                        hipStream_t s);
// bytes of ResidentDesc::xbuf (0: not used)
size_t chain_exchange_bytes(int n, int dtype_bytes);
hipError_t launch_tile_pass(const TilePassDesc *d_descs, const TileGroups &groups, int k, int dtype_bytes,
                            bool track, hipStream_t s);
// Untracked passes over 6- and 7-qubit tiles of at most 14 qubits
// (tile_chain.hip).
// Whether launch_tile_pass would run untracked passes of circuits of n qubits
// with such records (TileGroups::chain) through launch_tile_chain, which begins
// first passes itself; the other kernels read coef.
// kChainMaxN: their 32-bit offsets in HBM.
constexpr int kChainMaxN = 14;
bool tile_pass_chained(int k, int n, bool chain);
hipError_t launch_tile_chain(const TilePassDesc *d_descs, const TileGroups &groups, int k, int dtype_bytes,
                             hipStream_t s);
int num_cus();
// 0: one workgroup per tile; 1: persistent prefetching workgroups (k <= 6)
void set_tile_kernel_variant(int k, int variant);
int tile_kernel_variant(int k);
hipError_t launch_grad_pass(const GradPassDesc *d_desc, int ntiles, int k, hipStream_t s);
hipError_t launch_grad_init_state(double *r, int n, hipStream_t s);
hipError_t launch_grad_runs(const GradRunsDesc &d, int m0, int m1, int ntiles, hipStream_t s);
// grad[p] = sum, in order, of the rotations slots[off[p], off[p + 1])
hipError_t launch_grad_accumulate(const double *rot_grad, const int32_t *off, const int32_t *slots, double *grad,
                                  int nparams, hipStream_t s);
hipError_t launch_copy_f64(const double *src, double *dst, long long count, hipStream_t s);
// count > 1: count weight arrays of 4^n slots back to back (parameter sets);
// distinct: no string is repeated among the nterms; state (optional): count
// arrays that receive the coefficients of |0...0>
hipError_t launch_dense_init(void *coef, uint8_t *pres, int n, int dtype_bytes, const uint64_t *x,
                             const uint64_t *z, const double *c, int nterms, bool distinct, hipStream_t s,
                             int count = 1, void *state = nullptr);
// <O> = sum over the strings of coef x state, for count pairs of arrays back
// to back; part: count x kMeetDoubles
hipError_t launch_meet_readout(const void *coef, const void *state, int n, int dtype_bytes, double *part, double *out,
                               hipStream_t s, int count = 1);
hipError_t launch_meet_readout_many(const DenseIODesc *d_descs, int nd, int max_n, int dtype_bytes, hipStream_t s);
// transposes of the 3x3 maps [first, nmaps) of src into dst
hipError_t launch_transpose_maps(const double *src, double *dst, int first, int nmaps, hipStream_t s);
// one workgroup per tile, whatever the tuned launch shape (untracked)
hipError_t launch_tile_pass_plain(const TilePassDesc *d_descs, const TileGroups &groups, int k, int dtype_bytes,
                                  hipStream_t s);
hipError_t launch_dense_readout(const void *coef, int n, int dtype_bytes, double *out, hipStream_t s,
                                int count = 1);
// the same for the nd circuits of a batch (one fill, one scatter launch;
// one readout launch), each circuit with the single-circuit arithmetic
hipError_t launch_dense_init_many(const DenseIODesc *d_descs, int nd, int max_n, int dtype_bytes, hipStream_t s);
// rho (2^n x 2^n complex, row-major (re, im) doubles) from the 4^n Pauli
// weights of 2^n rho in slot order; n <= 12
hipError_t launch_density_decode(const void *coef, int n, int dtype_bytes, double *rho, hipStream_t s);
hipError_t launch_dense_readout_many(const DenseIODesc *d_descs, int nd, int dtype_bytes, hipStream_t s);
hipError_t launch_dense_count(const uint8_t *pres, int n, unsigned long long *out, hipStream_t s);
hipError_t launch_dense_compact(const void *coef, const uint8_t *pres, int n, int dtype_bytes, uint64_t *x,
                                uint64_t *z, double *c, unsigned long long *count, int *tile_flags,
                                unsigned long long *tile_vals, int *ticket, hipStream_t s);
size_t resident_lds_bytes(int n, int dtype_bytes, bool track);
constexpr size_t kStaticLdsReserve = 8192;  // op cache + reductions per workgroup
int max_lds_bytes();

// Sparse engine (sparse.hip)
struct SparseBuffers {
    uint64_t *x, *z;      // cap2 entries each
    void *c;
    uint64_t *x2, *z2;    // ping-pong for the sort
    void *c2;
    long long *count;     // [0] live strings, [1] overflow flag, [2] first child,
                          // [3] count before a merge, [4] scan total (8 words)
    long long *scan;      // per-workgroup sums of the multi-workgroup scan (256)
    unsigned long long *updates;
    unsigned int *hist;   // radix histograms (sort_hist_entries(cap2) entries)
    int *tile_flags;      // per-tile counts
    uint32_t *table;      // list passes: three hash tables of 2^table_bits positions
    int table_bits;       // 2^table_bits > cap2
    unsigned long long *lens;  // list lengths, rotating over four passes
    unsigned long long *exact; // exact sums: the readout, then the dropped weight
    int64_t cap2;         // capacity of each array (2x the term capacity)
    int64_t max_tiles;
};
hipError_t launch_sparse_init(SparseBuffers &b, int dtype_bytes, const uint64_t *x, const uint64_t *z,
                              const double *c, int nterms, hipStream_t s, double *dropped_total = nullptr);
// Radix-sort shape of the merge, per capacity class (cap2 up to 2^18, up to
// 2^22, larger): 0 = 8 key bits per pass and 8 terms per thread (the
// default), 1 = 8 and 4, 2 = 8 and 16, 3 = 7 and 8, 4 = 7 and 16, 5 = 6 and
// 16.  All shapes give the same order; the histogram array must hold
// sort_hist_entries(cap2) words for any of them.
constexpr int kSortShapeCount = 6;
constexpr int kSortClasses = 3;
int sort_shape_class(long long cap2);
void set_sort_shape(int cls, int shape);
int sort_shape(int cls);
long long sort_hist_entries(long long cap2);
// Truncated propagation (approximate; off when on == 0): a split child with
// more than max_weight non-identity letters is not written, and a merged
// string with more letters or with |weight| < eps is dropped.  The absolute
// weight dropped is summed per tile into dropped[0, tiles) and added, in a
// fixed order, to dropped[max_tiles] (reset by launch_sparse_init; the list
// passes' is summed exactly and added by launch_list_leave).
struct SparseTrunc {
    int32_t on = 0;
    int32_t max_weight = 64;
    double eps = 0.0;
    double *dropped = nullptr;  // max_tiles + 1 doubles
};
hipError_t launch_sparse_pass(SparseBuffers &b, int dtype_bytes, const uint32_t *cliff_codes,
                              const SparsePassDesc &p, const double *theta, hipStream_t s,
                              const SparseTrunc &tr = SparseTrunc{});
hipError_t launch_sparse_merge(SparseBuffers &b, int n, int dtype_bytes, hipStream_t s,
                               const SparseTrunc &tr = SparseTrunc{});
// Rotations without a sort: strings that differ by the rotation's letter find
// each other through a hash table.  launch_list_enter takes nterms distinct
// strings (or, with x null, the merged list in b) through pass 0's Clifford
// run; launch_list_pass then runs pass `step` (it closes with a rotation) and
// the Clifford run of `next`, if there is one, and leaves the merged,
// truncated list in an order of its own; launch_list_leave ends it (last: the
// Clifford-only pass that the list has been taken through, or null).
hipError_t launch_list_enter(SparseBuffers &b, int dtype_bytes, const uint64_t *x, const uint64_t *z, const double *c,
                             int nterms, const uint32_t *cliff_codes, const SparsePassDesc &first, hipStream_t s,
                             const SparseTrunc &tr);
hipError_t launch_list_pass(SparseBuffers &b, int dtype_bytes, const uint32_t *cliff_codes, const SparsePassDesc &p,
                            const SparsePassDesc *next, int step, const double *theta, hipStream_t s,
                            const SparseTrunc &tr);
hipError_t launch_list_leave(SparseBuffers &b, const SparsePassDesc *last, int step, hipStream_t s,
                             const SparseTrunc &tr);
constexpr int kListTables = 3;
// words of an exact sum (see exact_add)
constexpr int kExactWords = 70;
// <O>: the weights of the I/Z strings of the list, in any order (NaN after an
// overflow)
hipError_t launch_sparse_readout(SparseBuffers &b, int dtype_bytes, double *out, hipStream_t s);
// Clifford-frame engine (sparse.hip)
hipError_t launch_frame_init(FrameBuffers &f, int dtype_bytes, const uint64_t *x, const uint64_t *z,
                             const double *c, int nterms, hipStream_t s);
// pass: its index in the schedule (selects the counter slots)
hipError_t launch_frame_pass(FrameBuffers &f, int dtype_bytes, const FramePassDesc &p, const double *theta,
                             int pass, hipStream_t s);
// <O>: the signed weights of the strings whose actual form D^dag S D (codes:
// every Clifford in processing order) is made of I and Z only (NaN after an
// overflow).  xrows[j]: mask of the key bits whose parity is bit j of the
// actual x part.
hipError_t launch_frame_readout(FrameBuffers &f, int dtype_bytes, const uint64_t *xrows, const uint32_t *codes,
                                int ncodes, int npasses, double *out, hipStream_t s);
// Every string in its actual form into out (x, z, weight in out's type),
// count and overflow flag into out.count[0], [1].
// The frame's strings after its last pass, in their actual form, into a
// zeroed 4^n DENSE weight array (the ramp of a DENSE evaluation).
hipError_t launch_frame_to_dense(FrameBuffers &f, int dtype_bytes, const uint32_t *codes, int ncodes, int npasses,
                                 void *coef, hipStream_t s);
hipError_t launch_frame_materialize(FrameBuffers &f, int dtype_bytes, const uint32_t *codes, int ncodes,
                                    int npasses, SparseBuffers &out, hipStream_t s);
// list length after `npasses` passes (the counters of the last one)
__host__ __device__ inline int frame_slot_of(int pass) { return ((pass % 3) + 3) % 3; }

}  // namespace pp
