// Host planner of libpauliprop: gate list -> device schedule.
#pragma once

#include <stdint.h>

#include <string>
#include <vector>

#include "pp_device.h"

namespace pp {

struct GateList {
    int n = 0;
    int64_t m = 0;
    std::vector<uint8_t> op;
    std::vector<int32_t> q0, q1, param;
    int32_t n_params = 0;
};

struct DensePass {
    int k = 0;
    uint8_t qubit[8] = {0};
    int op_begin = 0, op_end = 0;
    int64_t ngates = 0;
};

// Dense schedule.  ops are in Heisenberg order (g_m first); maps are built on
// the device from the recipes (gate code and parameter per folded gate).
struct DensePlan {
    bool resident = false;  // whole circuit in one workgroup's LDS
    int k = 0;              // tile qubits (n if resident)
    std::vector<DOp> ops;
    std::vector<int32_t> roff;  // nmaps + 1
    std::vector<uint8_t> rop;
    std::vector<int32_t> rparam;
    std::vector<int32_t> rgate;  // gate index
    std::vector<DensePass> passes;
    // untracked resident plans: the same ops as chain records (their maps are
    // numbered in record order); nchain of them, then the forward half's
    std::vector<ChainOp> chain;
    int nchain = 0;
    int fwd_from = -1;  // first map of the forward half (-1: none)
    int fwd_pass = -1;  // tiled plans: first pass of the forward half (-1: none)
    int nmaps() const { return (int)roff.size() - 1; }
};

// Sparse schedule: runs of Clifford gates, each closed by one rotation.
struct SparsePlan {
    std::vector<uint32_t> codes;  // Clifford gate codes, Heisenberg order
    std::vector<SparsePassDesc> passes;
};

// compose: fold consecutive single-qubit gates of a wire into one U1 op.
// reorder: let gates on disjoint qubits move past each other when packing
// passes.  Tracked runs disable both, because the term-update count
// U = sum_g |set entering g| depends on the gate order.
// k == n: one resident pass; k < n: passes of k-qubit tiles that always
// contain the lowest `low` qubits.
DensePlan plan_dense(const GateList &g, int k, int low, bool compose, bool reorder);
constexpr int kMaxGroupOps = 16;

// Shape of a GROUP (stored in its header's perm field; 0 = general): a CX
// whose control is the lower (dir 0) or higher (dir 1) digit of the pair,
// then U1 ops on digit sequence code 0 "lower", 1 "higher", 2 "lower,
// higher", 3 "higher, lower": shape = 1 + 4 dir + code.  These eight cover
// most groups of random circuits; the kernels run them as straight-line code.
int group_shape(const DOp *members, int count, int lo);
// Tile size of the register-tile kernel: its passes are ordered into SEG
// segments (see segment_ops in plan.cpp).
constexpr int kSegTileDigits = 6;

// Larger of the tile sizes whose untracked passes run as record chains
// (tile_chain.hip); the other is 6.
constexpr int kChainTileDigits = 7;
// Records of a pass at most (one per lane of a wave); a pass with more units
// than kTileUnits, which leaves room for the records that only move the
// tile, is split.
constexpr int kTileRecords = 64;
constexpr int kTileUnits = kTileRecords - 2;

// Whether untracked passes over k-qubit tiles of an n-qubit circuit run as
// record chains.  Beyond kChainMaxN they run op by op, a group at a time: units
// of a CX and a map per digit are more sweeps there (3,000 random gates at n =
// 16: 484, 462 in groups).
inline bool chain_tiles(int k, int n, bool segments) {
    return n <= kChainMaxN && (k == kChainTileDigits || (k == 6 && !segments));
}

// General form: gates [g_begin, g_end) only; forward = g_begin first (the
// adjoint sweep) instead of Heisenberg order.
struct PlanOptions {
    bool compose = true;
    bool group = true;  // pack ops on a common digit pair into GROUP ops
    bool reorder = true;
    bool lookahead = true;  // grow a tile by the gate whose greedy completion of the tile takes the most gates
    // order tiled passes of kSegTileDigits qubits into register segments
    // (SEG headers, which the register-tile kernel needs); the LDS kernels
    // skip SEG headers, so without segments they decode fewer ops
    bool segments = true;
    // order passes over tiles for the record chain (see chain_tiles): units of
    // a CX and a map per digit, at most kTileUnits
    bool chain = false;
    bool forward = false;
    int64_t g_begin = 0, g_end = -1;
};
DensePlan plan_dense_opts(const GateList &g, int k, int low, const PlanOptions &o);

// Structural checks of a dense schedule (used by the host-side tests):
// GROUP headers name two distinct digits below k and their members act only
// on them, passes tile the op list, digits are below the tile size, map
// indices are in range.  Returns an empty string or the first violation.
std::string plan_check(const DensePlan &P, int n);

// True when every non-empty tiled pass of kSegTileDigits qubits opens with a
// SEG header (the register-tile kernel can run it).
bool plan_segmented(const DensePlan &P);

// Digit triple (bit mask) the register-tile kernel loads a pass into: the
// first segment's triple when it avoids digits 0 and 1 (lanes then cover 16
// consecutive slots), else digits 3, 4, 5.
uint32_t pass_reg_entry(const DensePlan &P, const DensePass &ps);

// Appends `part` to `all`, offsetting op, map and recipe indices.
void plan_append(DensePlan &all, const DensePlan &part);

// Adjoint-gradient schedule: segments [bounds[s], bounds[s+1]) of the gate
// list; Heisenberg plans per segment (composed) and forward per-gate plans
// per segment; rotation slots in gate order.
struct GradPlan {
    std::vector<int64_t> bounds;
    DensePlan heis, fwd;
    std::vector<int> heis_pass_begin, fwd_pass_begin;  // S + 1 entries each
    std::vector<int> heis_chain_begin;                 // resident Heisenberg sweep: records per pass, as above
    std::vector<int> fwd_chain_begin;                  // records per forward pass, as above
    std::vector<int> fwd_map_begin;                    // S + 1 entries
    int nslots = 0;                                    // rotations, numbered in gate order
    std::vector<int32_t> rslot;                        // rotation of every entry of fwd's recipes (-1: a Clifford)
    std::vector<int32_t> param_off, param_slot;        // each parameter's rotations, in gate order
};
// Renumbers the maps of grouped passes (resident, or over tiles) in op order
// and appends each pass's records to P.chain; begin[p] (optional) receives the
// first record of pass p, with the total behind the last.  The records' words
// are for tiles of doubles.  ends: a tiled pass begins and ends with records whose pairs avoid
// digits 0 and 1 (without a CX or map where the schedule has no such op
// there), and has at least two.
void build_chain(DensePlan &P, std::vector<int> *begin = nullptr, bool ends = true);
// Byte offsets, in the 4^n array (weights of dbytes), of the letters of record
// r's pair: as it reads them (after = false) or writes them.
void record_offsets(const ChainOp &r, const DensePass &ps, int dbytes, bool after, uint32_t out[4]);
// Untracked evaluation of gates [0, g_end) from both ends: some taken back from
// the observable, the others forward from the state.  k = n: split where half
// of the CX gates lie on either side (a record holds about one), one pass of
// both halves' chains; k < n: tile passes scheduled from either end in turn,
// the forward half's from fwd_pass on; rec receives the first record of each
// pass over tiles that run as record chains.
DensePlan plan_meet(const GateList &g, int k, int low, int64_t g_end, bool segments,
                    std::vector<int> *rec = nullptr);
// The forward half of a tiled meet plan run backwards, as the Heisenberg
// schedule of the same gates: its passes and ops in reverse order (no GROUP or
// SEG headers), whose maps are the transposes of the forward maps.
DensePlan plan_reversed_forward(const DensePlan &P);
GradPlan plan_gradient(const GateList &g, int k_heis, int k_fwd, int low, int64_t every, bool segments);
SparsePlan plan_sparse(const GateList &g);

// Clifford frame of a sparse schedule (n <= kFrameMaxN): the rotation axis of
// every pass in the stored frame, and the rows of the linear map from a
// stored key to the x part of its actual string after every Clifford.
struct FramePlan {
    std::vector<FramePassDesc> passes;  // one per sparse pass
    std::vector<uint64_t> xrows;        // n masks over the packed key
};
FramePlan plan_frame(const GateList &g, const SparsePlan &sp);

// structural 3x3 pattern of one gate's Heisenberg map (bit 3*row + col)
unsigned gate_smask(int op);
unsigned smask_compose(unsigned after, unsigned before);

}  // namespace pp
