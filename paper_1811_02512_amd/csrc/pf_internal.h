// Internal structures shared by the host analysis and the HIP kernels.
#pragma once

#include <hip/hip_vector_types.h>

#include <cstdint>
#include <string>
#include <vector>

namespace pf {

// Device view of one symbolic analysis.  Every pointer is a device address
// inside the caller's upload buffer.  Passed to kernels by value, or stored
// in a per-case table for batches with several sparsity patterns.
//
// Packed records (int4 = 4 x int32) let a lane fetch everything it needs
// about a node or a slot with one or two wide loads instead of a chain of
// dependent scalar loads:
//   node_info[x] (level order, 3 x int4): {j, bus, r0, r1}, {s0, s1, ydiag, 0},
//                                          {q0, q1, 0, 0}
//     j = position, [r0, r1) = its lower-neighbour range in rl,
//     [s0, s1) = its slots (higher neighbours), ydiag = Y entry (bus, bus),
//     [q0, q1) = the bus's admittance row
//   slot_info[s] (2 x int4): {k, bus_k, ylo, yup}, {u0, u1, j, bus_j}
//     k = higher neighbour, j = the owner, ylo/yup = Y entries (bus_k, bus_j) / (bus_j,
//     bus_k) or -1 for fill, [u0, u1) = its update pairs in upd
//   rl[r] = (i, slot(i;j))      upd[u] = (slot(i;k), slot(i;j))
//
// Tail: the top levels [tail_level, nlev) of the elimination tree, whose
// values fit in LDS, are factorised and solved in LDS.  Every higher
// neighbour of a tail node is itself in the tail.  Local numbering: tail
// nodes 0..K-1 in level order, tail slots 0..TS-1 in node order.
//   t_node[jl] (2 x int4): {j, bus, ydiag, sl0}, {sl1, rn0, rn1, rt1}
//     [sl0, sl1) local slots, [rn0, rn1) lower neighbours outside the tail
//     as (i, slot) global pairs in t_rl; [rn1, rt1), of a node of the clique,
//     those in the tail below the clique as (local i, local slot) pairs
//   t_slot[t] (int4): {s, kl, jl, 0}
//     s = global slot, kl = local node of k, jl = local node owning the slot
//   The clique is the last tail_clique local nodes: a chain of single-node
//   levels, each adjacent to every node above it (local slot of clique pair
//   (a, b), a < b, is t_node[a].sl0 + b - a - 1).
//   t_op (uint2, four 12-bit local indices and a 16-bit offset): {d | a << 12
//     | (b & 255) << 24, b >> 8 | j << 4 | next << 16}
//   t_lev[2 l] = {op0, ns, nd, ns2 | nd2 << 16}: the right-looking operations
//     of tail level l, one per destination d and node j of the level: at op0
//     every destination's first, ns on slots (W_d -= W_a D_j^-1 V_b, V_d -=
//     W_b D_j^-1 V_a), to nd on diagonals and the rhs (a = b: D_d -= W_a
//     D_j^-1 V_a, z_d -= W_a D_j^-1 z_j); then the second ones of the first
//     ns2 slots and the first nd2 diagonals, then further ones, each
//     destination's together; next > 0 in a first or second one: the
//     destination's next operation is that many places on, in a further one:
//     as many more follow.  Destinations with more operations come first.
//   t_lev[2 l + 1] = {op0, nb, ls | ld << 16, 0}: the backward operations of
//     level l below the clique: x_d -= U_a x_b for every slot a whose higher
//     neighbour b is on the level (d owns the slot); and the destinations of
//     the level with more than kTailSerial operations: the first ls slots
//     and the first ld diagonals (tail_longs: whether any level has some)
// Upper levels [mid_level, nlev) of a launch spread over several workgroups:
// all nodes' diagonals, rhs entries and slots there take the updates of lower
// levels in one pass; then the levels below the tail (the narrow ones) are
// factorised right-looking in global memory.  One workgroup alone pulls the
// tail's updates only, from all levels below it.
//   u_node[x] (2 x int4, x = level-ordered node - level_ptr[mid_level]):
//     {j, bus, ydiag, r2}, {r0, r1, s0, s1}: its lower neighbours as (i, slot)
//     pairs in u_rl, [r0, r1) those below mid_level, [r1, r2) those from there
//     to the tail; [s0, s1) = its slots
//   u_slot[t] (2 x int4, slots in the order of their nodes): {s, bus_j, bus_k,
//     ylo}, {yup, u0, u1, u2}: its update pairs in u_upd, as upd's, [u0, u1)
//     from below mid_level, [u1, u2) from there to the tail (in both lists
//     the second part is kept for the tail's nodes alone)
//   g_lev[2 i], g_lev[2 i + 1] (level mid_level + i): {op0, ns, nd, 0}, {ns2,
//     nd2, 0, 0}: its operations g_op = {d, a, b, j}, as t_lev's with global
//     slots and positions, the slots padded to a wavefront with d = -1 where
//     diagonals follow; g_next: the offset of a destination's next operation
struct DevSym {
    int32_t n, m, nn, slack;
    int32_t nnz_y, nnz_l, nlev, pad0;
    int64_t n_upd;
    int64_t vals_doubles, ws_doubles;
    int64_t lu_off;  // doubles before the LU section (D padded to 64 bytes)
    int64_t fd_lu, fd_mat;  // fast decoupled: d section (padded), one matrix
    // admittance matrix, CSR by bus
    const int32_t* yptr;     // n+1
    const int32_t* ycol;     // nnz_y
    const int32_t* ybr_ptr;  // nnz_y+1: branches contributing to each entry
    const int32_t* ybr;      // ascending branch ids
    // positions
    const int32_t* perm;     // nn: bus at position p
    const int32_t* pos;      // n: position of bus, -1 at the slack
    // filled pattern: S(p) = Li[Lp[p] .. Lp[p+1])
    const int32_t* Lp;       // nn+1
    const int32_t* Li;       // nnz_l
    const int32_t* ydiag;    // nn: Y entry (bus p, bus p)
    // hierarchical partition
    const int32_t* level_ptr;    // nlev+1
    const int32_t* level_nodes;  // nn
    const int32_t* level_g;      // nlev: lanes per node
    // packed records
    const int4* node_info;   // 3 nn
    const int4* slot_info;   // 2 nnz_l
    const int2* rl;          // nnz_l
    const int2* upd;         // n_upd
    // LDS tail
    int32_t tail_level, tail_nodes, tail_slots, tail_lds;
    int32_t tail_clique, tail_longs;
    int32_t ef_lds;  // bytes of the LDS copy of (e, f) per bus the Newton mismatch reads, 0 = none
    const int4* t_node;      // 2 K
    const int4* t_slot;      // TS
    const int2* t_rl;
    const int4* t_lev;       // 2 (nlev - tail_level)
    const uint2* t_op;
    // upper levels
    int32_t mid_level, u_slots;  // u_slots: entries of u_slot
    const int4* u_node;
    const int4* u_slot;
    const int2* u_rl;
    const int2* u_upd;
    const int4* g_lev;
    const int4* g_op;
    const int32_t* g_next;
    // Subtrees below a cut level (the group of workgroups that a spread
    // batch of grids gives a case hands each workgroup whole subtrees there,
    // so those levels need workgroup barriers only; a one-case spread launch
    // shares them and does not read these tables).  Roots: nodes of levels [0, sub_cut)
    // whose parent lies at level sub_cut or above (or is absent), numbered
    // by position.
    //   sub_idx[x] for x < level_ptr[sub_cut]: the level-ordered node
    //     records of each level again, grouped by root (ascending root,
    //     then record)
    //   sub_ptr[l (sub_roots + 1) + k]: entries of level l's group whose
    //     root is below k
    //   sub_cum[k]: work of the subtrees of roots below k (sub_roots + 1)
    int32_t sub_cut, sub_roots;
    const int32_t* sub_idx;
    const int32_t* sub_ptr;
    const int32_t* sub_cum;
};

// LDS budget of the tail until the caller sets one.
constexpr int64_t kDefaultTailBudget = 64 * 1024;

// Lists of the upper levels (DevSym's u_* and g_*).
struct UpperLists {
    int32_t mid_level = 0;
    bool whole = false;  // down to the first level wider than kMidWidth
    std::vector<int32_t> node, slot, rl, upd, lev, op, next;
};

struct HostSym {
    int32_t n = 0, m = 0, nn = 0, slack = 0, ordering = 0;
    std::vector<int32_t> from, to;
    std::vector<int32_t> yptr, ycol, ybr_ptr, ybr;
    std::vector<int32_t> perm, pos, parent, level;
    std::vector<int32_t> Lp, Li, ydiag;
    // Y entries (bus k, bus p) and (bus p, bus k) of slot (p; k), -1 if fill
    std::vector<int32_t> ylo, yup;
    std::vector<int32_t> owner;  // position that owns each slot
    // lower neighbours: descendants i with p in S(i), ascending, and p's slot there
    std::vector<int32_t> Rp, Ri, Rs;
    std::vector<int32_t> Up, Ua, Ub;
    std::vector<int32_t> level_ptr, level_nodes, level_g;
    std::vector<int32_t> node_info, slot_info, rl, upd;  // packed (int32 view)
    // tail
    int32_t tail_level = 0, tail_nodes = 0, tail_slots = 0, tail_lds = 0, tail_clique = 0;
    int32_t tail_longs = 0;
    int64_t tail_budget = kDefaultTailBudget;
    std::vector<int32_t> t_node, t_slot, t_rl, t_lev, t_op;
    // upper levels (DevSym); rebuilt with the tail
    UpperLists up;
    bool want_whole = false;  // a launch spreads this grid: build them whole
    // subtrees below a cut level (DevSym); rebuilt with the tail
    int32_t sub_cut = 0, sub_roots = 0;
    std::vector<int32_t> sub_idx, sub_ptr, sub_cum;
    int32_t ef_lds = 0;  // set at upload: 16 n when it fits in the device's LDS, else 0
    int32_t max_width = 0;
    int32_t threads = 0;  // 0: chosen per launch from the batch size
    int32_t interleave = 4;  // cases per interleaved workspace group
    // workgroups a one-case Newton launch spreads its wide phases over (the
    // bus loops and the levels below the LDS tail); 0 or 1: one workgroup
    int32_t spread = 0;
    // longest wait at a grid barrier of a spread launch, in ticks of the
    // 100 MHz constant clock, before the launch gives up (one second)
    uint64_t spread_wait = 100000000ull;
    // device copy
    DevSym dev{};
    bool uploaded = false;
    // counts uploads; a batch plan built over this symbolic records it and
    // refuses to run once the device copy has been replaced or gone stale
    uint64_t upload_gen = 0;

    // D [nn][4], zero padding to a multiple of 8 doubles, LU [nnz_l][8]: every
    // slot record (W, U) and bus record starts on a 64-byte boundary.
    int64_t lu_off() const { return 8 * (((int64_t)nn + 1) / 2); }
    int64_t vals_doubles() const { return lu_off() + 8 * (int64_t)Li.size(); }
    // fast decoupled matrices: per matrix d [fd_lu()] | (w, u) per slot; two
    // matrices (B', B'') per case
    int64_t fd_lu() const { return ((int64_t)nn + 7) & ~(int64_t)7; }
    int64_t fd_mat() const { return (fd_lu() + 2 * (int64_t)Li.size() + 7) & ~(int64_t)7; }
    int64_t fd_ws_doubles() const {
        // (cos, sin) | (e, f) | b | x, with room to spare
        int64_t w = 8 * (int64_t)n + 2 * (int64_t)nn;
        return (w + 31) & ~(int64_t)31;
    }
    // vals | bus records (8 n) | rhs (2 nn) | grid-barrier words of a one-case
    // launch spread over several workgroups (three 128-byte lines)
    int64_t sync_off() const {
        return (vals_doubles() + 8 * (int64_t)n + 2 * (int64_t)nn + 15) & ~(int64_t)15;
    }
    int64_t ws_doubles() const { return (sync_off() + 48 + 31) & ~(int64_t)31; }
    size_t dev_bytes() const;
};

// LDS bytes of a tail with K nodes and TS slots: W and U (or V) blocks per
// slot; the pivot block, the forward vector and the reciprocal of the pivot's
// determinant per node (an odd count of the latter padded to 16 bytes).
inline int64_t tail_bytes(int64_t K, int64_t TS) { return TS * 64 + K * 48 + (K + 1) / 2 * 16; }

// Operations of a tail destination that one thread or quad takes one after the
// other; what follows is shared by a wavefront.  The generated grids have at
// most 4 on a destination and level; one wavefront's share costs a barrier and
// a sum over its lanes.
constexpr int kTailSerial = 8;

// Tail nodes and slots have 12-bit local indices and offsets within a level's
// operations 16 bits (t_op).  The largest LDS budget holds fewer of all: 2,528
// slots, and a level at most 35,000 operations, as a row of d slots lies under
// a clique of d (d - 1) / 2.
constexpr int64_t kTailIndexMax = 4095;
constexpr int64_t kTailOpsMax = 65535;

// LDS bytes of the PV bitmask the Newton kernel keeps after the tail (one bit
// per bus, whole 64-bit ballot words).
inline int64_t pv_mask_bytes(int64_t n) { return 8 * ((n + 63) / 64); }

// Host analysis; returns a pf_status code and sets msg on failure.
int analyze(int n, int m, const int32_t* from, const int32_t* to, int slack, int ordering,
            HostSym& out, std::string& msg);
// Default lanes-per-node for every level from a simple work model.
void default_mapping(HostSym& s);
// (Re)builds the LDS tail for an LDS budget in bytes (0 disables it), and
// the subtrees below the cut level under it.
void build_tail(HostSym& s, int64_t budget);
void build_tail_ops(HostSym& s);
// The upper levels' lists: in a spread launch, the highest levels below the
// tail of at most kMidWidth nodes are factorised right-looking.  300, 600 and
// 1,200: one 10,000-bus case 1,248, 1,231 and 1,194 us, 64 mixed grids 3,359,
// 3,412 and 3,494: wider levels gain where 32 workgroups have them to
// themselves and lose where few share a grid.  An operation
// takes 20 bytes, and in a grid with much fill there are tens to hundreds per
// slot (a 100 x 100 mesh: 5.7 million, 113 MB and 0.4 s of analysis beside 65
// MB and 0.2 s without).  Whole lists are therefore for grids that a launch
// spreads, where they pay (there 131 -> 11 ms a solve); without, the lists end
// at kUpperTerms entries per slot of the factor, which the generated grids of
// up to 20,000 buses do not reach (at most 2.2 with a tail, 3.1 without).
constexpr int kMidWidth = 600;
constexpr int kUpperTerms = 4;
UpperLists build_upper(const HostSym& s, bool whole);
// Subtrees of the levels below the tail for spread launches: the highest cut
// at or below the tail level with at least kSubMinRoots roots (none if no
// such level).
constexpr int kSubMinRoots = 768;
void build_subtrees(HostSym& s);

}  // namespace pf
