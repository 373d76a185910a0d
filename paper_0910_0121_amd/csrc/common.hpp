// Internal declarations shared by the library's translation units (host launchers and the
// small device helpers they need).  Nothing here is part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

namespace tpm {

constexpr int kMaxLevel = 21;             // 21 bits per axis, 63-bit keys
constexpr uint32_t kCellTag = 0x80000000u; // list entry: node index | tag, else sorted index
constexpr int kSortBits = 8;               // radix digit width
constexpr int kSortBins = 1 << kSortBits;
constexpr int kSortThreads = 256;

// Flags raised by the validation/key kernel.
constexpr unsigned kFlagNonFinite = 1u; // non-finite position or mass, or mass <= 0
constexpr unsigned kFlagRange = 2u;     // position outside [0, L)

// Device arrays of one tree (structure of arrays).  Nodes are stored level by level; the
// children of a node are contiguous and in octant order.
struct NodeArrays {
    uint64_t *code;        // (1 << 3 level) | key prefix
    uint32_t *first;       // first particle (key order)
    uint32_t *count;       // particles
    uint32_t *child_first; // index of the first child
    uint32_t *parent;      // index of the parent (root: itself)
    uint8_t *nchild;       // 0 for a leaf
    uint8_t *level;
    double *mass;          // FP64 moments
    double *comx, *comy, *comz; // mass-weighted position sums (the centre of mass is in nsrc)
    double *cnx, *cny, *cnz; // cube centres ((i + 1/2) * L / 2^level)
    // Sources as 32-byte records, one cache-line sector per list entry:
    double4 *nsrc;        // per node: centre of mass and mass
    const double4 *psrc;  // per particle in key order: position and mass
};

// Everything the walk reads about one node, in one 64-byte record (one cache line), built
// once per tree after the moments.
struct alignas(64) WalkNode {
    double cn[3];  // cube centre
    double com[3]; // centre of mass
    uint32_t first, count, child_first;
    uint8_t level, nchild, pad0, pad1;
};
static_assert(sizeof(WalkNode) == 64, "WalkNode must be one 64-byte line");

struct GroupArrays {
    uint32_t *node, *first, *count;
    double *cgx, *cgy, *cgz;  // bbox centre (lo + hi) / 2
    double *hgx, *hgy, *hgz;  // bbox half size (hi - lo) / 2
    double *xgx, *xgy, *xgz;  // cube centre of the group node (FP32 origin)
    double *lox, *loy, *loz, *hix, *hiy, *hiz;
};

// Workgroups are dealt to the 8 XCDs (each with its own L2) round-robin by block index.
// xcd_block renumbers block b of n so that each XCD takes a contiguous run: neighbouring
// groups (key order) then share one L2.  A bijection on [0, n).
constexpr uint32_t kXcds = 8;
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t n)
{
    const uint32_t q = n / kXcds, r = n % kXcds, x = b % kXcds;
    return x * q + (x < r ? x : r) + b / kXcds;
}
// The same within every kXcds * RUN blocks: an XCD takes runs of RUN neighbours, dealt in turn, for
// work that is uneven along the order or ends before the grid does.  The blocks past the last
// whole deal keep their numbers.
template <uint32_t RUN>
__device__ __forceinline__ uint32_t xcd_run(uint32_t b, uint32_t n)
{
    constexpr uint32_t kDeal = kXcds * RUN;
    if (b >= n / kDeal * kDeal) return b;
    return b / kDeal * kDeal + b % kXcds * RUN + b % kDeal / kXcds;
}

// Work counters that many waves share lie kQueueStride words (256 bytes) apart: atomics on one
// cache line from all XCDs are served one at a time, 40 to 55 ns each.
constexpr uint32_t kQueueStride = 64;

// ------------------------------------------------------------------ launchers (k_scan.hip)
// Exclusive prefix sum in place over n values; the total is written to *total (device).
// tmp must hold scan_tmp_elems(n) values of the same type.
size_t scan_tmp_elems(size_t n);
// Host-visible results without a stream synchronisation: copies up to three runs of device
// words (n0 + n1 + n2 < kMailboxWords in all) into the host-mapped mailbox from word 1 on
// and then writes seq into word 0; the host waits for word 0 to read seq.
constexpr uint32_t kMailboxWords = 64;
void publish_words(const uint32_t *src0, uint32_t n0, const uint32_t *src1, uint32_t n1,
                   const uint32_t *src2, uint32_t n2, uint32_t *mailbox, uint32_t seq,
                   hipStream_t s);
void fill_u32(uint32_t *p, size_t n, uint32_t v, hipStream_t s);
void fill_u64(uint64_t *p, size_t n, uint64_t v, hipStream_t s);
void scan_u32(uint32_t *data, size_t n, uint32_t *total, uint32_t *tmp, hipStream_t s);
void scan_u64(uint64_t *data, size_t n, uint64_t *total, uint64_t *tmp, hipStream_t s);

// ------------------------------------------------------------------ launchers (k_build.hip)
// Also stores each particle's (x, y, z, m) as one 32-byte record for the gather.
void launch_keys(int64_t n, const double *x, const double *y, const double *z, const double *m,
                 double L, uint64_t *key, uint32_t *idx, unsigned *flags, double4 *rec,
                 hipStream_t s);
// Stable LSD radix sort of (key, idx) by key; results end in key/idx.  hist holds
// sort_hist_elems(n) values.
size_t sort_hist_elems(int64_t n);
void radix_sort(int64_t n, uint64_t *key, uint32_t *idx, uint64_t *key_alt, uint32_t *idx_alt,
                uint32_t *hist, uint32_t *scan_tmp, hipStream_t s);
// The sort in two steps: stable passes over bits [run_bits, 63) only, 63 - run_bits a multiple of 8,
// then each run of equal high bits sorted by (key, index) in place.  Returns true if the result is
// in key_alt / idx_alt (an odd number of passes).  long_runs holds long_cap entries; flags (device,
// two words, zeroed by the caller) ends with flags[1] != 0 if a run could not be sorted this way:
// the order is then incomplete, and a sort with fewer run_bits (or radix_sort) on the returned
// arrays must follow (equal keys are still in index order).
// sort_run_bits: the run_bits to try first, 39, 31 and 23 up to 2^16, 2^21 and more particles
// (three, four or five passes; cells of level 8, 10.7 and 13.3).  The fullest cells of clustered
// boxes at those limits hold 451, 168 and, of 256^3 particles, 43; a pass less would meet runs of
// 1,601 at 2^19 particles and of 3,774, more than kLongRun, at 2^21.  Builds by three and by four
// passes: 65,536 particles 195 and 208 us uniform, 260 and 245 clustered (the runs' own sort);
// by four and by five: 2 million 532 and 563, 643 and 644, and 4 million 867 and 907, 928 and 943,
// where the line stays short of what denser boxes put into a cell.
constexpr int kLeastRunBits = 23;
int sort_run_bits(int64_t n);
constexpr uint32_t kShortRun = 64; // sorted within a tile of k_fix_runs
constexpr uint32_t kLongRun = 2048;
bool radix_sort_high(int64_t n, int run_bits, uint64_t *key, uint32_t *idx, uint64_t *key_alt,
                     uint32_t *idx_alt, uint32_t *hist, uint32_t *scan_tmp, uint2 *long_runs,
                     uint32_t long_cap, unsigned *flags, hipStream_t s);
// Zeroes flags (6 words) and *mmax and resets the groups' extremes (launch_groups).
void launch_build_init(unsigned *flags, unsigned long long *mmax, unsigned *min_level,
                       unsigned *max_count, hipStream_t s);
// Writes the key-ordered records psrc (x, y, z, m) and the bit pattern of the largest mass
// into *mmax, zeroed by the caller (the particle mesh scales its fixed-point sums by it).
void launch_permute(int64_t n, const uint32_t *idx, const double4 *rec, double4 *psrc,
                    unsigned long long *mmax, hipStream_t s);
void launch_root(NodeArrays nd, uint32_t n, double L, hipStream_t s);
// Level step: nodes [lo, hi) of level `level`; writes nchild, per-node child counts into
// cnt (hi - lo values) for the scan, and the octant bounds of subdivided nodes into bnd
// (7 (hi - lo) values).  Levels of at most kWideSplitNodes nodes use one wave per node.
constexpr uint32_t kWideSplitNodes = 16384;
void launch_split(NodeArrays nd, const uint64_t *key, uint32_t lo, uint32_t hi, int level,
                  int n_leaf, uint32_t *cnt, uint32_t *bnd, hipStream_t s);
// Emit children of nodes [lo, hi) at base + exclusive prefix in cnt, from the bounds in bnd.
void launch_emit(NodeArrays nd, const uint32_t *bnd, uint32_t lo, uint32_t hi, int level,
                 uint32_t base, const uint32_t *cnt, double L, hipStream_t s);
// The octree straight from the sorted keys (n >= 1, n_leaf - 1 <= kTreeWin): the same nodes in
// the same order as the level-by-level split.  launch_tree_levels writes per particle the
// levels of the nodes that start there and its leaf's count (sl, n words), per block of
// tree_blocks(n) the counts per level (blk, kMaxLevel + 1 rows of tree_blocks(n) words, left as exclusive prefixes) and
// the nodes per level into tot (kMaxLevel + 1 words).  With off[] from tot, launch_tree_emit
// writes every node but nchild and the internal counts (left to the moments with derive = 1).
constexpr int kTreeWin = 256;
struct TreeOffsets {
    uint32_t off[kMaxLevel + 3]; // first node of each level; past the last, the node count
};
// Levels of at most this many nodes next to each other share a launch of the moments.
constexpr uint32_t kFewNodes = 2048;
// Moments of all nodes, deepest level first (levels 0 .. max_level at to.off): mass, position
// sums S (comx/comy/comz; the centre of mass S / M goes to nsrc and the walk records wn).
// derive = 1 for a tree from launch_tree_emit: nchild and internal counts are set here, the
// children of a level's nodes being the next level's from child_first on.
void launch_moments(NodeArrays nd, const double4 *ps, const TreeOffsets &to, int max_level,
                    int derive, WalkNode *wn, hipStream_t s);
uint32_t tree_blocks(int64_t n);
// It also zeroes gstart (n words) and gflag (n + 1) for launch_group_mark.
void launch_tree_levels(const uint64_t *key, uint32_t n, int n_leaf, uint32_t *sl, uint32_t *blk,
                        uint32_t *tot, uint32_t *gstart, uint32_t *gflag, hipStream_t s);
void launch_tree_emit(NodeArrays nd, const uint64_t *key, const uint32_t *sl, const uint32_t *blk,
                      const TreeOffsets &to, uint32_t n, double L, hipStream_t s);
// Groups: mark in gstart[first] and gflag[first] (n and n + 1 words, zeroed here if `clear`)
// every maximal node with count <= n_crit or no children.  With gpos the prefix sums of gflag
// and *n_groups their total (device), launch_groups then lists the first cap groups in key
// order, with their boxes, lowers *min_level to the shallowest group level and raises
// *max_count to the largest group.
void launch_group_mark(NodeArrays nd, uint32_t n_nodes, int n_crit, uint32_t *gstart,
                       uint32_t *gflag, int64_t n, bool clear, hipStream_t s);
void launch_groups(NodeArrays nd, GroupArrays gr, const uint32_t *gstart, const uint32_t *gpos,
                   int64_t n, const uint32_t *n_groups, uint32_t cap, const double4 *ps,
                   unsigned *min_level, unsigned *max_count, hipStream_t s);

// ------------------------------------------------------------------ launchers (k_walk.hip)
// open = 0: fixed angle, th2 = theta^2.  open = 1: theta(d) of eq. (12) from eta = r_cut/2,
// theta0 and the cap theta_max; th2 = theta_max^2 and th2lo = theta_lo^2, where theta_lo =
// min(theta_max, theta0 / sqrt(0.46)) is below every value theta(d) takes (R g(R) peaks at
// 0.45273 near R = 0.650).
struct WalkParams {
    double L, rc2, th2, th2lo;
    double eta, theta0, theta_max;
    uint32_t n_nodes;
    uint32_t open;
};
// Group g's interaction list is entries[off[g] .. off[g] + len[g]).
// Lists in slots: list g at entry g size; one longer than that in room of its length from
// [spill_at, spill_end), handed out through *next, which starts at zero.  A list that fits
// neither sets bit 4 of the overflow flags.  size 0: no slots.
struct Slots {
    uint64_t size, spill_at, spill_end;
    unsigned long long *next;
};
// Two passes: the count pass writes each list length to counts[g]; after the caller's prefix
// sum (counts -> off) the emit pass writes the lists, len and gcells (cell entries), and sets bit
// 4 of *overflow if they need more than entries_cap entries.  With slots the emit pass runs alone.
void launch_walk_count(const WalkNode *wn, GroupArrays gr, uint32_t n_groups, WalkParams wp,
                       uint64_t *counts, unsigned *overflow, hipStream_t s);
void launch_walk_emit(const WalkNode *wn, GroupArrays gr, uint32_t n_groups, WalkParams wp,
                      uint64_t *off, uint32_t *len, uint32_t *entries, uint64_t entries_cap,
                      const Slots &slots, unsigned *overflow, uint32_t *gcells, hipStream_t s);
// One pass: n_waves waves write the lists into chunks of `chunk` entries taken from the
// pool entries[0, pool_cap); a group is walked into the wave's current chunk if at least
// `reserve` entries are left there, else (or if it did not fit) into a fresh chunk.  Sets bit 4 of
// *overflow if a list or the pool ran out of room (the lists are then incomplete).  counters holds kWalkCounterWords words (8-byte aligned).
constexpr uint32_t kWalkCounterWords = (kXcds + 1) * kQueueStride;
void launch_walk_pool(const WalkNode *wn, GroupArrays gr, uint32_t n_groups, WalkParams wp,
                      uint32_t n_waves, uint64_t pool_cap, uint64_t chunk, uint64_t reserve,
                      uint32_t *counters, uint64_t *off, uint32_t *len, uint32_t *entries,
                      unsigned *overflow, uint32_t *gcells, hipStream_t s);
// Adds (cell entries, particle entries, interactions) into stats[0..2] and the longest list
// into stats[3] (all zeroed by the caller).
void launch_walk_stats(GroupArrays gr, uint32_t n_groups, const uint32_t *len,
                       const uint32_t *gcells, unsigned long long *stats, hipStream_t s);

// Shared launches over several boxes.  The groups of boxes 0 .. nb-1 are laid end to end as
// one sequence of work items; box b holds items [g0, g0 + n_groups).  Each box keeps its own
// tree, lists and flags, exactly as in a walk of that box alone.
struct ForceItem;
constexpr int kMaxBatch = 16;
struct WalkBox {
    const WalkNode *wn;
    GroupArrays gr;
    WalkParams wp;
    uint64_t *off;                 // counts (count pass) or list offsets
    uint32_t *len, *entries, *gcells;
    unsigned long long *pool_next; // one-pass walk: the box's pool counter
    uint64_t pool_cap, chunk, reserve;
    unsigned *overflow;
    uint32_t g0, n_groups;
    uint64_t entries_cap;          // two passes: room at entries
    Slots slots;                   // or the room of each list, and no count pass
    unsigned long long *stats;     // see launch_walk_stats
    uint32_t *cls;                 // queue buffer of the force, and its pieces
    ForceItem *items;
    uint32_t *mailbox;             // launch_walk_results_one: where the results go, and
    uint32_t seq;                  // the sequence number that marks them
};
// Clears a walk's flags, statistics, queue bins and the word after its list lengths.
void launch_walk_init(const WalkBox &box, hipStream_t s);
void launch_walk_init_multi(const WalkBox *boxes, int nb, hipStream_t s); // device array
// off[0 .. n_groups] of each box to its exclusive prefix sums, for boxes of at most
// kOneBlockGroups groups (one workgroup per box).
constexpr uint32_t kOneBlockGroups = 16384;
void launch_walk_scan_multi(const WalkBox *boxes, int nb, hipStream_t s);
// The two passes over all items of the boxes (one wave per item; descriptors in device
// memory, total = sum of n_groups).
void launch_walk_count_multi(const WalkBox *boxes, int nb, uint32_t total, hipStream_t s);
void launch_walk_emit_multi(const WalkBox *boxes, int nb, uint32_t total, hipStream_t s);
// One pass over all items: n_waves waves take items in batches from kXcds counters (zeroed
// here; counters holds kXcds * kQueueStride words) and write each box's lists into chunks of that box's
// pool.  A box whose list or pool runs out of room gets bit 4 of its overflow flag; the other
// boxes are not affected.
void launch_walk_pool_multi(const WalkBox *boxes, int nb, uint32_t total, uint32_t n_waves,
                            uint32_t *counters, hipStream_t s);

// ------------------------------------------------------------------ launchers (k_force.hip)
struct ForceParams {
    double L, eps2, inv_eta, eta, rc2, rc;
    unsigned long long *pairs; // per group, the pairs left by the cutoff cull
};

// The FP32 pair law G(s) = g(2 sqrt(s)) / (s + (eps/r_cut)^2)^(3/2) (s = r^2 in units of
// r_cut^2) as pieces G = G_a (1 + r)^5, r quadratic in u = min(c + (1 - c) s, 1) less the piece's
// lower edge: 2^kTabSegBits pieces per octave of u, located by the bit pattern of u, from u = c up
// to u = 1 (R = 2); the last entry is zero and takes u = 1.
constexpr int kTabSegBits = 6;
constexpr int kTabShift = 23 - kTabSegBits;
constexpr int kTabAddrShift = kTabShift - 2; // bits(edge) >> this = byte address of its entry
constexpr int kTabMinExp = -27;              // c >= 2^-27: eps / r_cut down to 2^-13
struct ForceTable {
    const float *coef;  // device: the entries' G_a, then r's linear and its quadratic terms
    uint32_t entries;
    uint32_t base;      // byte address of the first entry: bits(c) >> kTabAddrShift
    float c;            // a power of two at most (eps/r_cut)^2 / 2
};
// Fills the table for eps / r_cut (host, FP64 fit, rounded to float) and ft but for its device
// pointer; false if eps / r_cut is not in [2^-13, 8).
bool build_force_table(double eps_over_rcut, std::vector<float> &coef, ForceTable &ft);

// The FP64 kernel's table: pieces of G = G_a (1 + r(t))^5, r a polynomial of degree kTab64Deg
// without a constant, 64 per octave over kTab64Oct octaves of u = c + (1 - c) s, c = 2^-kTab64Oct
// (see force_table64.cpp); the entry of u = 1 is zero.  G_a and the coefficients of powers 1 ..
// kTab64F64 - 1 are doubles, the others floats, each power an array of kTab64Entries.
constexpr int kTab64Exp = 18;
constexpr int kTab64Deg = 6, kTab64Oct = 24, kTab64F64 = 5;
constexpr uint32_t kTab64Entries = (uint32_t)kTab64Oct * 64u + 1u;
// False if (eps / r_cut)^2 is below 2^(1 - kTab64Oct) (the first pieces would not resolve it) or
// above 64: the kernel then evaluates eq. (2) pair by pair.
bool build_force_table64(double eps_over_rcut, std::vector<double> &hi, std::vector<float> &lo);

// The FP32 quadrupole kernel's table: U = 2 dG/du as cubic pieces in t, 2^kQuadSegBits per octave
// of the same u from the same c, the entry of u = 1 zero; its derivative V = dU/du by the same
// coefficients: per piece U's constant, V's constant, linear and quadratic term, each an array of
// `entries` floats.  U and V carry a factor 2^scale_exp, which the moments make up for.
constexpr int kQuadSegBits = 7;
constexpr int kQuadShift = 23 - kQuadSegBits;
constexpr int kQuadAddrShift = kQuadShift - 2;
struct QuadTable {
    const float *coef;
    uint32_t entries;
    uint32_t base; // byte address of the first entry: bits(c) >> kQuadAddrShift
    int scale_exp;
};
// For the c (a power of two) of the FP32 table of this eps / r_cut.
void build_quad_table(double eps_over_rcut, double c, std::vector<float> &coef, QuadTable &qt);

// Layout of the queue buffer (u32 words): the kXcds + 1 part starts of the whole groups (absolute
// word positions in the buffer), the number of pieces, the queue counters of the force kernel and
// of the quadrupole kernel (every wave reads the starts for each group: on the first counter's
// line they cost the 256^3 box 5 % of its force), the (part, cost bucket) cursors, then the group
// ids, each part's longest first.
constexpr uint32_t kClsStarts = 0;
constexpr uint32_t kClsItems = kClsStarts + kXcds + 1;
constexpr uint32_t kClsQueue = kQueueStride;
static_assert(kClsItems < kClsQueue, "");
constexpr uint32_t kClsQuadQueue = kClsQueue + kXcds * kQueueStride; // k_quad_f32's
constexpr uint32_t kClsBins = kClsQuadQueue + kXcds * kQueueStride;
constexpr uint32_t kClsLists = kClsBins + kXcds * 64;
// A group of more than 2^t pairs, 2^t about a 2^13th of the box's pairs, is taken in pieces: up to
// kPieceChunk of its particles against a segment of its list.  The sums of a chunk whose list is
// one segment go straight to the records, those of several to rows of three doubles, base +
// seg (particles of the chunk) + i.
struct ForceItem {
    uint32_t g, chunk, seg_segs, base; // seg_segs: segment, from bit 8 their number, from 16 s
};
constexpr uint32_t kPieceChunk = 128;
constexpr uint32_t kMaxSegs = 64;
constexpr uint32_t kSegMin = 64; // a segment is kSegMin 2^s entries
// An upper bound on the pieces of a box of n particles in G groups: a group in pieces has more
// than a 2^14th of the pairs, and its chunks are pieces of at least 2^(t-1) pairs but for the last
// of each list.
__host__ __device__ __forceinline__ size_t max_force_items(uint64_t n, uint64_t G)
{
    const uint64_t by_pairs = (1ull << 17) + n / kPieceChunk;
    const uint64_t by_groups = (G + n / kPieceChunk) * kMaxSegs;
    return (size_t)(by_pairs < by_groups ? by_pairs : by_groups);
}
// Parts and longest-first order of the groups (len: list lengths; stats: the walk's, of which the
// third is the box's interactions) into cls (kClsLists + n_groups words), and the pieces of long
// ones into items (max_force_items); the rows they need and their number into stats[4] and [5].
// The bins and stats have been cleared (launch_walk_init).
void launch_classify(GroupArrays gr, uint32_t n_groups, const uint32_t *len,
                     unsigned long long *stats, uint32_t *cls, ForceItem *items, hipStream_t s);
// launch_walk_stats and launch_classify in one launch of a workgroup (boxes of at most
// kOneBlockGroups groups), which then publishes the overflow word and the six statistics to
// the box's mailbox.
void launch_walk_results_one(const WalkBox &box, hipStream_t s);
// (boxes in device memory; most: the most groups of one)
void launch_walk_results_multi(const WalkBox *boxes, int nb, uint32_t most, hipStream_t s);
// A box's units in the force kernels, from the host so that no wave works them out (and holds them in
// vector registers): FP32, x' = x inv, sums times scale; FP64, u = r^2 k2 + c, sums times scale
// (1 without a table), and inv_f = 1 / r_cut and len_f = L / r_cut for the cull; 1 / L; r_cut with
// room for rounding.
struct ForceUnits {
    double inv, scale, k2, inv_L, rc_wrap;
    float inv_f, len_f;
};
// One box as the FP32 force kernel reads it.
struct ForceBox {
    NodeArrays nd;
    GroupArrays gr;
    uint32_t *cls;
    const uint64_t *off;
    const uint32_t *len, *entries;
    const double4 *ps;
    const uint32_t *pidx;
    ForceParams fp;
    ForceTable ft;
    ForceUnits units;
    void *rec;
    int rec64; // rec holds double4 records
    QuadTable qt;         // with quadrupole terms, FP32: its table
    const double *moments; // and the cells' second moments, six per node
    const ForceItem *items; // the pieces of long groups, their number, and the rows of their sums
    uint32_t n_items;
    double *rows;
    const double *tab64_hi; // FP64 kernel: its table, or null (pair by pair)
    const float *tab64_lo;
    uint32_t n_groups;
    unsigned long long *pair_sum; // pairs evaluated, over all groups
    int64_t n;
    void *out[3]; // launch_force_out_multi: the float outputs
};
// Empties a box's force and quadrupole queues and zeroes its pairs (which the pieces add to) and
// *pair_sum (which the output pass adds to).
void launch_force_prep(const ForceBox &box, hipStream_t s);
void launch_force_prep_multi(const ForceBox *boxes, int nb, hipStream_t s); // device array
// A persistent launch of at most two workgroups per CU over the box's pieces and queues.
void launch_force_f32(const ForceBox &box, int n_cu, hipStream_t s);
// The same over nb <= kMaxBatch boxes with equal tables (descriptors in device memory; the
// queues of all boxes are taken as one, through the first box's counters; n_work: groups and
// pieces in all).
void launch_force_f32_multi(const ForceBox *boxes, int nb, uint32_t n_work, int n_cu,
                            hipStream_t s);
// After the force and the FP32 quadrupole kernel: the rows of groups taken in pieces into their
// records (no launch without pieces).  The FP64 quadrupole kernel follows it.
void launch_force_merge(const ForceBox &box, hipStream_t s);
void launch_force_merge_multi(const ForceBox *boxes, int nb, uint32_t most_items, hipStream_t s);
// rec of the force launchers: one record per particle in the caller's order (pidx), float4
// (ax, ay, az, 0) or, with rec64, double4.  launch_force_out then writes them out: mode 0
// float arrays, 1 double arrays (from float4 / double4 records), 2 kick (v += dt a into double
// velocities, double4 records), walking the records in order; and adds the groups' pairs (the
// pairs the force kernel evaluated) into *pair_sum.
void launch_force_out(const void *rec, int mode, int64_t n, void *ax, void *ay, void *az,
                      double dt, uint32_t n_groups, const unsigned long long *pairs,
                      unsigned long long *pair_sum, hipStream_t s);
void launch_force_out_multi(const ForceBox *boxes, int nb, int64_t most, hipStream_t s);
// FP32 pair routine on explicit positions, pair by pair (xg: host, 3 values).
void launch_pairwise_f32(int64_t n_i, const double *xi, int64_t n_j, const double *xj,
                         const double *mj, const double *xg, double eta, ForceTable ft,
                         double *out, hipStream_t s);
// The FP64 force (k_force64.hip), over the same queues.
void launch_force_f64(const ForceBox &box, int n_cu, hipStream_t s);

// Particle-mesh long-range force (k_pm.hip), mesh N^3 with N a power of two in [16, 1024].
// Octant table of the Green's function ((N/2+1)^3 floats) and N/2 twiddles.
void launch_pm_green(int N, double L, double eta, float *green, double2 *tw, hipStream_t s);
// Fills the fixed-point mass mesh (N^3 words, every word written) from the key-ordered records
// and their sorted keys; mx holds the largest mass.  Scratch: cell_start (cells + 1 words),
// item_start (cells + 1 words), scan_tmp (scan_tmp_elems(cells) words) and slots
// (pm_assign_items_max x pm_assign_slot_words() words), cells = pm_assign_cells(N).
size_t pm_assign_cells(int N);
size_t pm_assign_items_max(int N, int64_t n);
size_t pm_assign_slot_words();
void launch_pm_assign(const double4 *ps, const uint64_t *key, int64_t n, int N, double L,
                      const unsigned long long *mx, uint32_t *cell_start, uint32_t *item_start,
                      uint32_t *scan_tmp, unsigned long long *slots, unsigned long long *mass,
                      hipStream_t s);
// Potential phi (N^3 floats; may lie where the masses do) from the mass mesh, through the complex
// work mesh grid (the half spectrum, pm_grid_points values).
size_t pm_grid_points(int N);
void launch_pm_potential(const unsigned long long *mass, const unsigned long long *mx,
                         int64_t n, int N, float2 *grid, float *phi, const float *green,
                         const double2 *tw, hipStream_t s);
// Interpolated force of key-ordered particle k (ps[k]) into stage[idx[k]] = (ax, ay, az, 0),
// i.e. in the caller's order (idx is the sort permutation).  cell_start and item_start as
// launch_pm_assign left them for the same particles.
void launch_pm_interp(const double4 *ps, int64_t n, int N, double L, const float *phi,
                      const uint32_t *idx, float4 *stage, const uint32_t *cell_start,
                      const uint32_t *item_start, hipStream_t s);
// ax[o] = stage[o].x etc. (float or double; accumulate adds).
void launch_pm_split(const float4 *stage, int64_t n, void *ax, void *ay, void *az,
                     int out_fp64, int accumulate, hipStream_t s);

// Quadrupole terms of the cell entries (k_quad.hip).  Q: 6 doubles per node (xx, yy, zz,
// xy, xz, yz about the centre of mass), filled level by level from the deepest.
void launch_second_moments(NodeArrays nd, const double4 *ps, const TreeOffsets &to, int max_level,
                           double *Q, hipStream_t s);
// Adds the cells' second-order terms to the box's force records, computed in FP64 or FP32 (then
// box.qt is its table; a persistent launch over queues of its own, emptied by launch_force_prep).
void launch_quad(const ForceBox &box, int fp64, int n_cu, hipStream_t s);

// Time stepping (k_step.hip).  Accelerations are float (acc_fp64 = 0) or double arrays.
// out receives the bit pattern of min_i(sqrt(eps / |a_i|), eps / |v_i|) (+inf if none binds).
void launch_timestep(int64_t n, const double *vx, const double *vy, const double *vz,
                     const void *ax, const void *ay, const void *az, int acc_fp64, double eps,
                     unsigned long long *out, hipStream_t s);
// Device scratch of the allocation-free time step (a static device array, 256 bytes): its
// address on `device`, which must be the current device, looked up once per device.
constexpr int kStepScratchWords = 32;
constexpr int kMaxDevices = 64;
hipError_t step_scratch(int device, unsigned long long **out);
// v += a dt_kick, then x += v dt_drift wrapped into [0, L), in place.
void launch_kick_drift(int64_t n, double *x, double *y, double *z, double *vx, double *vy,
                       double *vz, const void *ax, const void *ay, const void *az, int acc_fp64,
                       double dt_kick, double dt_drift, double L, hipStream_t s);

} // namespace tpm
