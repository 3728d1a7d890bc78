// Definitions shared by the host-side plan and the gfx950 kernels of libdgs.
#pragma once
#include <stdint.h>
#include <stddef.h>

namespace dgs {

// A tile is the unit one wavefront streams: 1024 consecutive elements of the
// flat buffer, tile t = [1024 t, 1024 t + 1024), regardless of tensor borders.
constexpr uint32_t TILE = 1024;
// Candidate slots reserved per tile.  A tile that would need more marks itself
// overflowed and its tensors are re-selected densely.
constexpr uint32_t CAPT = 256;
// The first HEAD candidates of every tile live in one 64-byte line of a dense
// array (tile t at heads[HEAD * t]), so that the selection kernel fetches a
// tensor's candidates with contiguous loads.  Candidates HEAD .. NEAR - 1 of a tile lie in a second
// dense array (at near[(NEAR - HEAD) * t]), the rest in slots of their own (at far[(CAPT - NEAR) * t]): at densities
// around 1 %, where a tile has 10 to 30 candidates, the lines of consecutive tiles are then neighbours in
// memory too, for the streaming pass that writes them and the passes that read them (1 % of 1e9 parameters: worker
// pass 2145 -> 2105 us, pull pass 713 -> 698, against 2 KB per tile for all behind the first line).
constexpr uint32_t HEAD = 8;
constexpr uint32_t NEAR = 32;
// Candidates of a tile that the streaming wavefront stages in LDS and writes out as
// whole 64-byte lines (later ones are stored one by one).
constexpr uint32_t STAGE = 64;
constexpr uint32_t WAVES_PER_BLOCK = 4;            // one "quad" = 4 tiles = 4096 elements
constexpr uint32_t STREAM_THREADS = 64 * WAVES_PER_BLOCK;
// Tensors up to this size are selected directly from the state buffer by one
// workgroup; larger ones ("big") go through candidate collection.
constexpr uint32_t SMALL_N = 8192;
// Threshold value that no 31-bit magnitude key reaches.
constexpr uint32_t TAU_NEVER = 0x80000000u;
constexpr uint32_t CNT_OVERFLOW = 0xFFFFFFFFu;
// Histogram of the streaming pass: key bits [30:19] (exponent + 4 mantissa bits).
constexpr uint32_t HBITS = 12;
constexpr uint32_t HBINS = 1u << HBITS;
constexpr uint32_t HSHIFT = 31 - HBITS;
// Selection workgroup.
constexpr uint32_t SEL_THREADS = 1024;
constexpr uint32_t SEL_WAVES = SEL_THREADS / 64;
constexpr uint32_t SEL_LDS_LIST = 16384;           // candidates kept in LDS (128 KB); longer lists continue in global scratch
// Longest candidate list one workgroup is planned for (rank 2 k).  One workgroup / the chain, us: flat tensors
// of 400 K / 550 K / 700 K / 900 K elements at 1 % (lists of 8 / 11 / 14 / 18 K), a round 51.3 / 56.5, 56.3 / 55.5,
// 63.7 / 57.0, 80.0 / 60.1, a step without momentum 26.3 / 26.9, 28.2 / 25.9, 33.9 / 27.3 (700 K); 2.4M at 0.3 % (15 K) a round
// 78.3 / 64.0; ResNet-50 shapes at 0.2 / 0.3 / 0.36 % (10 / 14 / 17 K), a round 124.7 / 126.7, 140.1 / 130.8, 152.6 / 134.0,
// a step 72.3 / 71.0, 79.8 / 72.3 (0.3 %).
constexpr uint32_t SEL_LIST_MAX = 10240;
// Tensors of fewer than SEL_CROWDED_TILES tiles are joined in half a round, and one workgroup keeps up for longer: 250 K
// elements with lists of 11 / 15 K a round 51.3 / 57.7, 56.3 / 63.1, 400 K with 11 / 19 K 55.1 / 57.9, 66.2 / 62.1, 500 K with 11 / 15 K
// 53.8 / 55.0, 59.5 / 56.9.  From SEL_LONG_TILES on the same line stands, but not because one workgroup were faster
// (4M with 11 / 20 K 71.1 / 67.1, 92.1 / 68.1, 6M with 12 / 18 K 86.7 / 74.6, 105.3 / 75.5, four of 7M with 10 / 14 K 139.3 /
// 140.4, 152.2 / 141.7): the tests of trimmed lists and of joins of several rounds have tensors of that size and state that
// the chain resolves none of them (segmented_tensors).  Nothing else speaks against SEL_LIST_MAX there.
constexpr uint32_t SEL_LIST_MAX_OTHER = 20480, SEL_LONG_TILES = 3584;
// One workgroup's time grows with its list, whatever the number of tensors (up to one per compute unit); the chain's grows with
// its slabs, two workgroups each, one to a compute unit.  A plan without a list beyond SEL_LIST_MAX_OTHER has the chain
// only while CHAIN_SLAB_COST entries of its longest list come on each slab.  Selection of a worker step, one workgroup / chain, us, tensors of
// 1.2M elements (10 slabs), lists of 11 K: 16 of them 32.0 / 25.3, 24 32.1 / 27.3, 32 32.1 / 32.5, 48 34.5 / 41.2, 64 38.8 / 50.6,
// 128 57.1 / 83.5; of 18 K: 32 47.2 / 33.0, 48 49.5 / 43.1, 64 56.2 / 57.1, 128 85.2 / 99.0.
constexpr uint32_t CHAIN_SLAB_COST = 32;
// Where the plan holds a tensor beyond its line, so that the chain's workgroups are there anyway, it also serves shorter lists,
// for tensors of at least SEL_CROWDED_TILES tiles (their join is then what the launch waits for).  us with the
// line at 8192 / 5000: ResNet-50 shapes, a round at 0.3 % 130.8 / 134.0, at 0.36 % 134.0 / 137.5, at 1 % 159.0 / 161.9, a step
// without momentum at 0.3 % 72.3 / 74.6, a server at 0.36 % 87.9 / 78.7; transformer shapes at 0.4 % 470.6 / 471.1.
constexpr uint32_t SEL_LIST_CROWDED = 8192, SEL_CROWDED_TILES = 512;
constexpr uint32_t SEL_LIST_HARD = 65536;          // longest it accepts when a tail has grown beyond the plan
// Above this density candidates stop paying off; such requests select densely.
constexpr double DENSE_DENSITY = 1.0 / 32.0;

// Parts.  Every tensor is cut into parts of up to SEG_TILES tiles, one workgroup each: a part
// joins its tiles' candidates into one ordered list, and the workgroup that arrives last for a
// tensor selects from the parts' lists.  Tensors whose candidate lists outgrow one workgroup
// (or whose request is dense) continue through the chain kernels, one workgroup per part.
#ifndef DGS_SEG_TILES          // (a CPU test build shrinks the parts so that small layouts have several)
#define DGS_SEG_TILES 256
#endif
constexpr uint32_t SEG_TILES = DGS_SEG_TILES;
// Join groups.  The candidates of consecutive parts of a tensor, up to about GROUP_TILES tiles,
// are joined by one workgroup: a tensor of one group is selected by that workgroup straight
// from LDS with no hand-over, larger tensors hand their groups' lists to the last to arrive.
#ifndef DGS_GROUP_TILES
#define DGS_GROUP_TILES 4096
#endif
constexpr uint32_t GROUP_TILES = DGS_GROUP_TILES;
constexpr uint32_t SEG_MIN_N = 65536;              // smaller tensors never take the chain
constexpr uint32_t SEG_LOWBITS = 12;               // key bits resolved by the second level
constexpr uint32_t SEG_WBINS = 2048;               // window of key >> SEG_LOWBITS above the threshold
constexpr uint32_t SEG_LBINS = 1u << SEG_LOWBITS;
// The chain: tiles of one workgroup (64 / 128 / 256 of them: 405 / 394 / 398 us a round on transformer
// shapes, 5398 / 5338 / 5368 us at 1 % of 1e9 parameters).
constexpr uint32_t CSLAB_TILES = SEG_TILES < 128 ? SEG_TILES : 128;
// Dense requests: tiles of one workgroup of the passes over the tensors themselves, 4 per wavefront.
constexpr uint32_t SLAB_TILES = SEG_TILES < 32 ? SEG_TILES : 32;
constexpr uint32_t SLAB_THREADS = SLAB_TILES / 4 * 64;
static_assert(SLAB_TILES * TILE >= SMALL_N + TILE && SLAB_TILES <= SEG_TILES, "a small tensor is one slab");
// The chain in the selection's launch, for plans of at most CHAIN_HERE slabs, or CHAIN_HERE_ONE of a single tensor: two
// launches less, and the chain runs beside the joins.  Beyond that the workgroups of one launch, one to a compute unit,
// are too few.  us in one launch / in three, over and over on the same few gradients (a step on ResNet-50 shapes takes 13 us more
// on gradients that the last-level cache does not hold): one tensor of 2^20 elements at 1 % (8 slabs) a round 57.0 / 67.5,
// ResNet-50 shapes at 1 % (130) a step without momentum 75.9 / 87.0, an event of a server with 8 sent rows 111.6 / 132.2, with
// difference rows 168.9 / 184.2, transformer shapes at 0.1 % (180) 367.7 / 376.9;
// one tensor of 30M at 0.3 % (230) 178.5 / 182.6, of 100M at 0.1 and 1 % (763) 436 / 459 and 587 / 607, of 250M at 0.3 %
// (1900) 1098 / 1069; 8 tensors of 96M in all at 1 % (732) 514.5 / 515, transformer shapes at 1 % (800) 603 / 587, 24
// tensors of 240M 1278 / 1243.
// (A CPU test build with small parts has layouts on either side of the line.)
constexpr uint32_t CHAIN_HERE = SEG_TILES < 128 ? 12 : 512, CHAIN_HERE_ONE = SEG_TILES < 128 ? 16 : 1024;
// There one workgroup counts the window histogram of a run of parts, so that a tensor has at most WINDOW_MAX histograms
// (the compute unit that adds them up reads 29 bytes a ns), or WINDOW_MAX_ONE where it is the only one (transformer
// shapes with 16 / 32 / 64 of them 373.5 / 367 / 367.8 us; one tensor of 100M at 0.1 % 510 / 457 / 437; 8 of 96M 521 /
// 514 / 531).
constexpr uint32_t WINDOW_MAX = 32, WINDOW_MAX_ONE = 64;
constexpr uint32_t window_parts(uint32_t nseg, uint32_t most) { return (nseg + most - 1u) / most; }
constexpr uint32_t window_blocks(uint32_t nseg, uint32_t most) { return (nseg + window_parts(nseg, most) - 1u) / window_parts(nseg, most); }
constexpr uint32_t SEG_MAX_PER_TENSOR = 512;       // parts per tensor whose list positions fit the selection's LDS
// Status of a tensor inside one selection call.
//   SEG_IDLE      nothing decided yet
//   SEG_DONE      selected and emitted
//   SEG_ACTIVE    the chain kernels finish it (prefix of the k-th key known), reading the tiles' candidates
//   SEG_LISTS     the same, reading the parts' lists (collected again after a failed prediction)
//   SEG_ALL       dense request with k_j = n_j: the emission sends every element
//   SEG_ZERO      fewer candidates than k, every nonzero among them: the chain emits them and the zeros
//   SEG_PENDING   the prediction failed: the parts collect again with a fresh threshold
//   SEG_FALLBACK  left to the dense single-workgroup selection
enum SegStatus { SEG_IDLE = 0, SEG_DONE = 1, SEG_FALLBACK = 2, SEG_PENDING = 4, SEG_ALL = 6, SEG_ACTIVE = 8, SEG_LISTS = 10, SEG_ZERO = 12 };
// A whole call in one launch (k_step).  Its units have 4, 8 or 16 tiles, as small as the compute units (of the device's at most STEP_CUS
// are counted) allow one for each unit of the tensors beyond SMALL_N, and a 16th more for small tensors; or 16 tiles and two units to a compute
// unit, for STEP_FEW tensors.  us in several launches / in one, a worker step with momentum, without, an event of a server with 4 difference
// rows, with 4 rows of the printed state:
//   one tensor of 100 K elements at 0.1 %     14.4 / 11.0   14.4 / 11.0   14.8 / 13.1   16.0 / 13.1
//   of 600 K at 1 %                           26.2 / 23.0   26.5 / 24.2   28.9 / 26.5   31.9 / 25.9
//   of 4M at 0.1 %                            31.7 / 24.6   31.7 / 25.8   33.9 / 26.0   36.1 / 28.0
//   of 8M at 0.1 % (489 units of 16)          60.9 / 40.1   58.9 / 40.2   54.8 / 39.1   58.5 / 43.1
//   64 of 2M in all at 1 % (256 of 8)         17.3 / 15.2   17.6 / 15.5   23.0 / 21.6   21.9 / 20.7
//   8 of 4M at 1 %                            30.4 / 26.1   30.7 / 25.6   44.8 / 37.9   42.8 / 35.9
// Beyond: 24 of 4M at 1 % (264) 24.0 / 24.3, 24.1 / 24.3, 31.5 / 32.3, 30.4 / 31.9, at 2 % 27.0 / 30.0, 27.6 / 30.2, 43.5 / 50.3, 39.1 / 45.9;
// 3 of 5M at 0.5 % (306) 34.2 / 36.7, 34.1 / 38.3, 40.2 / 39.8, 41.5 / 40.2.  Larger units than there is room for smaller ones: 64 of 2M at 1 %
// in units of 16 17.5, 17.4, 23.1, 22.7.  But a ranking workgroup reads a list per unit, and a tensor does not get more than
// STEP_UNITS_SMALLEST units of 4: one of 1M at 0.2 % 18.6 / 17.2 / 16.7 and 22.4 / 20.5 / 20.1 in units of 4 / of 8.  Units of 16 beside many small tensors,
// a 4th of STEP_CUS and more, give nothing: 120 mixed of 2M at 2 % 20.1 / 20.5, 20.5 / 20.2, 30.6 / 32.8, 29.9 / 32.3.
constexpr uint32_t STEP_CUS = SEG_TILES < 128 ? 0 : 256, STEP_UNITS_OVER = 16, STEP_UNITS_FEW = 2;
constexpr uint32_t STEP_FEW = 2, STEP_UNITS_SMALLEST = 192, STEP_SMALL = 4;
// (The CPU test build with small parts keeps to the kernels that larger layouts take.)
constexpr uint32_t DIES = 8;                         // XCDs: a launch's workgroups are dealt out to them in turn
// Where a tensor would take the chain, a worker step is one launch up to planned lists of STEP_CHAIN_LIST entries, or STEP_CHAIN_LIST_FEW with
// momentum and at most STEP_CHAIN_UNITS units; a pull always, as the chain gains it nothing there.  On one tensor of 2M at 0.5 %, 10 K pairs, in
// several launches / in one, as above, 26.8 / 28.1, 26.8 / 29.3, 32.9 / 32.4, 34.1 / 31.3; of 1M at 1 %, 10 K pairs and 123 units,
// 25.6 / 25.1, 25.8 / 27.1, 32.6 / 30.6, 35.4 / 30.6.
constexpr uint32_t STEP_CHAIN_LIST = 13312, STEP_CHAIN_LIST_FEW = 16384, STEP_CHAIN_UNITS = 128;
// A pull whose ranking workgroups emit more pairs than this in all takes several launches: 24 tensors of 2M at 2 %, 40 K pairs, an event
// 30.0 / 31.3 and 29.1 / 30.3 (a step 20.1 / 19.0), of 3M 36.4 / 37.3 and 34.1 / 35.6 (23.9 / 21.3); at 1 % of 3M 27.5 / 26.5, 29.6 / 25.3.
constexpr uint32_t STEP_PULL_K = 32768;
// Where a tensor of at least SEG_MIN_N elements has more than STEP_EMIT_K pairs, those tensors have emitting workgroups.
constexpr uint32_t STEP_EMIT_K = 2500;
constexpr uint32_t STEP_ITEMS = 16, STEP_ITEMS_KEYS = 32;      // entries, or keys, that a thread of the ranking holds in registers
constexpr uint32_t STEP_DONE = 0xFFFFFFFFu;          // SegState::key.x: nothing for the emitting workgroups to do
enum SegMode { SEG_MODE_AUTO = 0, SEG_MODE_ALWAYS = 1, SEG_MODE_NEVER = 2 };

struct TensorDesc {
    uint32_t off;        // first element
    uint32_t n;          // elements
    uint32_t big;        // n > SMALL_N
    uint32_t seg_first;  // first entry of this tensor in the segment table
    uint32_t nseg;       // segments (0: the tensor never goes segmented)
    uint32_t ds_first;   // its first entry in the table of dense slabs
    uint32_t grp_first;  // first entry of this tensor in the group table
    uint32_t ngrp;       // its join groups (>= 1)
    uint32_t cs_first;   // first entry of this tensor in the table of chain slabs
    uint32_t ncs;        // its chain slabs (0: never takes the chain)
};

struct PlanEntry {
    uint32_t k;       // ceil(density * n_j)
    uint32_t k2;      // rank whose key becomes the next predicted threshold (>= k, <= n_j)
    uint32_t outoff;  // sum of k over earlier tensors
    uint32_t k2_pull; // same for a pull, whose sent entries vanish: 2k to 2.5k (<= n_j), see fill_plan
    uint32_t seg;     // 1: segmented selection at this density
    uint32_t wire_off;   // wire form: first 32-bit word of the tensor's index block (after the values)
    uint32_t wire_bits;  // wire form: bits per local index = bit length of n_j - 1 (>= 1)
    uint32_t k2_zero; // same for a worker without momentum, whose sent entries vanish too: about 2k (<= n_j)
};

struct SegDesc {
    uint32_t j;       // tensor
    uint32_t tile0;   // first tile (of the flat buffer) of the segment
    uint32_t ntiles;  // tiles in the segment (<= SEG_TILES)
    uint32_t sidx;    // index of the segment within its tensor
};

constexpr uint32_t CHAIN_STATUS_SHIFT = 20, KEY_READY = 0x80000000u;      // (pfx: 31 - SEG_LOWBITS bits)

// A unit of a whole call in one launch: a run of elements of one tensor (a small tensor is one), and where in the
// ordered-list scratch its list lies: one line, then room for `cap` values, then for as many indices.
struct StepUnit {
    uint32_t j, e0, count;        // its tensor, first element, elements
    uint32_t n;                   // elements of the tensor
    uint32_t ord0;                // its list in SelectArgs::ord
    uint32_t cap;                 // a quarter of its elements, less the line
    uint32_t rows;                // rows of 256 elements of a wavefront: 1, 2 or 4 (16 such wavefronts are a unit)
    uint32_t pad;
};
constexpr uint32_t STEP_LINE = 16;                   // words; the second two of a run's first unit: what the run publishes
constexpr uint32_t STEP_READY = 0x80000000u, STEP_OVER = 0x40000000u;      // (over: more than there was room for)

struct SegState {        // per tensor, rewritten by every selection
    uint32_t status;     // SegStatus
    uint32_t pfx;        // key >> SEG_LOWBITS of the k-th entry (dense request: its leading bits so far)
    uint32_t r2;         // its rank among the entries sharing that prefix (SEG_ZERO: the zeros to add)
    uint32_t T;          // the k-th key (dense request, until it is known: 1 if the accumulate pass has listed the keys with pfx)
    uint32_t rT;         // how many of the entries equal to it are taken (lowest index first)
    // Hand-over between the workgroups of one launch (all zero between launches).  These words share a line with the plain
    // ones above, which the tensor's deciding workgroup stores through its cache: a die's L2 writes back the bytes that were
    // written in it and no others (the messages of neighbouring tensors, from workgroups on different dies, rely on
    // the same), and these words are only ever accessed past it.
    uint32_t verdict;    // 0 = not decided; else 0x100 | SegStatus, written by the last joining part
    uint32_t tau_ready;  // 1: the fresh threshold of a pending tensor is in place
    uint32_t pad0;
    uint2 chain;         // the chain in the selection's launch: 0 = not decided; else r2, and status << CHAIN_STATUS_SHIFT | pfx
    uint2 key;           // chain, and k_step's emission: 0 = not ranked; else rT, and KEY_READY | T (one store either, which needs
                         // no second)
    uint32_t pad1[20];
    // What is counted in, on a line of its own: a line that is added to all the time is fetched anew by everybody who
    // polls a word of it (transformer shapes, 180 slabs of one tensor: the arrivals alone took 7 us).
    uint32_t arrive[4];  // parts that have finished: [0] join, [1] re-histogram, [2] re-collection, [3] chain prefix
    uint32_t seen[2];    // readers of verdict / tau_ready that have passed (the last one clears)
    uint32_t chain_seen; // the same for chain and key (k_step: key alone)
    uint32_t pad2[25];
};
static_assert(sizeof(SegState) == 256, "two lines of 128 bytes");

struct DevStats {
    unsigned long long fallback_tensors;
    unsigned long long fallback_elems;
    unsigned long long candidates;
    unsigned long long internal_errors;
    unsigned long long segmented_tensors;
    unsigned long long repaired_tensors;
};

// OP_FMA: a = fmaf(lr, grad, state), state <- a (worker);  OP_IDENT: a = state (pull on a
// difference row);  OP_SUB: a = grad - state, nothing stored (pull on model - sent_k).
enum StreamOp { OP_FMA = 0, OP_IDENT = 1, OP_SUB = 2 };
// MODE_SAMPLE: the histogram of a sample of the buffer (the tiles in tile_list, zero keys counted
// too so that a tensor's counters add up to its sampled elements), nothing stored.
enum StreamMode { MODE_PLAIN = 0, MODE_COLLECT = 1, MODE_HIST = 2, MODE_SAMPLE = 3 };
enum StoreMode { STORE_PLAIN = 0, STORE_WT = 1, STORE_NT = 2 };
// What happens to a sent entry: SEL_WORKER state <- m * val;  SEL_PULL state <- +0;
// SEL_PULL_V state <- state + val (the values themselves are model - state).
enum SelectOp { SEL_WORKER = 0, SEL_PULL = 1, SEL_PULL_V = 2 };

// Dense requests: a tile's scratch for tensor j (SelectArgs::ord, CAPT * (tile + j)) holds, until the emission, how many of its
// keys are in the bucket that held the k-th key the call before, and those keys.  Words before and between are the slabs'.
// (dprev, per stream and tensor: one more than that bucket, 0 = unknown, and DPREV_STABLE if it was the same the call before that:
// nothing is listed otherwise.  A pull on Gaussian ResNet-50 shapes at 0.1 whose keys are scaled by 1.3 in every second call,
// nothing listed / listed after every call / so: 134 / 139 / 132 us, the row left as it is 133 / 129 / 129.)
constexpr uint32_t DPREV_STABLE = 0x80000000u;
constexpr uint32_t TKEYS_COUNT = 8, TKEYS_AT = 16, TKEYS_ROOM = 2 * CAPT - TKEYS_AT;
constexpr uint32_t TKEYS_STAGE = 64;                  // of them that a wavefront has in LDS and writes at once

struct StreamArgs {
    const float *grad;            // OP_FMA only
    float *state;                 // OP_FMA: in/out.  OP_IDENT: read only.
    const uint32_t *toff;         // J + 1 tensor offsets (elements)
    const uint32_t *tau;          // per tensor: candidate threshold (TAU_NEVER for small tensors)
    uint32_t *tile_cnt;           // per tile: low 16 = candidates of the leading tensor part, high 16 = trailing part
    uint2 *heads;                 // per tile HEAD x (index, value bits): candidates 0 .. HEAD-1
    uint2 *near;                  // per tile: candidates HEAD .. NEAR-1
    uint2 *far;                   // per tile: candidates NEAR .. CAPT-1
    uint32_t *ghist;              // per tensor HBINS counters
    uint32_t *keys;               // MODE_HIST for a dense request: the tiles' scratch (SelectArgs::ord); tau is dprev then
    uint32_t n, ntiles, nquads, quads_per_block, J;
    const uint32_t *tile_list;    // MODE_SAMPLE: the tiles to visit, nlist of them, four per "quad"
    uint32_t nlist;               //   (nquads = ceil(nlist / 4))
    float lr;
    uint32_t store_mode;          // OP_FMA: how the state is written back (StoreMode)
};

struct SelectArgs {
    float *state;                 // worker state, difference row, or sent_k row
    const float *model;           // SEL_PULL_V only: values are model - state
    const TensorDesc *tdesc;
    const PlanEntry *plan;
    const SegDesc *segtab;        // the parts, tensor after tensor
    const SegDesc *grptab;        // the join groups in launch order (tensors of several groups first)
    uint32_t *tau;                // hints of this stream, updated
    uint32_t *tile_cnt;
    uint2 *heads;
    uint32_t near0, far0;         // where the arrays near and far begin, counted from heads
    uint2 *ord;                   // ordered candidates of a part start at CAPT * (tile0 + j)
    uint32_t *hint2;              // per tensor: candidates expected at the hinted threshold (0 = unknown)
    uint32_t *tprev;              // per tensor: k-th key of the previous selection on this stream (0 = unknown)
    uint32_t *ghist;              // per tensor HBINS counters, all zero between uses
    SegState *segstate;
    uint32_t *segcnt;             // per part: candidates (bit 31: a tile of the part overflowed)
    uint32_t *grpcnt;             // per join group: the same, for the lists joined by groups
    const SegDesc *cslabs;        // chain slabs (sidx: the part they lie in), tensor after tensor
    uint2 *slabs_done;            // per chain slab: what it has published (slab_publish)
    uint32_t ncslabs;
    uint32_t *out_idx;
    float *out_val;
    DevStats *stats;
    const uint32_t *toff;         // J + 1 tensor offsets
    float m;                      // SEL_WORKER: sent entries keep m * a
    uint32_t n, ntiles, J, nparts;
    uint32_t ngroups, gparts;     // join groups; parts per group
    uint32_t dense;               // dense request: no candidate lists; tensors with parts take the chain
                                  // reading their own elements, the others select from the state buffer
    uint32_t write_hint;
    uint32_t young;               // pull: one of the first on this row, which aim at rank k2_zero
    uint32_t exact_mode;          // the threshold came from this call's histogram
    uint32_t repair;              // the launch carries the re-collecting workgroups
    uint32_t spin_limit;          // polls before a waiting workgroup gives up
    uint32_t bgroup;              // parts looked after by one re-collecting workgroup
    uint32_t later;               // SEL_PULL_V: k_add_sent moves the row behind the selection kernel, which leaves it alone
    const uint32_t *dslabs;       // dense requests: the tensor of every slab (run of SLAB_TILES tiles of a tensor), tensor after tensor
    uint32_t ndslabs;
    // The chain in the selection's launch: its workgroups' runs of parts (sidx: the first part; ntiles: of the whole
    // run), and the slabs of the tensors that take it.  nwin = 0: it has launches of its own.
    const SegDesc *wintab;
    const uint32_t *slabtab;
    uint32_t nwin, nslab;
    uint32_t window_max;          // histograms of a tensor at most
    // A whole call in one launch (k_step).
    const StepUnit *steptab;      // its units: nstep of them, a tensor's one after the other
    const SegDesc *ranktab;       // its ranking workgroups (tile0: the tensor's first unit in steptab, ntiles: how many), nrank of them
    const SegDesc *emittab;       // the runs of up to SEL_WAVES units that an emitting workgroup takes (sidx: which run of the tensor)
    uint32_t *stepflag;           // per unit, for the ranking: 0, or STEP_READY and the entries of its list; then as many for the emission
    uint32_t nstep, nrank, nemit;
    uint32_t multi;               // some tensor has several parts
    const float *grad;            // SEL_WORKER
    float lr;
};

// Host-callable launchers (defined next to the kernels).
// ev0 / ev1: optional hipEvent_t recorded at the begin / end of the kernel (both or neither).
void launch_stream(int op, int mode, const StreamArgs &a, uint32_t blocks, void *stream, void *ev0, void *ev1);
void launch_pick(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t *ghist, uint32_t *tau,
                 uint32_t *tprev, DevStats *stats, uint32_t J, bool sample, void *stream);
// Dense request: the accumulate pass's histogram -> the leading 12 bits of each k-th key, into segstate.
void launch_pick_dense(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t *ghist, uint32_t *dprev, SegState *segstate,
                       DevStats *stats, uint32_t J, void *stream);
// The selection: one launch for every tensor (join, exact k-th key, ordered emission, state
// fix-up, next hint; failed predictions are collected again inside the same launch).
void launch_select(int op, const SelectArgs &a, void *stream, void *ev0, void *ev1);
// SEL_PULL_V with SelectArgs::later: sent_k += G for the K pairs of the message.
void launch_add_sent(const SelectArgs &a, uint32_t K, void *stream, void *ev1);
// A whole worker step or pull.
void launch_step(int op, const SelectArgs &a, void *stream, void *ev0, void *ev1);
// Long candidate lists: the parts' window histograms, before the selection kernel, and what
// remains behind it for tensors left SEG_ACTIVE / SEG_LISTS / SEG_ZERO.
void launch_window(const SelectArgs &a, void *stream, void *ev0);
void launch_chain(int op, const SelectArgs &a, void *stream, void *ev0, void *ev1);
// Dense request: exact k-th keys and emission, reading the tensors themselves.
void launch_dense(int op, const SelectArgs &a, void *stream, void *ev0, void *ev1);
void launch_push(float *model, float *diff, uint32_t W, uint32_t n, const uint32_t *idx,
                 const float *val, uint32_t nnz, void *stream, void *ev0, void *ev1);
void launch_validate_idx(const uint32_t *idx, uint32_t nnz, uint32_t n, uint32_t *flag, void *stream);
void launch_wire_pack(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t J, uint32_t K, uint32_t words,
                      uint32_t value_bits, const uint32_t *idx, const float *val, uint32_t *wire, uint32_t *flag,
                      void *stream, void *ev0, void *ev1);
void launch_wire_unpack(const TensorDesc *tdesc, const PlanEntry *plan, uint32_t J, uint32_t K,
                        uint32_t value_bits, const uint32_t *wire, uint32_t *idx, float *val, uint32_t *flag,
                        void *stream, void *ev0, void *ev1);
void launch_apply(float *dst, uint32_t n, const uint32_t *idx, const float *val, uint32_t nnz, float sign,
                  void *stream);
void launch_fill_u32(uint32_t *p, uint32_t v, size_t count, void *stream);
// Host words -> device through kernel arguments (for the entry point that must not copy).
void launch_put_words(uint32_t *dst, const uint32_t *src_host, size_t words, void *stream);
// Pull without secondary compression.  scratch: ntiles + 2 ceil(ntiles / PULL_CHUNK) words; arrive: a
// counter, zero between calls; counted: hipEvent_t that completes once *host_total is in place.  The
// row and the outputs are left alone if there are more nonzeros than `capacity`.
constexpr uint32_t PULL_CHUNK = 4096;      // tiles of one workgroup of the position scan
void launch_pull_all(float *row, const float *model, uint32_t n, uint32_t ntiles, uint32_t *tile_cnt, uint2 *slots,
                     uint32_t *scratch, uint32_t *arrive, uint32_t *total, uint32_t *host_total, uint64_t capacity,
                     uint32_t *out_idx, float *out_val, void *stream, void *counted);

}  // namespace dgs
