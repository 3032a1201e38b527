// Interface between the host API code and the HIP kernels.
#pragma once
#include <hip/hip_runtime_api.h>
#include "zf_device.h"

namespace zf {

static const int LANE_CAP_MAX = 2048;      // upper limit of the walk kernel's item budget per wavefront (LDS)
static const int LANE_CAP_DEFAULT = 96; 
static const int WALK_WAVES = 8;           // wavefronts (= queued chunks) per block of the walk kernel; they share the staged tables
static const int WALK_BLOCK = WALK_WAVES * 64;
static const int WALK_RUN_MAX = 2;         // consecutive queue items a wavefront takes at a time (one when the queue is short)
static const int WALK_NODES_LDS = 80;      // trie nodes of a chunk the walk kernel stages in LDS (bigger chunks go to the fallback)
static const int WALK_DEPTH_MAX = 32;      // trie depth the walk kernel follows (deeper paths go to the fallback)
static const int BASE_SETS_LDS = 31;       // a row's chart is staged into LDS when it has at most this many sets ...
static const int BASE_ITEMS_LDS = 64;      // ... and items (the mask-automaton kernel takes larger limits from the host when LDS allows)
// The builds of mask_automaton_kernel, by the byte step they hold.  Charts whose sets are all of up to AUT_NARROW_SET_MAX items run the narrow one, of up to
// AUT_LANES_SET_MAX the one for a dozen items (a set that outgrows 64 items there goes to the fallback pass, and the engine's next calls to the build behind it; chart addresses known to be LDS and no hash table:
// 64 rows of the expression grammar without pruning, 8 steps of a decode loop, 988 us against 1,056 in the build that follows, while token-mask cache rows left
// its strings to this kernel: today they leave none, and with the cache off the same 8 steps take 673), others the one that
// holds the wide step as well, to which source sets of more than AUT_STEP_WIDE_FROM items go at once (the line at 16 measured the same).
static const int AUT_STEP_NARROW = 0, AUT_STEP_LANES = 1, AUT_STEP_WIDE = 2;
static const int AUT_NARROW_SET_MAX = 8, AUT_LANES_SET_MAX = 16, AUT_STEP_WIDE_FROM = 32;
static const int AUT_BASE_SETS_MAX = 1023; // the largest limits the host asks for
static const int AUT_BASE_ITEMS_MAX = 4096;
static const int TABLE_LDS_BUDGET = 56 * 1024;
// Wavefronts per block of the mask-automaton kernel.  The wavefronts of a block share the automaton they build, so a row of few large blocks works its
// steps out fewer times; but a compute unit holds one block of 16 (two of 8, three where registers allow).  So: 16 while every row can have such a
// block at once, 8 for larger batches, and where sets are so wide that 16 would not have their scratch (grammar of expressions without pruning,
// 8 steps, us, blocks of 8 / of 16: 64 rows x 152,064 893 / 801, 100 rows x 20,001 813 / 724, 200 rows 1,472 / 1,197, 512 rows 2,514 / 2,751; JSON 16 rows x 32,000 1,353 / 1,134).
static const int AUT_WAVES_MANY_ROWS = 8, AUT_WAVES = 16;
// A block takes a pass of its row's words with one word of the rank-ordered bitmap (32 strings) per thread; ...
static const int AUT_PART_WORDS = 128;     // ... the fewest a block of a row is made for ...
static const int AUT_GROUP_WORDS = 4;      // ... taken from the row in groups of this many neighbouring words (two batches of 64 ranks), dealt to the blocks round robin
static const int AUT_ENT_LDS = 64;         // token-mask-cache rows of the row's current set kept in LDS (more are read from global memory)
static_assert(AUT_LANES_SET_MAX <= AUT_ENT_LDS, "the kernel builds for small sets keep all cache-row numbers of a row in LDS");
static const int AUT_TABLE_LOADS = (TABLE_LDS_BUDGET + AUT_WAVES_MANY_ROWS * 1024 - 1) / (AUT_WAVES_MANY_ROWS * 1024);   // 16-byte pieces of the staged tables per thread
static const int AUT_HELP_QUEUE = 512;     // transitions one block can leave for free wavefronts in the course of a launch
// Automaton states a block can hold, and items of theirs per state (tables that leave no room for so many get fewer).  With 64, a vocabulary of a JSON grammar left thousands of
// strings per row to the fallback pass: 8 steps of 16 rows x 32,000 without pruning 858 us, 522 with 96, 523 with 128; a first step of 256 rows x 40,037 3,300, 1,130 and
// 370.  Blocks of 8 wavefronts keep 64 where two of them would not fit a compute unit otherwise.
static const int AUT_STATES_DEFAULT = 128, AUT_STATES_TIGHT = 64, AUT_ARENA_PER_STATE = 16;
static const int AUT_SPIN_LIMIT = 1 << 16; // polls of a transition another wavefront is computing before giving the strings to the fallback
static const int FB_DEPTH_MAX = 256;
static const int FB_WAVES = 512;           // wavefronts of the closing kernel that run the fallback pass (each has its own arena)
static const int FB_ITEMS_PER_WAVE = 65536; // its arena in global memory: items per wavefront (256 MB in all)
// The entry point that may not allocate keeps every per-call device buffer in one static device array:
static const size_t NOALLOC_SCRATCH_BYTES = 16u << 20;
static const int NOALLOC_FB_WAVES = 32;          // its fallback pass: fewer wavefronts ...
static const int NOALLOC_FB_ITEMS_PER_WAVE = 16384;   // ... with smaller arenas (4 MB of the array)
static const size_t NOALLOC_STAGE_BYTES = 256u << 10;  // pinned staging room per slot that every engine has from the start

// The persistent automaton (zf_options.walk_mode = 2): one store per engine in device memory.
#ifndef ZF_STORE_WAVES
#define ZF_STORE_WAVES 4
#endif
#ifndef ZF_STORE_LC_BITS
#define ZF_STORE_LC_BITS 10
#endif
static const int STORE_WAVES = ZF_STORE_WAVES;  // wavefronts per block of the mask kernel over the persistent automaton
static const int STORE_BLOCK = STORE_WAVES * 64;
static const int STORE_LDS_MAX = 159 * 1024;   // dynamic LDS a block of that kernel may ask for (the hand-over of the call's status has a static word of its own)
static const int STORE_SEG_WORDS_MAX = 64;     // mask words (of 32 tokens) a wavefront merges and checks per pass: 1 to 64, chosen per group so that a pass holds about one batch of undecided tokens
static const int STORE_AHEAD_BYTES = 2 * 64 * 16;  // of the logits a wavefront requests one pass ahead (two pieces per lane)
static const int LOOK_MEMBER_WORDS = 1024;     // mask words a wavefront of mask_look_kernel stores per pass, all members of the group together, at most
static const int STORE_WARM_ROWS = 32;         // rows of the transition table (states one byte from a row's current state) a block reads ahead into its LDS cache
static const int STORE_LC_BITS = ZF_STORE_LC_BITS;       // log2 of the entries of a block's LDS cache of table entries (8 bytes each)
#ifndef ZF_STORE_BLOCKS_PER_CU
#define ZF_STORE_BLOCKS_PER_CU 3
#endif
static const int STORE_BLOCKS_PER_CU = ZF_STORE_BLOCKS_PER_CU;   // blocks per compute unit the grid is made of at most (fewer when a compute unit holds fewer at once)
static const uint64_t STORE_FUSE_BYTES = 16u << 20;   // logits read and written by zf_compute_mask_apply_async up to which mask_store_kernel masks them itself
static const int STORE_PENDING_MAX = 4096;      // beyond this many bytes since its state was last known a row comes in through its chart again
// Flags of a group of rows (StoreGroup::meta, StoreRow::flags):
static const uint32_t STORE_ROW_CACHE = 1u;     // the token-mask cache rows of the group's current set are listed
static const uint32_t STORE_ROW_IMPORTED = 2u;  // the group's start state is the one the import kernel made from its chart
static const uint32_t STORE_ROW_SPILL = 4u;     // the record does not fit the short form: it is in StoreArgs::spilled
static const uint32_t STORE_ROW_POOLED = 8u;    // the mask is a finished row of the state cache's pool (row number: start): copied, nothing to check
static const uint32_t STORE_ROW_KEEP = 16u;     // the finished mask goes to the state cache's pool as well (row number: slot)
static const uint32_t STORE_ROW_DECIDED = 64u;  // mask_look_kernel: the listed cache rows, all in the record, leave no token to the parser
static const uint32_t STORE_ROW_REPORT = 32u;   // the host does not know the state the group stands in: the kernel reports it
struct StoreView {
    uint2 *hdr;                 // [cap_states] (first item in the arena, item count); count 0xFFFFFFFF = not published
    uint2 *arena;               // [cap_items] (item word, name of the set the item's rule started in)
    uint32_t *trans;            // [cap_states][n_cls] next state or AT_*
    unsigned long long *intern; // [intern_mask + 1] content signature << 32 | state; 0 = free
    uint32_t *ctl;              // [0] states handed out (the next name), [1] items handed out, [2] requests the store had no room for
    uint32_t cap_states, cap_items, intern_mask;
};
static const int STORE_ROW_ENT = 10, STORE_ROW_ENT_AT = 6;      // token-mask-cache rows a full record holds inline, and the word they start at
static const int STORE_ROW_PEND = 64, STORE_ROW_PEND_AT = 16;   // pending bytes a full record holds inline, and the word they start at
struct StoreRow {               // full record of a group of rows: 128 bytes, read by a wavefront with one load (lane k = word k)
    uint32_t start;             // [0] the state the group was last known to be in
    uint32_t n_pending;         // [1] bytes (as byte classes) fed to its rows since then: inline when they fit ...
    uint32_t pend_off;          // [2] ... else at this offset of the call's pending bytes
    uint32_t n_ent, ent_off;    // [3] [4] token-mask-cache rows of the current set: inline when they fit, else in StoreArgs::entries
    uint32_t flags;             // [5]
    uint32_t ent[STORE_ROW_ENT];
    uint8_t pend[STORE_ROW_PEND];
};
static_assert(sizeof(StoreRow) == 128, "a wavefront reads a full record as 32 words");
// One group of rows of a call: the rows that stand in the same state of the automaton, whose mask is worked out once.  The
// records of up to STORE_INLINE_GROUPS groups travel in the kernel's argument block, which the wavefronts read without a trip to
// the host's memory; larger calls upload them.  A record that does not fit (more pending bytes, more or larger cache row
// numbers) says so in its flags and is read from StoreArgs::spilled.
static const int STORE_INLINE_GROUPS = 64, STORE_INLINE_ROWS = 256, STORE_GROUP_PEND = 16, STORE_GROUP_ENT = 9;
struct StoreGroup {
    uint32_t start;                               // [0] as StoreRow::start
    uint32_t meta;                                // [1] n_pending | n_ent << 8 | flags << 16 | (mask words per pass - 1) << 24
    uint8_t pend[STORE_GROUP_PEND];               // [2 .. 5]
    uint16_t ent[STORE_GROUP_ENT];                // [6 .. 10 low half]
    uint16_t slot;                                // [10 high half] row of the state cache's pool (STORE_ROW_KEEP)
    uint16_t member_at, n_members;                // [11] the group's rows: members[member_at ..]
};
static_assert(sizeof(StoreGroup) == 48, "group records are twelve words");
struct StoreInline {
    uint16_t first_block[STORE_INLINE_GROUPS + 8];   // first block of each group, ascending; 0xFFFF beyond the call's groups
    uint16_t member[STORE_INLINE_ROWS];
    StoreGroup g[STORE_INLINE_GROUPS];
};
// What only a wavefront that computes a transition reads: in device memory, once per engine.
struct StoreConst {
    DeviceTables tab;
    StoreView view;
};
struct StoreArgs {
    const uint2 *cache;                // DeviceTables::ci_tok
    const Str16 *tok16;
    uint32_t *trans;                   // StoreView::trans
    uint32_t *out_mask;                // the caller's [batch][W] tensor
    uint32_t *pool;                    // the state cache's rows, [entries][W]
    const void *logits;                // zf_compute_mask_apply_async: the logits to be masked by the same kernel (APPLY builds)
    void *out;
    int64_t stride;                    // elements between their rows
    const StoreConst *konst;
    const StoreRow *spilled;           // pinned: full records, by group
    const uint32_t *entries;           // pinned: cache row numbers that do not fit a full record
    const uint8_t *pending;            // pinned: pending bytes that do not fit a full record
    const uint32_t *import_root;       // [group] device memory: written by the import kernel
    const StoreGroup *groups;          // null: in the argument block; else device memory, with ...
    const uint32_t *block_of;          // ... group | part << 16 of every block
    const uint16_t *members;           // row numbers of the groups, one group after the other; null: in the argument block
    unsigned long long *tickets;       // device memory, STORE_TICKETS words, zero when the kernel starts (see hand_over_store)
    unsigned long long *tickets_next;  // the same number of words for the next kernel, which this one clears
    unsigned long long *status;        // pinned host memory: (seq << 32 | value) words, see StoreStatus
    uint32_t seq;                      // the call's number (never 0)
    uint32_t V, W, ncls, cap_states, tab_mode;
    int32_t scratch;                   // items of one set under construction (per wavefront)
    uint8_t wide;                      // the rows' sets hold many items: the wide byte step first on larger sets
    uint8_t complete;                  // the host takes the status word for the mask's completion: the mask goes out write-through, ahead of the status
    uint8_t report_size;               // report the store's size whether or not a transition was computed
    uint8_t dtype;                     // of the logits: 0 = none, 1 = fp32, 2 = bf16
    uint32_t n_blocks;
};
static_assert(sizeof(StoreArgs) + sizeof(StoreInline) <= 4096, "the kernel's argument block");
// mask_look_kernel (zf_mask_look.hip): calls whose groups all stand in states whose vocabulary has been walked before.
#ifndef ZF_LOOK_BLOCKS_PER_CU
#define ZF_LOOK_BLOCKS_PER_CU 3
#endif
static const int LOOK_BLOCKS_PER_CU = ZF_LOOK_BLOCKS_PER_CU;
static const int LOOK_WORDS = 9;
static const uint32_t LOOK_ENT_OF_MORE = 8, LOOK_ENT_MAX = 255;
static const uint32_t LOOK_POLLS = 1024;   // LookArgs::polls: a millisecond and more, where a wait lasts as long as a block of the mask is at work (6 to 130 us)
static const int LOOK_UNIT_KB = 4;      // logits that a wavefront of mask_look_kernel holds while the mask is worked out, at most: a register quadruple per lane and KB
struct LookGroup {                     // as StoreGroup, without what a known state does not need, in nine words:
    uint32_t w[LOOK_WORDS];            // [0] state; [1] n_ent | flags << 8 | (mask words per pass - 1) << 16; [2] first block | segments << 16;
};                                     // [3] first member | members << 16; [4] pool row | cache row 0 << 16; [5 ..] cache rows 1, 2, ... two to a word; of more than STORE_GROUP_ENT the first
                                       // LOOK_ENT_OF_MORE, then where in the list of members, behind them, the others are
struct LookInline {
    LookGroup g[STORE_INLINE_GROUPS];
    uint16_t member[STORE_INLINE_ROWS];
};
struct LookArgs {
    const uint32_t *trans;             // as in StoreArgs:
    const uint2 *cache;
    const Str16 *tok16;
    uint32_t *out_mask, *pool;
    const StoreConst *konst;
    const LookGroup *groups;
    const uint32_t *block_of;
    const uint16_t *members;
    unsigned long long *tickets, *tickets_next, *status;
    uint32_t seq, V, W, ncls, n_groups, complete;
    uint32_t mask_blocks;              // blocks that work the masks out; behind them, where the logits are masked along:
    uint32_t units, row_units, unit_kb, dtype;   // units of logits, one per wavefront, of unit_kb KB each; of a row; 1 = fp32, 2 = bf16
    uint32_t polls;                    // how often such a wavefront looks for its mask words before it leaves its unit to its group of blocks
    unsigned long long *tagged;        // [groups][W] mask words on their way to those wavefronts: call's number << 32 | word; behind them a word per block with logits, likewise
    const void *logits;
    void *out;
    int64_t stride;                    // elements between rows of logits
    uint32_t done_groups;              // groups of blocks that report to the host, each in a status word of its own (STORE_ST_ROW + group)
    const uint16_t *group_of;          // of the k-th entry of `members`, where the records are in device memory
};
static_assert(sizeof(LookArgs) + sizeof(LookInline) <= 4096, "the kernel's argument block");
// Units of a call: its blocks report in 16 groups, each counted in 16 bits.
static const uint32_t LOOK_UNITS_MAX = 4000000;
inline uint32_t look_grid(const LookArgs &a) { return a.mask_blocks + (a.units + STORE_WAVES - 1) / STORE_WAVES; }
// Words of a call's status in pinned host memory.  Every word carries the call's number in its upper half, so the host knows of
// each word by itself whether it has arrived: no order between them is needed (a release would write the L2 back first).
enum : uint32_t { STORE_ST_DONE = 0,       // low half: walks that failed (24 bits) | STORE_ST_MORE; written last, by the block that finishes last
                  STORE_ST_STEPS = 1,      // Earley byte steps   (this word and the next three only with STORE_ST_MORE)
                  STORE_ST_STATES = 2, STORE_ST_ITEMS = 3, STORE_ST_REFUSED = 4,
                  STORE_ST_ROW = 8 };      // + group: the state the group arrived in (groups with STORE_ROW_REPORT); mask_look_kernel: + group of blocks: its failed walks, when it is done
static const uint32_t STORE_ST_MORE = 0x80000000u;
// A ticket word lies 64 bytes from the next: additions to words of one line queue up behind each other like additions to one word
// (launches of 768 blocks that do nothing else: 10.2 us to the status word with the words side by side, 8.2 apart, 6.8 without tickets).
static const int STORE_TICKET_GROUPS = 64, STORE_TICKET_STRIDE = 8, STORE_TICKETS = (STORE_TICKET_GROUPS + 1) * STORE_TICKET_STRIDE;

// A set of per-call counters: words 0-7 as listed at MaskArgs::counters, then the tickets the blocks of a call's last kernel
// draw when they are done (one word per group of blocks, so that thousands of blocks do not queue up at one address, and a
// top word the last block of each group draws from).
static const int COUNTER_SET_WORDS = 160, TICKET_GROUPS = 64, TICKET_AT = 16, TICKET_TOP = 144;
static const int FB_WALKED = 96, FB_CLAIMED = 112;   // words of it, a line each: shares of the fallback pass that have been walked; a bit per share that somebody walks
static_assert(FB_WAVES <= 32 * 16 && FB_CLAIMED + 16 <= TICKET_TOP, "a line of bits");

struct MaskArgs {
    DeviceTables tab;
    const RowChart *rows;      // [batch]
    const uint32_t *set_off;   // shared CSR offsets of all rows' sets
    const Item *items;         // shared item array of all rows
    const uint32_t *entries;   // shared array of token-mask-cache rows (see RowChart)
    uint32_t so_stride, it_stride, ent_stride;   // not 0: row r's sections start at r * stride in set_off / items / entries (every row has the same room)
    uint32_t *rank_mask;       // [batch][Wr] verdicts in trie (rank) order
    uint32_t *out_mask;        // token-order rows: the caller's tensor, or the state cache's pool
    const uint32_t *dst_row;   // [batch] row of out_mask that row r of this launch is written to; null = row r
    const uint32_t *row_slot;  // [user_batch] pool slot that holds the finished mask of each of the caller's rows
    uint32_t *user_mask;       // the caller's [user_batch][W] tensor (target of the gather)
    int32_t user_batch;
    int32_t handoff_in_permute; // 1: permute is the call's last kernel (state cache off), else the gather is
    uint32_t *counters;        // [0] chunks passed to the fallback, [1] length of the work queue, [2] chunks nobody could resolve,
                               // [3] Earley byte steps, [16..144] tickets and the fallback pass's counts (FB_...) of the call's last kernel;
                               // COUNTER_SET_WORDS words per set
    uint32_t *host_status;     // pinned host memory, 8 words: this call's counters [0..3], written by its last kernel, then [4] = seq
    uint32_t seq;              // the call's number (never 0): the last word the call's last kernel writes, which is what the host waits for
    uint32_t *counters_next;   // the next call's counters: cleared by this call's last kernel (no separate memset)
    uint4 *work;               // queue of (row, chunk, undecided strings, -) that need the parser walk
    uint4 *overflow_list;      // (row, chunk, undecided strings, -) for the fallback
    uint32_t overflow_cap;
    uint2 *fb_items;           // [fb_waves][fb_stride]
    uint32_t *fb_set_start;    // [fb_waves][FB_DEPTH_MAX + 2]
    uint32_t fb_waves;         // wavefronts of the fallback pass (each has its own arena) ...
    uint32_t fb_stride;        // ... of this many items
    int32_t batch;
    int32_t lane_cap;          // item budget of a walking wavefront
    int32_t fb_cap;            // item budget of a fallback wavefront (<= FB_ITEMS_PER_WAVE)
    int32_t walk_blocks;       // blocks of the walk grid (one and a half times what the chip holds at once)
    int32_t mode;              // 0: all tables staged in LDS, 1: the small ones only, 2: none
    // mask-automaton kernel: capacities of one block's automaton in LDS
    int32_t aut_states;        // states (rows of the transition table)
    int32_t aut_arena;         // items of all states together
    int32_t aut_scratch;       // items of one set under construction (per wavefront)
    int32_t aut_parts;         // blocks per row (grid.x)
    int32_t aut_base_sets;     // a row's chart is staged into LDS when it has at most this many sets ...
    int32_t aut_base_items;    // ... and items (both at least BASE_SETS_LDS / BASE_ITEMS_LDS)
    int32_t aut_step;          // the kernel build (AUT_STEP_*) ...
    int32_t aut_waves;         // ... and the wavefronts of its blocks
    // logits that the closing kernel masks along (zf_compute_mask_apply_async; dst_row is null then)
    const void *logits;        // [batch] rows, logit_stride elements apart
    void *logits_out;
    int64_t logit_stride;
    int32_t logit_dtype;       // 0: none, 1: fp32, 2: bf16
};

int choose_table_mode(const DeviceTables &t);
uint32_t walk_lds_bytes(const DeviceTables &t, int mode, int lane_cap);   // dynamic LDS of one block of the walk kernel
hipError_t walk_blocks_per_cu(int mode, uint32_t lds_bytes, int *out);   // resident blocks of the walk kernel per compute unit
hipError_t prepare_kernels();   // one-time function attributes (dynamic LDS above 64 KB) of all kernels:
hipError_t prepare_walk_kernels();
hipError_t prepare_automaton_kernels();
hipError_t launch_upload(const void *pinned_src, void *dst, size_t bytes, hipStream_t s);   // bytes rounded up to 16: both buffers must hold that much
hipError_t launch_cache_merge(const MaskArgs &a, hipStream_t s);
hipError_t launch_mask_walk(const MaskArgs &a, hipStream_t s);
uint32_t automaton_lds_bytes(const DeviceTables &t, int mode, int states, int arena, int scratch, int base_sets, int base_items, bool wide, int waves);
int automaton_blocks_per_cu(const MaskArgs &a);   // of the build and the LDS size that a's call launches
hipError_t launch_mask_automaton(const MaskArgs &a, hipStream_t s);
hipError_t prepare_store_kernels();
uint32_t store_lds_bytes(const DeviceTables &t, int mode, int scratch);
int store_blocks_per_cu(const DeviceTables &t, int mode, int scratch);
hipError_t launch_mask_store(const StoreArgs &a, const StoreInline &in, uint32_t lds_bytes, hipStream_t s);
int look_blocks_per_cu();
hipError_t launch_mask_look(const LookArgs &a, const LookInline &in, hipStream_t s);
hipError_t launch_store_clear(const StoreView &G, uint32_t ncls, const void *root_items, uint32_t n_root, hipStream_t s);
// The store, cleared, whose headers, items and table rows of the states below n_states were copied in from the host: their places in the
// hash table, and how far the store is filled.
hipError_t launch_store_adopt(const StoreView &G, uint32_t n_states, uint32_t n_items, hipStream_t s);
// n charts (packed as for the other mask kernels) become states; import_root[group[k]] = the state of chart k's current set (AT_FAIL: no room)
hipError_t launch_store_import(const StoreView &G, const RowChart *charts, const uint32_t *set_off, const Item *items, const uint32_t *group,
                               uint32_t n, uint32_t *import_root, hipStream_t s);
hipError_t launch_finish(const MaskArgs &a, int cus, hipStream_t s);   // fallback pass (when anything was listed) + permutation into token order
hipError_t launch_gather(const MaskArgs &a, hipStream_t s);
// Per-device address of the static device array behind the entry point that may not allocate.
hipError_t scratch_init(int device);            // resolves it once per device; `device` must be current
void *scratch_ptr(int device);                  // null before scratch_init(device) has succeeded
hipError_t launch_clear_words(uint32_t *p, uint32_t n_words, hipStream_t s);   // a fill kernel (no memset node in a captured graph)
// What zf_compile derives from the vocabulary on the device (zf_vocab.hip): rows of the token-mask cache over n strings, `words` words each, rows of
// the Q DFA states and then of the N nonterminals; both: (valid, undecided) pairs, or valid and undecided apart; counts: [Q + N] undecided strings per row,
// added to (null: not counted).  first_off / first_state: per nonterminal, the start states of the terminals that can begin it.
struct VocabRows {
    const uint8_t *bytes, *cls, *qflags;
    const uint16_t *delta;             // [Q][n_cls] next state, DFA_DEAD = none
    const uint32_t *first_off, *first_state;
    const uint16_t *behind, *follow;   // what may follow a terminal (Follow): [Q] state behind it, [states][n_cls] next state
    const uint16_t *sure_behind, *sure_next;   // what every context takes behind it, likewise
    uint2 *both;
    uint32_t *valid, *undecided, *counts;
    uint32_t n, words, Q, N, n_cls;
};
hipError_t launch_vocab_rows(const VocabRows &a, const int64_t *off, hipStream_t s);    // tokens: offsets of 64 bits
hipError_t launch_vocab_rows(const VocabRows &a, const uint32_t *off, hipStream_t s);   // strings in rank order
hipError_t launch_vocab_tokens(const int64_t *off, const uint8_t *bytes, const uint8_t *cls, uint32_t n, Str16 *out, hipStream_t s);
hipError_t launch_vocab_strings(const uint32_t *off, const uint8_t *bytes, const uint8_t *cls, uint32_t n, uint8_t *str_cls, Str16 *out, hipStream_t s);
hipError_t launch_apply_mask(const void *logits, void *out, int dtype, int batch, int64_t row_stride, int V, int W,
                             const uint32_t *mask, hipStream_t s);

}  // namespace zf
