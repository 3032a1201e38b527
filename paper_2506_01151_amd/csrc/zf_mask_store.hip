// Mask kernel over the persistent automaton (zf_options.walk_mode = 2): mask_store_kernel, with the
// kernels that set the store up and bring a row's chart into it.
//
// Every Earley set is named by its content: its items, each with the NAME of the set its rule started
// in (not a position in some row's chart).  Named that way the sets of all rows and of all decode
// steps are the states of ONE deterministic automaton over byte classes, kept in device memory for
// the life of the engine:
//   - feeding the token that was just decoded (Section 4.1: the update after every decoding step) is
//     a walk of its bytes through the automaton from the row's current state: the host sends the
//     bytes, not the chart;
//   - the per-step token check walks every undecided vocabulary string through the same table;
//   - a transition is computed by one wavefront-cooperative Earley byte step (Scan + Complete with
//     tabulated Predict, Section 3.2) the first time any row, token or step needs it, and is a
//     look-up for everybody ever after (the reuse across steps that Sections 4.4 and 5.2 aim at).
// A state refers only to the sets its items started in, transitively, which is exactly what
// ZapFormat's reachability closure keeps of a chart (Section 4.2.3); completed items are dropped
// when a set is closed (Figure 3, first rule).  Nothing is ever removed from the store: when it
// fills up the host clears it and the rows come back in from their host charts (import_kernel).
//
// Concurrency.  A transition entry goes NONE -> BUSY -> final value, once; whoever swaps NONE for
// BUSY computes it; everybody else polls (the owner is a running wavefront that waits for nothing,
// so the wait ends; it is bounded all the same).  A new state is written completely (items, dead
// transitions, header) and released at device scope before any entry or hash-table slot names it.
// Table entries are read with device-scope atomic loads (they bypass the per-CU cache); a
// wavefront makes an acquire fence before it reads items it learnt of through such a load.
#include "zf_kernel_common.h"
#include "zf_aut_step.h"

namespace zf {
namespace {

static const uint32_t STORE_ROOT = 1;                  // the state of the empty prefix
static const uint32_t UNPUBLISHED = 0xFFFFFFFFu;
static const int LC_BITS = STORE_LC_BITS;               // block-local cache of table entries
static const uint32_t LC_ENTRIES = 1u << LC_BITS;
static const unsigned long long LC_EMPTY = 0xFFFFFFFF00000000ull;

__device__ __forceinline__ uint32_t g_load(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void g_store_release(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ bool t_final(uint32_t t) { return t != AT_NONE && t != AT_BUSY; }
// A table entry changes NONE -> BUSY -> final value and never again, so a copy read through the caches is either
// right or "not there yet": look-ups read through the caches first and ask device memory (an atomic load, or the
// compare-and-swap that claims the entry) only when the cached answer is not final.

// Hundreds of wavefronts of a group can wait for the same entry: they ask less and less often, so that their polls do not
// slow the memory channel the owner works through.  A byte step takes 3 to 10 us; the pauses are 24, 64 and 100 times 64 cycles (0.6, 1.7,
// 2.7 us; at 8, 24 and 64 times, which was enough when rows had blocks of their own and fewer wavefronts waited, calls of
// 5 to 8 steps took 46.5 instead of 45 us; at 48, 100 and 127 times 44).
__device__ __forceinline__ void poll_pause(uint32_t spins) {
    if (spins < 2) __builtin_amdgcn_s_sleep(24);
    else if (spins < 6) __builtin_amdgcn_s_sleep(64);
    else __builtin_amdgcn_s_sleep(100);
}

struct Staging { uint32_t *ctl; uint8_t *smem; const uint8_t *blob; uint32_t n16; uint8_t *rep; const uint8_t *rep_src; uint32_t ncls; bool wide_sets; };   // what ensure_tables needs; wide_sets: the rows' charts hold sets of many items
// The grammar tables are needed only by a wavefront that computes a transition, which is rare once the automaton has
// grown: the first such wavefront of a block copies them into LDS (ctl[4]: 0 = not there, 1 = being copied, 2 = there).
__device__ __forceinline__ bool ensure_tables(const Staging &g, uint32_t lane) {
    uint32_t *ctl = g.ctl;
    uint8_t *smem = g.smem;
    const uint8_t *blob = g.blob;
    const uint32_t n16 = g.n16;
    uint32_t st = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_load(&ctl[4]));
    if (st == 0) {
        uint32_t old = 0;
        if (lane == 0) old = atomicCAS(&ctl[4], 0u, 1u);
        old = (uint32_t)__builtin_amdgcn_readfirstlane((int)old);
        if (old == 0) {
            const uint4 *src = reinterpret_cast<const uint4 *>(blob);
            uint4 *dst = reinterpret_cast<uint4 *>(smem);
            for (uint32_t k0 = 0; k0 < n16; k0 += 64 * 8) {   // eight 16-byte loads in flight per lane
                uint4 x[8];
#pragma unroll
                for (int u = 0; u < 8; u++) { const uint32_t k = k0 + (uint32_t)u * 64 + lane; x[u] = k < n16 ? src[k] : make_uint4(0, 0, 0, 0); }
#pragma unroll
                for (int u = 0; u < 8; u++) { const uint32_t k = k0 + (uint32_t)u * 64 + lane; if (k < n16) dst[k] = x[u]; }
            }
            for (uint32_t k = lane; k < g.ncls; k += 64) g.rep[k] = g.rep_src[k];   // one byte of every class
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            if (lane == 0) lds_store(&ctl[4], 2u);
            return true;
        }
        st = old;
    }
    for (uint32_t spins = 0; st != 2 && spins < (uint32_t)AUT_SPIN_LIMIT; spins++) {   // the copying wavefront waits for nothing
        __builtin_amdgcn_s_sleep(2);
        st = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_load(&ctl[4]));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    return st == 2;
}

struct StoreSets {             // resolves the name of a set to its items (device memory)
    const StoreView &G;
    uint32_t *errors;
    __device__ __forceinline__ uint2 item(uint64_t h, uint32_t i) const { return reinterpret_cast<const uint2 *>((uintptr_t)h)[i]; }
    __device__ __forceinline__ void view(uint32_t ref, uint64_t &p, uint32_t &n) const {   // the handle is the address of the set's first item
        uint2 h = make_uint2(0, 0);
        if (ref < G.cap_states) h = G.hdr[ref];
        // a name that leads nowhere cannot come from a correct store: read nothing, and fail the call loudly
        if (ref >= G.cap_states || h.y > G.cap_items || h.x > G.cap_items - h.y) { h = make_uint2(0, 0); atomicAdd(errors, 1u); }
        p = (uint64_t)(uintptr_t)(G.arena + h.x);
        n = h.y;
    }
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct Scratch { uint32_t *w, *o, *h; uint32_t cap; };   // one wavefront's set under construction (+ hash table of the wide step)

// Lane l: the sum of the lanes up to l (data-parallel-primitive moves, no trip through LDS).
__device__ __forceinline__ uint32_t wave_sums(uint32_t x) {
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);    // row_shr:1
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);    // row_shr:2
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);    // row_shr:4
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);    // row_shr:8
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
    return x;
}

// A set's signature does not depend on the order of its items (the host, which fills the store when the engine is compiled, the
// narrow and the wide byte step each make them in an order of their own): the sum of its items' words, closed with their count.
__host__ __device__ __forceinline__ uint32_t item_sum(uint32_t w, uint32_t o) {
    uint32_t x = (w * 0x9E3779B1u) ^ (o * 0x85EBCA77u);
    x ^= x >> 15; x *= 0x2C1B3C6Du; x ^= x >> 13;
    return x * 0x297A2D39u;
}
__host__ __device__ __forceinline__ uint32_t set_signature(uint32_t sum, uint32_t n) { const uint32_t h = (sum ^ n) * 0x9E3779B1u; return (h ^ h >> 16) | 1u; }   // never 0: 0 marks a free slot of the hash table

// true when state `id` holds exactly the `kept` items in the scratch, in whatever order
__device__ __forceinline__ bool same_content(const StoreView &G, uint32_t id, const Scratch &sc, uint32_t kept, uint32_t lane) {
    if (id == 0 || id >= G.cap_states) return false;
    const uint2 hj = G.hdr[id];
    if (hj.y != kept || hj.x > G.cap_items - kept) return false;
    unsigned long long diff = 0;
    for (uint32_t i0 = 0; i0 < kept; i0 += 64) {
        bool ne = false;
        if (i0 + lane < kept) { const uint2 x = G.arena[hj.x + i0 + lane]; ne = x.x != lds_load(&sc.w[i0 + lane]) || x.y != lds_load(&sc.o[i0 + lane]); }
        diff |= __ballot(ne);
    }
    if (diff == 0) return true;
    // another order, if it is the same set: both hold each item once, so it is when every one of these is among those
    for (uint32_t i0 = 0; i0 < kept; i0 += 64) {
        const bool mine = i0 + lane < kept;
        const uint32_t w = mine ? lds_load(&sc.w[i0 + lane]) : 0u, o = mine ? lds_load(&sc.o[i0 + lane]) : 0u;
        bool found = !mine;
        for (uint32_t j0 = 0; j0 < kept && __ballot(!found); j0 += 64) {
            uint2 x = make_uint2(0, 0);
            if (j0 + lane < kept) x = G.arena[hj.x + j0 + lane];
            const uint32_t n = kept - j0 < 64u ? kept - j0 : 64u;
            for (uint32_t j = 0; j < n; j++) found |= w == (uint32_t)__builtin_amdgcn_readlane((int)x.x, (int)j) && o == (uint32_t)__builtin_amdgcn_readlane((int)x.y, (int)j);
        }
        if (__ballot(!found)) return false;
    }
    return true;
}

// The transition of state s on class cl: one Earley byte step, then the state that holds the
// resulting set -- found by content in the store's hash table, or made.  Uniform over the wavefront.
// Returns a state id, AT_DEAD, AT_SINK or AT_FAIL (no room in the scratch or in the store).
__device__ __forceinline__ uint32_t store_transition(const TV &T, const StoreView &G, const Scratch &sc, const Staging &stg, uint32_t *errors,
                                                     uint32_t s, uint32_t cl, uint32_t lane) {
    if (!ensure_tables(stg, lane)) return AT_FAIL;
    const uint8_t *rep = stg.rep;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");      // s and every set it refers to were released before the entry that led here
    const StoreSets S{G, errors};
    uint32_t nnew = 0, kept = 0;
    uint64_t src_p;
    uint32_t src_n;
    S.view(s, src_p, src_n);
    const uint32_t byte = rep[cl];
    // the narrow step takes sets of up to 64 items; where the charts hold wide sets (an ambiguous grammar) a source set of more
    // than a few items rarely leaves a narrow one, and the narrow step's one-candidate-at-a-time Complete would be wasted
    const bool wide_first = src_n > 64u || (stg.wide_sets && src_n > (uint32_t)AUT_NARROW_SET_MAX);
    int st = wide_first ? (int)AUT_WIDE : aut_step_narrow<true>(T, S, sc.w, sc.o, sc.cap, s, byte, cl, lane, nnew, kept);
    if (st == AUT_WIDE) st = aut_step_wide(T, S, sc.w, sc.o, sc.h, sc.cap, s, byte, cl, lane, nnew, kept);
    if (st != AUT_OK) return AT_FAIL;
    if (nnew == 0) return AT_DEAD;
    if (kept == 0) return AT_SINK;
    uint32_t sum = 0;
    for (uint32_t i0 = 0; i0 < kept; i0 += 64) if (i0 + lane < kept) sum += item_sum(lds_load(&sc.w[i0 + lane]), lds_load(&sc.o[i0 + lane]));
    sum = wave_sums(sum);
    const uint32_t h = set_signature((uint32_t)__builtin_amdgcn_readlane((int)sum, 63), kept);
    uint32_t slot = (h * 0x9E3779B1u) & G.intern_mask;
    for (uint32_t probes = 0; probes <= G.intern_mask; probes++) {
        const unsigned long long e = __hip_atomic_load(&G.intern[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (e == 0) break;
        if ((uint32_t)(e >> 32) == h) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // the state was released before its slot was written
            if (same_content(G, (uint32_t)e, sc, kept, lane)) return (uint32_t)e;
        }
        slot = (slot + 1) & G.intern_mask;
    }
    uint32_t id = 0, at = 0;
    if (lane == 0) { id = atomicAdd(&G.ctl[0], 1u); at = atomicAdd(&G.ctl[1], kept); }
    id = (uint32_t)__builtin_amdgcn_readfirstlane((int)id);
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    if (id >= G.cap_states || at > G.cap_items - kept) { if (lane == 0) atomicAdd(&G.ctl[2], 1u); return AT_FAIL; }   // the store is full
    for (uint32_t i0 = 0; i0 < kept; i0 += 64)
        if (i0 + lane < kept) G.arena[at + i0 + lane] = make_uint2(lds_load(&sc.w[i0 + lane]), lds_load(&sc.o[i0 + lane]));
    uint32_t *row = G.trans + (size_t)id * T.ncls;
    aut_mark_dead<true>(T, T.ncls, rep, [&](uint32_t i) { return lds_load(&sc.w[i]); }, kept, lane, [&](uint32_t c) { row[c] = AT_DEAD; });
    if (lane == 0) G.hdr[id] = make_uint2(at, kept);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");      // items, dead entries and header before anything that names the state
    for (uint32_t probes = 0; probes <= G.intern_mask; probes++) {
        unsigned long long old = 0;
        if (lane == 0) old = atomicCAS(&G.intern[slot], 0ull, ((unsigned long long)h << 32) | id);
        old = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(old >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)old);
        if (old == 0) return id;
        if ((uint32_t)(old >> 32) == h) {                    // somebody made the same set meanwhile: theirs is the name
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (same_content(G, (uint32_t)old, sc, kept, lane)) return (uint32_t)old;
        }
        slot = (slot + 1) & G.intern_mask;
    }
    return id;                                               // the table has twice as many slots as states: not reached
}

// The same with the LDS laid out: cache of table entries, staging flag, verdict words; then the staged tables, class representatives, scratch.
// In line, and with D and G loaded once at the kernel's head: as a function of its own that read them at every call a chain of byte
// steps took 13 % longer (kernel time of 16 rows of a JSON schema from an empty store, calls of 17 to 32 steps: 74.5 us that way, 71 in line with
// the loads in place, 66 like this; 64 rows of the query language, calls of 33 to 64 steps: 94, 91.5, 82).
static const uint32_t SCRATCH_WIDE = 1u << 16;           // with the scratch's capacity (at most LANE_CAP_MAX) below and the wavefront's number above it
static const uint32_t TABLES_AT = LC_ENTRIES * 8 + 32 + STORE_WAVES * 64 * 4;
template <int MODE>
__device__ __forceinline__ uint32_t store_transition_at(const DeviceTables &D, const StoreView &G, uint8_t *smem, uint32_t how, uint32_t *errors, uint32_t s, uint32_t cl) {
    const uint32_t lane = threadIdx.x & 63u;
    uint8_t *const tables_at = smem + TABLES_AT;
    TV T;
    uint32_t off = table_view<MODE>(D, tables_at, T);
    const uint32_t n16 = off / 16;
    uint8_t *l_rep = tables_at + off; off += 256;
    const Staging stg{reinterpret_cast<uint32_t *>(smem + LC_ENTRIES * 8), tables_at, D.table_blob, n16, l_rep, D.cls_rep, (uint32_t)D.n_cls, (how & SCRATCH_WIDE) != 0};
    Scratch sc;
    sc.cap = how & 0xFFFFu;
    sc.w = reinterpret_cast<uint32_t *>(tables_at + off) + (size_t)(how >> 24) * (2 * sc.cap + aut_hash_places(sc.cap));
    sc.o = sc.w + sc.cap;
    sc.h = sc.o + sc.cap;
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)store_transition(T, G, sc, stg, errors, s, cl, lane));
}

// Look a transition up for the whole wavefront (uniform arguments), computing it if nobody has.
template <class Compute>
__device__ __forceinline__ uint32_t store_lookup_uniform(uint32_t *entry, uint32_t lane, Compute compute) {
    // the read through the caches answers at once when the entry is final; else the claim itself (a compare-and-swap,
    // which returns what device memory holds) is the fresh read
    uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)__hip_atomic_load(entry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT));
    if (t_final(t)) return t;
    if (lane == 0) t = atomicCAS(entry, (uint32_t)AT_NONE, (uint32_t)AT_BUSY);
    t = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
    if (t == AT_NONE) {
        const uint32_t r = compute();
        if (lane == 0) g_store_release(entry, r);            // everything the transition wrote, then the entry
        return r;
    }
    for (uint32_t spins = 0; !t_final(t) && spins < (uint32_t)AUT_SPIN_LIMIT; spins++) {   // the owner is a running wavefront that waits for nothing
        poll_pause(spins);
        t = (uint32_t)__builtin_amdgcn_readfirstlane((int)g_load(entry));
    }
    return t_final(t) ? t : (uint32_t)AT_FAIL;
}

// The status of a call goes to the host from the block that finishes last: every block draws a ticket, which carries the block's
// failed walks and byte steps along (bits 0-15 blocks, 16-39 failures, 40-63 steps), so that the one that draws the last ticket
// has the sums in hand and nothing is left to be read.  A few blocks draw from one word; more blocks draw from one word per
// sixteen of them first (additions to one word queue up at the memory channel that holds it, about 15 ns each).  There are two
// sets of words, taken in turns: a kernel's first wavefront clears the other set, which the kernel before has done with and the
// one behind will draw from, so that nothing of it is outstanding when the status goes out.
//   The words of the status go out as system-scope stores that each carry the call's number, so there is no order to keep
// between them and no release, which would write back an L2 full of masks and logits first (the closing sequence of two
// tickets, counters read back and a release took 3 us of a 12 us kernel at one row).
__device__ __forceinline__ void hand_over_store(const StoreArgs &a, const uint32_t *blk) {
    const uint32_t n_blocks = gridDim.x, lin = blockIdx.x;
    const uint32_t n_groups = n_blocks <= 48u ? 1u : (n_blocks / 16u < (uint32_t)STORE_TICKET_GROUPS ? n_blocks / 16u : (uint32_t)STORE_TICKET_GROUPS);
    const uint32_t g = lin % n_groups, size = n_blocks / n_groups + (g < n_blocks % n_groups ? 1u : 0u);
    const unsigned long long err = lds_load(&blk[0]), stp = lds_load(&blk[1]);
    unsigned long long mine = 1ull | (err < 4095ull ? err : 4095ull) << 16 | (stp < 4095ull ? stp : 4095ull) << 40;
    unsigned long long sum = atomicAdd(&a.tickets[g * STORE_TICKET_STRIDE], mine) + mine;
    if ((sum & 0xFFFFull) != size) return;
    if (n_groups > 1u) {
        mine = (sum & ~0xFFFFull) | 1ull;
        sum = atomicAdd(&a.tickets[STORE_TICKET_GROUPS * STORE_TICKET_STRIDE], mine) + mine;
        if ((sum & 0xFFFFull) != n_groups) return;
    }
    auto tell = [&](uint32_t k, uint32_t value) {
        __hip_atomic_store(&a.status[k], ((unsigned long long)a.seq << 32) | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };
    const uint32_t steps = (uint32_t)(sum >> 40);
    uint32_t more = 0;
    if (steps || a.report_size) {                            // the store has grown: how far
        const uint32_t *ctl = a.konst->view.ctl;
        const uint32_t c0 = g_load(&ctl[0]), c1 = g_load(&ctl[1]), c2 = g_load(&ctl[2]);
        tell(STORE_ST_STEPS, steps);
        tell(STORE_ST_STATES, c0);
        tell(STORE_ST_ITEMS, c1);
        tell(STORE_ST_REFUSED, c2);
        more = STORE_ST_MORE;
    }
    tell(STORE_ST_DONE, ((uint32_t)(sum >> 16) & 0xFFFFFFu) | more);
}

// A piece of 16 bytes of a row of logits, wherever the row begins (rows of a vocabulary that is no multiple of a piece lie at
// any multiple of an element; the memory system takes such accesses as they are).
template <int APPLY> struct Piece { typedef u32x4 __attribute__((aligned(4))) type; };
template <> struct Piece<2> { typedef u32x4 __attribute__((aligned(2))) type; };

// Grid: the blocks of all groups, blocks of STORE_WAVES wavefronts.  A group = the rows of the call that stand in the same state:
// they have the same mask, which is worked out once and stored to every one of them.  The kernel works in TOKEN order and writes
// the caller's mask rows itself: nothing has to be permuted afterwards.  The wavefronts of a block work on their own; what they
// share is the block's LDS cache of table entries and (once somebody needs them) the staged grammar tables.  A wavefront
//  (a) takes its group's record -- start state, pending bytes, token-mask-cache row numbers, member rows -- from the kernel's
//      argument block;
//  (b) requests the token-mask cache words (Section 4.3) of its segment of mask words, and while they are on their way walks the
//      group's pending bytes (the tokens fed since its state was last known) from that state to the current one, then warms the
//      LDS cache with the current state's table row;
//  (c) takes the undecided tokens of the segment, 64 at a time, one lane per token, through the transition table: first the
//      LDS cache, then device memory, and an Earley byte step for what nobody has computed yet;
//  (d) stores the segment's words to the mask rows of the group's members and, in the APPLY builds (1 = fp32, 2 = bf16), masks the
//      segment of their logits (Section 3.3).
// A group served by the state cache (STORE_ROW_POOLED) takes the words from the pool in (b) and skips (c).
// No block-wide barrier between the first one and the hand-over of the call's status at the end.
template <int MODE, int APPLY>
__global__ __launch_bounds__(STORE_BLOCK, STORE_BLOCKS_PER_CU) void mask_store_kernel(StoreArgs a, StoreInline in) {
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ uint32_t blk[2];                              // the block's failed walks and Earley byte steps
    const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // LDS: the cache of table entries, the staging flag and the verdict words come first, at offsets that do not depend on the
    // kernel's arguments: they are cleared while the arguments are still on their way
    unsigned long long *lc = reinterpret_cast<unsigned long long *>(smem);
    uint32_t *ctl = reinterpret_cast<uint32_t *>(smem + LC_ENTRIES * 8);   // [4] state of the staged tables
    uint32_t *vbuf = reinterpret_cast<uint32_t *>(smem + LC_ENTRIES * 8 + 32) + wave * 64;   // per wavefront: verdicts of the pass's words
    for (uint32_t k = tid; k < LC_ENTRIES; k += STORE_BLOCK) lc[k] = LC_EMPTY;
    if (tid < 2) blk[tid] = 0;
    if (tid == 0) ctl[4] = 0;
    __syncthreads();
    const uint32_t W = a.W, ncls = a.ncls;
    // The record of the block's group.  Which group that is is known only once the groups' first blocks have been read, and the
    // record only after that: so lane l asks for the first block AND the twelve words of the record of group l, all at once,
    // and the wavefront picks its group's out of the lanes (one trip to the argument block instead of two, one after the
    // other).  Calls of more groups say which group a block belongs to in device memory.
    static_assert(STORE_INLINE_GROUPS == 64 && sizeof(StoreGroup) == 48, "one short record per lane");
    uint32_t rec = 0, group, part, parts;                    // rec: lane k holds word k of the record
    if (!a.groups) {
        const uint4 *gp = reinterpret_cast<const uint4 *>(&in.g[lane]);
        const uint4 r0 = gp[0], r1 = gp[1], r2 = gp[2];
        const uint32_t fbv = in.first_block[lane], fbv2 = in.first_block[lane + 1u];
        group = (uint32_t)__popcll(__ballot(blockIdx.x >= fbv)) - 1u;    // groups that start at or before this block (0xFFFF beyond the call's groups)
        const uint32_t rw[12] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w, r2.x, r2.y, r2.z, r2.w};
#pragma unroll
        for (int k = 0; k < 12; k++) asm("v_writelane_b32 %0, %1, %2" : "+v"(rec) : "s"(__builtin_amdgcn_readlane((int)rw[k], (int)group)), "n"(k));
        const uint32_t fb0 = (uint32_t)__builtin_amdgcn_readlane((int)fbv, (int)group), fb1 = (uint32_t)__builtin_amdgcn_readlane((int)fbv2, (int)group);
        part = blockIdx.x - fb0;
        parts = fb1 - fb0;
    } else {
        const uint32_t b0 = a.block_of[2u * blockIdx.x], b1 = a.block_of[2u * blockIdx.x + 1u];
        group = (uint32_t)__builtin_amdgcn_readfirstlane((int)b0);
        parts = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b1 >> 16));
        part = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b1 & 0xFFFFu));
        if (lane < 12u) rec = reinterpret_cast<const uint32_t *>(a.groups + group)[lane];
    }
    auto word = [&](uint32_t k) { return (uint32_t)__builtin_amdgcn_readlane((int)rec, (int)k); };
    const uint32_t meta = word(1), flags = (meta >> 16) & 0xFFu, sw = (meta >> 24) + 1u;   // sw: mask words a wavefront takes per pass
    const uint32_t keep_slot = word(10) >> 16, member_at = word(11) & 0xFFFFu, n_members = word(11) >> 16;
    // lanes per copy of the segment: the wavefront holds the segment's words 64 / slots times over, and each copy ORs its
    // share of the group's cache rows (16 words: four copies; up to 64 words -- groups few of whose tokens are undecided: one)
    const uint32_t slots_log2 = sw <= 16u ? 4u : (sw <= 32u ? 5u : 6u), slots = 1u << slots_log2, n_grp = 64u >> slots_log2;
    const uint32_t n_seg = (W + sw - 1) / sw;
    const uint32_t unit = part * STORE_WAVES + wave, n_units = parts * STORE_WAVES;   // a unit = one wavefront of one of the group's blocks
    const bool pooled = (flags & STORE_ROW_POOLED) != 0;
    if (unit < n_seg || unit == 0) {                         // the group's first wavefront reports its state even when there is no mask word
    uint32_t start = word(0), n_pending = meta & 0xFFu, n_ent = (meta >> 8) & 0xFFu, pend_off = 0, ent_off = 0;
    const bool spilled = (flags & STORE_ROW_SPILL) != 0;
    if (spilled) {                                           // the full record in its place
        rec = lane < sizeof(StoreRow) / 4 ? reinterpret_cast<const uint32_t *>(a.spilled + group)[lane] : 0u;
        n_pending = word(1); pend_off = word(2); n_ent = word(3); ent_off = word(4);
    }
    if (flags & STORE_ROW_IMPORTED) start = a.import_root[group];
    const bool use_cache = (flags & STORE_ROW_CACHE) != 0;
    const bool ent_inline = n_ent <= (uint32_t)(spilled ? STORE_ROW_ENT : STORE_GROUP_ENT);
    auto entry = [&](uint32_t k) -> uint32_t {               // number of the group's cache row k, uniform (only of an inline list)
        return spilled ? word(STORE_ROW_ENT_AT + k) : (word(6u + (k >> 1)) >> ((k & 1u) * 16u)) & 0xFFFFu;
    };
    auto pending = [&](uint32_t k) -> uint32_t {
        if (spilled && n_pending > (uint32_t)STORE_ROW_PEND) return (uint32_t)a.pending[pend_off + k];
        return (word((spilled ? (uint32_t)STORE_ROW_PEND_AT : 2u) + (k >> 2)) >> ((k & 3u) * 8u)) & 0xFFu;
    };
    uint32_t root = AT_FAIL, steps = 0;
    uint32_t *errors = &blk[0];
    const DeviceTables tables = a.konst->tab;                // what a byte step reads of them, on its way while the record is looked at
    const StoreView store = a.konst->view;
    if (blockIdx.x == 0 && wave == 0) clear_tickets(a.tickets_next, lane);   // (a store ahead of the two would make vector loads of their scalar ones)
    const uint32_t slot16 = lane & (slots - 1u), grp = lane >> slots_log2;    // lane = (word of the segment, which copy)
    // The token-mask cache words of segment g: every copy ORs its share of the group's cache rows.  The first three rounds stay
    // as they were loaded until they are needed (an OR here would wait for them here), which covers three to twelve cache rows.
    constexpr int RAW = 3;
    struct Words { uint32_t v[RAW], c[RAW], v_more, c_more; };
    auto request = [&](uint32_t g) __attribute__((always_inline)) -> Words {
        Words x;
        const uint32_t w = slot16 < sw && g < n_seg ? g * sw + slot16 : 0xFFFFFFFFu;
#pragma unroll
        for (int j = 0; j < RAW; j++) { x.v[j] = 0; x.c[j] = 0; }
        x.v_more = 0; x.c_more = use_cache || pooled ? 0u : 0xFFFFFFFFu;
        if (pooled) { if (w < W) x.v[0] = a.pool[(size_t)start * W + w]; return x; }
        if (!use_cache || g >= n_seg) return x;
        // the number of cache row k0 + (the lane's copy): the copies' numbers are read out of the record one by one (lane reads
        // with a uniform index: no trip through LDS, which a shuffle would be) and each lane keeps its copy's
        auto one = [&](uint32_t k0, uint32_t &v, uint32_t &c) __attribute__((always_inline)) {
            uint32_t er = 0;
            if (ent_inline) for (uint32_t j = 0; j < n_grp; j++) { const uint32_t ej = entry(k0 + j < n_ent ? k0 + j : 0u); er = grp == j ? ej : er; }
            const uint32_t k = k0 + grp;
            if (k < n_ent && w < W) {
                if (!ent_inline) er = a.entries[ent_off + k];
                const size_t r = (size_t)er * W + w;
                const uint2 vc = a.cache[r];
                v = vc.x; c = vc.y;
            }
        };
#pragma unroll
        for (int j = 0; j < RAW; j++) if ((uint32_t)j * n_grp < n_ent) one((uint32_t)j * n_grp, x.v[j], x.c[j]);
        for (uint32_t k0 = (uint32_t)RAW * n_grp; k0 < n_ent; k0 += n_grp) { uint32_t v = 0, c = 0; one(k0, v, c); x.v_more |= v; x.c_more |= c; }
        return x;
    };
    // the first look-up of the pending walk is requested ahead of the cache words: loads come back in the order they were issued
    uint32_t hop0 = AT_NONE;
    const bool start_ok = start != 0 && start < a.cap_states;
    if (n_pending && start_ok && pending(0) < ncls) hop0 = __hip_atomic_load(&a.trans[start * ncls + pending(0)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    Words wd = request(unit);
    // the group's rows: lane l holds the l-th of the 64 in hand (a larger group goes through them 64 at a time)
    auto members_from = [&](uint32_t m0) __attribute__((always_inline)) -> uint32_t {
        const uint32_t k = member_at + m0 + lane;
        return m0 + lane < n_members ? (a.members ? a.members[k] : in.member[k]) : 0u;
    };
    uint32_t members = members_from(0);
    // Logits (APPLY builds): the segment's 16-byte pieces of all members in hand as ONE run -- the first member's pieces, then the
    // second's, ... -- so that every lane has one to move whatever the width of the segment, and so that the pieces of
    // several members travel together (one member after the other, a memory round trip each, cost a group of 16 rows 8 us).  The
    // first PRE pieces of every lane are requested one pass ahead (those of the first segment here): they wait in registers when
    // the segment's verdicts are in.
    typedef typename Piece<APPLY>::type piece_t;
    constexpr uint32_t tp = APPLY == 2 ? 8u : 4u, esz = APPLY == 2 ? 2u : 4u;   // tokens per 16-byte piece, bytes per logit
    auto tokens_of = [&](uint32_t g) -> uint32_t {
        const uint32_t tok0 = g * sw * 32u;
        return g < n_seg && tok0 < a.V ? (sw * 32u < a.V - tok0 ? sw * 32u : a.V - tok0) : 0u;
    };
    // number i of a run of `per` things per member: which member, and which of its things.  i < 2^15 and per <= 512, so the
    // half added keeps the product at least 1 / 1024 away from the next whole number, far more than single precision loses
    auto split = [&](uint32_t i, uint32_t per, float inv, uint32_t &k) -> uint32_t { k = (uint32_t)(((float)i + 0.5f) * inv); return i - k * per; };
    auto byte_of = [&](uint32_t k, uint32_t g, uint32_t t) -> size_t {   // of token t of segment g in the k-th member's row
        return ((size_t)(uint32_t)__shfl((int)members, (int)(k & 63u)) * (size_t)a.stride + g * sw * 32u + t) * esz;
    };
    constexpr int PRE = 2;
    auto logits_ahead = [&](uint32_t g, u32x4 (&pre)[PRE]) __attribute__((always_inline)) {
        const uint32_t per = tokens_of(g) / tp, total = per * (n_members < 64u ? n_members : 64u);
        const float inv = __builtin_amdgcn_rcpf((float)(per ? per : 1u));
#pragma unroll
        for (int u = 0; u < PRE; u++) {
            const uint32_t i = (uint32_t)u * 64u + lane;
            uint32_t k;
            const uint32_t p = split(i < total ? i : 0u, per, inv, k);
            const size_t at = byte_of(k, g, p * tp);
            pre[u] = u32x4{0, 0, 0, 0};
            if (i < total) pre[u] = __builtin_nontemporal_load(reinterpret_cast<const piece_t *>(reinterpret_cast<const uint8_t *>(a.logits) + at));
        }
    };
    u32x4 l_pre[PRE];
    if (APPLY) logits_ahead(unit, l_pre);
    auto transition = [&](uint32_t s, uint32_t cl) __attribute__((always_inline)) -> uint32_t {
        steps++;
        return store_transition_at<MODE>(tables, store, smem, (uint32_t)a.scratch | (a.wide ? SCRATCH_WIDE : 0u) | wave << 24, errors, s, cl);
    };
    auto find_root = [&]() __attribute__((always_inline)) {
        // ---- the group's current state: walk the bytes fed since `start` was its state (the loads above are in flight) ----
        uint32_t s = start;
        bool bad = s == 0 || (s >= a.cap_states && s != AT_SINK);
        for (uint32_t k = 0; k < n_pending && !bad; k++) {
            const uint32_t cl = pending(k);
            if (s == AT_SINK || cl >= ncls) { bad = true; break; }
            uint32_t t = k == 0 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)hop0) : (uint32_t)AT_NONE;
            if (!t_final(t)) t = store_lookup_uniform(a.trans + (size_t)s * ncls + cl, lane, [&]() { return transition(s, cl); });
            if (t == AT_DEAD || t == AT_FAIL) { bad = true; break; }   // the host accepted these bytes: a dead end here is an error
            s = t;
        }
        if (bad) { s = AT_FAIL; if (lane == 0 && unit == 0) atomicAdd(errors, 1u); }
        if (unit == 0 && lane == 0 && (flags & STORE_ROW_REPORT))
            __hip_atomic_store(&a.status[STORE_ST_ROW + group], ((unsigned long long)a.seq << 32) | s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        root = s;
        if (root < AT_FAIL) {
            // Warm the block's cache with the current state's row of the table, and with the rows of the states one byte
            // away (every wavefront of the block takes its share of them): a row is read by neighbouring lanes, once per
            // block.  Left to the walk below, thousands of wavefronts would ask for the same few lines at the same
            // moment, lane by lane, and queue up at the one memory channel that holds them (8 us and more).
            auto warm_row = [&](uint32_t st) __attribute__((always_inline)) {
                for (uint32_t c0 = 0; c0 < ncls; c0 += 64) {
                    const uint32_t cl = c0 + lane;
                    uint32_t t = AT_NONE;
                    const uint32_t key = st * ncls + cl;
                    if (cl < ncls) t = __hip_atomic_load(&a.trans[key], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                    if (cl < ncls && t_final(t) && t != AT_FAIL)
                        __hip_atomic_store(&lc[(key * 0x9E3779B1u) >> (32 - LC_BITS)], ((unsigned long long)key << 32) | t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    // the states this row leads to, each once: the wavefront's share of them is warmed in turn
                    if (st == root) {
                        unsigned long long todo = __ballot(cl < ncls && t < AT_FAIL && t != root);
                        constexpr int SHARE = (STORE_WARM_ROWS + STORE_WAVES - 1) / STORE_WAVES;
                        uint32_t mine[SHARE], n_mine = 0, n_done = 0;
#pragma unroll
                        for (int k = 0; k < SHARE; k++) mine[k] = 0;
                        while (todo && n_done < (uint32_t)STORE_WARM_ROWS) {
                            const int l = __ffsll((long long)todo) - 1;
                            const uint32_t nx = (uint32_t)__builtin_amdgcn_readlane((int)t, l);
                            todo &= ~__ballot(t == nx);
                            if (n_done % STORE_WAVES == wave && ncls <= 64u) {
#pragma unroll
                                for (int k = 0; k < SHARE; k++) mine[k] = n_mine == (uint32_t)k ? nx : mine[k];
                                n_mine++;
                            }
                            n_done++;
                        }
                        uint32_t t2[SHARE];                  // the rows' loads travel together
#pragma unroll
                        for (int k = 0; k < SHARE; k++) {
                            t2[k] = AT_NONE;
                            if ((uint32_t)k < n_mine && lane < ncls) t2[k] = __hip_atomic_load(&a.trans[mine[k] * ncls + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                        }
#pragma unroll
                        for (int k = 0; k < SHARE; k++) {
                            const uint32_t k2 = mine[k] * ncls + lane;
                            if ((uint32_t)k < n_mine && lane < ncls && t_final(t2[k]) && t2[k] != AT_FAIL)
                                __hip_atomic_store(&lc[(k2 * 0x9E3779B1u) >> (32 - LC_BITS)], ((unsigned long long)k2 << 32) | t2[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                    }
                }
            };
            warm_row(root);
        }
    };
    // One token of a batch: where its verdict goes, and its string (requested here, used a batch later).
    struct Tok { uint32_t slot, bit, token; Str16 c16; bool live; };
    uint32_t incl = 0, want = 0;                             // of the segment in hand: running bit counts of its words, undecided bits
    auto fetch = [&](uint32_t g, uint32_t b0, uint32_t total) __attribute__((always_inline)) -> Tok {
        Tok k;
        const uint32_t i = b0 + lane;
        k.live = i < total;
        k.slot = 0;                                          // the word that holds the lane's token: the first whose running count exceeds i (by bisection)
        for (uint32_t half = slots >> 1; half; half >>= 1) k.slot += i >= (uint32_t)__shfl((int)incl, (int)(k.slot + half - 1u)) ? half : 0u;
        const uint32_t before = (uint32_t)__shfl((int)incl, (int)(k.slot ? k.slot - 1 : 0));
        const uint32_t bits = (uint32_t)__shfl((int)want, (int)k.slot);
        uint32_t n = i - (k.slot ? before : 0u);             // the n-th set bit of the word, by halving
        k.bit = 0;
#pragma unroll
        for (int sh = 16; sh >= 1; sh >>= 1) {
            const uint32_t low = (uint32_t)__popc(bits & (((1u << sh) - 1u) << k.bit));
            if (n >= low) { n -= low; k.bit += (uint32_t)sh; }
        }
        k.token = (g * sw + k.slot) * 32u + k.bit;
        k.c16 = Str16{{TOK_END, 0, 0, 0}};
        if (k.live) k.c16 = a.tok16[k.token];                // requested here, looked at a batch later: nothing below waits for it
        return k;
    };
    bool root_ok = pooled;
    // the first pass runs even for a wavefront without a segment (the group's first wavefront reports its state)
    for (uint32_t g = unit, first = 1; first || g < n_seg; g += n_units, first = 0) {
        const uint32_t w = slot16 < sw && g < n_seg ? g * sw + slot16 : 0xFFFFFFFFu;
        uint32_t v = wd.v[0] | wd.v_more, c = wd.c[0] | wd.c_more;
#pragma unroll
        for (int j = 1; j < RAW; j++) { v |= wd.v[j]; c |= wd.c[j]; }
        wd = request(g + n_units);                           // the next segment's words travel while this one's tokens are checked
        u32x4 l_nxt[PRE];
        if (APPLY) logits_ahead(g + n_units, l_nxt);         // and so do its first logits
        if (!pooled) {
            if (slots_log2 <= 4u) { v |= __shfl_xor(v, 16); c |= __shfl_xor(c, 16); }
            if (slots_log2 <= 5u) { v |= __shfl_xor(v, 32); c |= __shfl_xor(c, 32); }
        }
        want = c & ~v;
        {
            const uint32_t t0 = w * 32u;
            if (w >= W || t0 >= a.V) want = 0;
            else if (a.V - t0 < 32u) want &= (1u << (a.V - t0)) - 1u;
        }
        // ---- one lane per undecided token through the table.  The undecided tokens of the segment's words are numbered
        // through (prefix sum of the words' bit counts) and taken 64 at a time, so that a batch is full whatever the
        // pattern of the bits; verdicts go back to their words through LDS.  The strings of a batch are requested one
        // batch ahead; those of the first batch travel while the group's current state is worked out ----
        incl = (uint32_t)__popc(want);                       // every copy holds the same words
        // running sums over each copy's lanes by data-parallel-primitive moves (a row of 16 lanes shifts by 1, 2, 4, 8 with
        // zeros coming in; then the last lane of a row is broadcast into the next row, of the lower half into the upper half):
        // six vector instructions where shuffles would be six trips through LDS
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x111, 0xF, 0xF, true);   // row_shr:1
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x112, 0xF, 0xF, true);   // row_shr:2
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x114, 0xF, 0xF, true);   // row_shr:4
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x118, 0xF, 0xF, true);   // row_shr:8
        if (slots_log2 >= 5u) incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
        if (slots_log2 >= 6u) incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
        uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, (int)(slots - 1u));
        Tok nxt;
        if (total) nxt = fetch(g, 0, total);
        if (first && !pooled) { find_root(); root_ok = root < AT_FAIL; }   // AT_SINK: nothing can follow; AT_FAIL: the call fails
        if (!root_ok) { total = 0; v = 0; }                  // no token can follow a finished sentence
        if (lane < slots) lds_store(&vbuf[lane], 0u);
        for (uint32_t b0 = 0; b0 < total; b0 += 64) {
            const Tok cur = nxt;
            if (b0 + 64 < total) nxt = fetch(g, b0 + 64, total);
            // Where a lane stands with its string, in ONE register: the loop below carries no per-lane truth value from one
            // round to the next.  (Carried truth values live in scalar register pairs, and every one of them costs three
            // scalar instructions per round to merge; the four vector units of a compute unit share one scalar unit, which
            // was what bounded the walk.)
            enum : uint32_t { PH_GO = 0,      // takes a step in the next round
                              PH_NONE = 1,    // waits: nobody has computed the entry it needs
                              PH_BUSY = 2,    // waits: somebody is computing it
                              PH_FAR = 3,     // at the end of the bytes at hand: the next fifteen have to be fetched
                              PH_OK = 4,      // done: the whole string went through (codes from here on: done)
                              PH_DEAD = 5,    // done: the string cannot follow
                              PH_FAIL = 6 };  // done: no room, or a wait that did not end
            // what a step that found no state makes of a lane, a nibble per special value (~value = 0 .. 4): not computed,
            // dead, nothing can follow (the one string that ends right here is picked out below), being computed, no room
            constexpr uint32_t PH_OF_SPECIAL = (PH_NONE << 0) | (PH_DEAD << 4) | (PH_DEAD << 8) | (PH_BUSY << 12) | (PH_FAIL << 16);
            static_assert(AT_NONE == ~0u && AT_DEAD == ~1u && AT_SINK == ~2u && AT_BUSY == ~3u && AT_FAIL == ~4u, "the nibbles above");
            uint32_t w0 = cur.c16.w[0], w1 = cur.c16.w[1], w2 = cur.c16.w[2], w3 = cur.c16.w[3];
            uint32_t cl = w0 & 0xFFu;                        // the class the lane's next step takes
            uint32_t ph = cur.live && cl != TOK_END ? (uint32_t)PH_GO : (uint32_t)PH_DEAD;   // an empty token is never allowed
            uint32_t s = root, pos = 0, spins = 0, rounds = 0, passed = 0;   // passed: classes of the string before the ones at hand
            for (;;) {
                // Every lane follows its own string as far as the table goes: all lanes that can move take a step together,
                // written without branches on per-lane conditions (selects; an entry that is not in the block's LDS cache
                // sits behind a wavefront-uniform test).  No result of a load from device memory is used on the way round
                // when every lane finds its entry: the loop never waits for what was requested ahead (the next batch's
                // strings, the next segment's words and logits).
                ph = ph == PH_NONE || ph == PH_BUSY ? (uint32_t)PH_GO : ph;   // those that waited look again
                for (;;) {
                    const bool go = ph == PH_GO;
                    if (!__builtin_amdgcn_ballot_w64(go)) break;
                    const uint32_t key = __umul24(s, ncls) + cl;             // a state has at most 18 bits, a class 8
                    const uint32_t lslot = go ? (key * 0x9E3779B1u) >> (32 - LC_BITS) : 0u;
                    const unsigned long long e = __hip_atomic_load(&lc[lslot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    const bool hit = (uint32_t)(e >> 32) == key;
                    uint32_t t_new = hit ? (uint32_t)e : (uint32_t)AT_NONE;
                    const bool miss = go & !hit;
                    if (__builtin_amdgcn_ballot_w64(miss)) {
                        if (miss) {
                            // through the caches first; an entry seen unfinished is asked of device memory only on the
                            // way back from the claim below, which is itself a fresh read of the entry it claims
                            t_new = __hip_atomic_load(&a.trans[key], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                            if (!t_final(t_new) && rounds) t_new = g_load(&a.trans[key]);
                            if (t_final(t_new) && t_new != AT_FAIL) __hip_atomic_store(&lc[lslot], ((unsigned long long)key << 32) | t_new, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                    }
                    const uint32_t pos1 = pos + 1u;          // at most 15: the sixteenth byte at hand is a mark, never a class
                    const bool upper = (pos1 & 8u) != 0;
                    const uint32_t c1 = __builtin_amdgcn_perm(upper ? w3 : w1, upper ? w2 : w0, (pos1 & 7u) | 0x0C0C0C00u);   // the class behind it, or a mark
                    const bool state = t_new < AT_FAIL;      // a state: the lane moves on
                    const bool ends = c1 == TOK_END;
                    uint32_t nx = __builtin_amdgcn_ubfe(PH_OF_SPECIAL, (~t_new) << 2, 4u);
                    nx = state ? (c1 == TOK_MORE ? (uint32_t)PH_FAR : (uint32_t)PH_GO) : nx;
                    nx = ((state | (t_new == AT_SINK)) & ends) ? (uint32_t)PH_OK : nx;   // (& and | on purpose: && and || would ask for a branch apiece)
                    const bool adv = go & state;
                    s = adv ? t_new : s;
                    pos = adv ? pos1 : pos;
                    cl = adv ? c1 : cl;
                    ph = go ? nx : ph;
                }
                if (!__builtin_amdgcn_ballot_w64(ph < PH_OK)) break;
                if (__builtin_amdgcn_ballot_w64(ph == PH_FAR)) {   // strings beyond the bytes at hand: the next fifteen classes, then round again
                    if (ph == PH_FAR) {
                        const DeviceTables &D = a.konst->tab;
                        const uint32_t rank = D.rank_of[cur.token], at = D.str_off[rank], len = D.str_off[rank + 1] - at;
                        passed += TOK_AT_HAND;
                        const uint32_t left = len - passed, n = left < TOK_AT_HAND ? left : TOK_AT_HAND;   // left >= 1: the mark says that the string goes on
                        uint32_t nw[4] = {0, 0, 0, 0};
                        for (uint32_t k = 0; k < n; k++) { const uint32_t b = (uint32_t)D.str_cls[at + passed + k] << ((k & 3u) * 8u); nw[0] |= k < 4u ? b : 0u; nw[1] |= (k >> 2) == 1u ? b : 0u; nw[2] |= (k >> 2) == 2u ? b : 0u; nw[3] |= (k >> 2) == 3u ? b : 0u; }
                        const uint32_t mark = (left > TOK_AT_HAND ? TOK_MORE : TOK_END) << ((n & 3u) * 8u);
                        w0 = nw[0] | (n < 4u ? mark : 0u); w1 = nw[1] | ((n >> 2) == 1u ? mark : 0u); w2 = nw[2] | ((n >> 2) == 2u ? mark : 0u); w3 = nw[3] | ((n >> 2) == 3u ? mark : 0u);
                        asm volatile("" : "+v"(w0), "+v"(w1), "+v"(w2), "+v"(w3));   // waited for here, not at the top of the loop above
                        cl = w0 & 0xFFu; pos = 0;
                        ph = PH_GO;
                    }
                    continue;
                }
                rounds++;
                // one of the waiting lanes' transitions is claimed and computed here; the other lanes look again afterwards
                const unsigned long long missing = __builtin_amdgcn_ballot_w64(ph == PH_NONE);
                bool progress = false;
                if (missing) {
                    const int l = __ffsll((long long)missing) - 1;
                    const uint32_t rs = (uint32_t)__builtin_amdgcn_readlane((int)s, l), rc = (uint32_t)__builtin_amdgcn_readlane((int)cl, l);
                    uint32_t old = 0;
                    if (lane == 0) old = atomicCAS(&a.trans[rs * ncls + rc], (uint32_t)AT_NONE, (uint32_t)AT_BUSY);
                    old = (uint32_t)__builtin_amdgcn_readfirstlane((int)old);
                    if (old == AT_NONE) {
                        const uint32_t r = transition(rs, rc);
                        if (lane == 0) g_store_release(&a.trans[rs * ncls + rc], r);   // everything the transition wrote, then the entry
                        progress = true;
                    } else progress = old != AT_BUSY;        // somebody else has it, or has finished it meanwhile
                }
                if (progress) spins = 0;
                else {
                    poll_pause(spins);
                    if (++spins > (uint32_t)AUT_SPIN_LIMIT) ph = ph < PH_OK ? (uint32_t)PH_FAIL : ph;   // bounded wait
                }
                // Nothing this slow path asked of device memory is outstanding when the walk above starts again (vmcnt 0; the
                // other two counters left alone).  Said explicitly, because the compiler otherwise has to assume that one of
                // the loads in here may still be on its way to a register the walk reuses, and waits at the top of the walk on
                // every round -- for the strings, words and logits requested ahead as well.
                __builtin_amdgcn_s_waitcnt(0x0F70);
            }
            if (ph == PH_OK) atomicOr(&vbuf[cur.slot], 1u << cur.bit);
            const unsigned long long fm = __builtin_amdgcn_ballot_w64(ph == PH_FAIL);    // no room in the scratch or the store, or a wait that did not end
            if (lane == 0 && fm) atomicAdd(errors, (uint32_t)__popcll(fm));
        }
        if (total) v |= lds_load(&vbuf[slot16]);             // LDS serves one wavefront's accesses in issue order
        // ---- the segment's words go to every member's mask row (and to the state cache) ----
        for (uint32_t m0 = 0; m0 < n_members; m0 += 64) {
            if (n_members > 64u) members = members_from(m0);
            const uint32_t n = n_members - m0 < 64u ? n_members - m0 : 64u;
            for (uint32_t k = 0; k < n; k++) {
                uint32_t *dst = a.out_mask + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)members, (int)k) * W + w;
                if (lane < slots && w < W) put_word(dst, v, a.complete);
            }
            if (APPLY) {
                // Logit masking (Section 3.3) of the segment's tokens, right here: 16-byte pieces, consecutive lanes on consecutive
                // pieces, the mask word from the lane that holds it.  Allowed logits are copied bit for bit, the others become -inf.
                const uint32_t n_tok = tokens_of(g), pieces = n_tok / tp, tail = n_tok % tp;
                auto masked = [&](u32x4 x, uint32_t mb) -> u32x4 {
                    if (APPLY == 2) {
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            uint32_t e = x[j];
                            if (!((mb >> (2 * j)) & 1u)) e = (e & 0xFFFF0000u) | 0xFF80u;
                            if (!((mb >> (2 * j + 1)) & 1u)) e = (e & 0x0000FFFFu) | 0xFF800000u;
                            x[j] = e;
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; j++) if (!((mb >> j) & 1u)) x[j] = 0xFF800000u;
                    }
                    return x;
                };
                auto bits_at = [&](uint32_t t) -> uint32_t { return (uint32_t)__shfl((int)v, (int)((t >> 5) & 63u)) >> (t & 31u); };   // all lanes call it together
                const uint32_t run = pieces * n;
                const float inv = __builtin_amdgcn_rcpf((float)(pieces ? pieces : 1u));
                const uint8_t *src = reinterpret_cast<const uint8_t *>(a.logits);
                uint8_t *dst = reinterpret_cast<uint8_t *>(a.out);
                auto where = [&](uint32_t i, uint32_t &p) -> size_t { uint32_t k; p = split(i < run ? i : 0u, pieces, inv, k); return byte_of(k, g, p * tp); };
                auto put = [&](uint32_t i, u32x4 x) { uint32_t p; const size_t at = where(i, p); const uint32_t mb = bits_at(p * tp); if (i < run) __builtin_nontemporal_store(masked(x, mb), reinterpret_cast<piece_t *>(dst + at)); };
                uint32_t i0 = 0;
                if (m0 == 0) {                               // what was requested ahead
#pragma unroll
                    for (int u = 0; u < PRE; u++) if ((uint32_t)u * 64u < run) put((uint32_t)u * 64u + lane, l_pre[u]);
                    i0 = PRE * 64u;
                }
                for (; i0 < run; i0 += 256) {                // the others: four pieces per lane in flight
                    u32x4 x[4];
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        const uint32_t i = i0 + (uint32_t)u * 64u + lane;
                        uint32_t p;
                        const size_t at = where(i, p);
                        x[u] = u32x4{0, 0, 0, 0};
                        if (i < run) x[u] = __builtin_nontemporal_load(reinterpret_cast<const piece_t *>(src + at));
                    }
#pragma unroll
                    for (int u = 0; u < 4; u++) if (i0 + (uint32_t)u * 64u < run) put(i0 + (uint32_t)u * 64u + lane, x[u]);
                }
                if (tail) {                                  // the last tokens of a vocabulary that is no multiple of a piece
                    const uint32_t tails = tail * n;
                    const float tinv = __builtin_amdgcn_rcpf((float)tail);
                    for (uint32_t i = 0; i < tails; i += 64) {
                        uint32_t k;
                        const uint32_t t = pieces * tp + split(i + lane < tails ? i + lane : 0u, tail, tinv, k), keep = bits_at(t) & 1u;
                        const size_t at = byte_of(k, g, t);
                        if (i + lane < tails) {
                            if (APPLY == 2) *reinterpret_cast<uint16_t *>(dst + at) = keep ? *reinterpret_cast<const uint16_t *>(src + at) : (uint16_t)0xFF80u;
                            else *reinterpret_cast<uint32_t *>(dst + at) = keep ? *reinterpret_cast<const uint32_t *>(src + at) : 0xFF800000u;
                        }
                    }
                }
            }
        }
        if ((flags & STORE_ROW_KEEP) && lane < slots && w < W) put_word(&a.pool[(size_t)keep_slot * W + w], v, a.complete);
        if (n_members > 64u) members = members_from(0);
        if (APPLY) {
#pragma unroll
            for (int u = 0; u < PRE; u++) l_pre[u] = l_nxt[u];
        }
    }
    if (lane == 0 && steps) atomicAdd(&blk[1], steps);
    }
    if (a.complete) stores_arrived();                        // every word this wavefront wrote has reached memory before the block's ticket is drawn
    __syncthreads();
    if (tid == 0) hand_over_store(a, blk);
}

// Clear the store: every transition unknown, every header unpublished, the hash table empty; then the
// state of the empty prefix, whose items started in that very set.
__global__ __launch_bounds__(256) void store_clear_kernel(StoreView G, uint32_t ncls, const uint2 *root_items, uint32_t n_root) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
    for (size_t k = i; k < (size_t)G.cap_states * ncls; k += stride) G.trans[k] = AT_NONE;
    for (size_t k = i; k < G.cap_states; k += stride) G.hdr[k] = k == STORE_ROOT ? make_uint2(0, n_root) : make_uint2(0, UNPUBLISHED);
    for (size_t k = i; k <= G.intern_mask; k += stride) G.intern[k] = 0;
    for (size_t k = i; k < n_root; k += stride) G.arena[k] = make_uint2(root_items[k].x, STORE_ROOT);
    if (i == 0) { G.ctl[0] = STORE_ROOT + 1; G.ctl[1] = n_root; G.ctl[2] = 0; G.ctl[3] = 0; }
}

// The states the host has filled in get their places in the hash table, one lane per state (sets of a few items), and the store
// its counts.  State 1 is never looked for.
__global__ __launch_bounds__(256) void store_adopt_kernel(StoreView G, uint32_t n_states, uint32_t n_items) {
    const uint32_t id = blockIdx.x * 256 + threadIdx.x;
    if (id == 0) { G.ctl[0] = n_states; G.ctl[1] = n_items; }
    if (id <= STORE_ROOT || id >= n_states) return;
    const uint2 hj = G.hdr[id];
    if (hj.x > n_items || hj.y > n_items - hj.x) return;
    uint32_t sum = 0;
    for (uint32_t i = 0; i < hj.y; i++) { const uint2 x = G.arena[hj.x + i]; sum += item_sum(x.x, x.y); }
    const uint32_t h = set_signature(sum, hj.y);
    uint32_t slot = (h * 0x9E3779B1u) & G.intern_mask;
    for (uint32_t probes = 0; probes <= G.intern_mask; probes++) {
        if (atomicCAS(&G.intern[slot], 0ull, ((unsigned long long)h << 32) | id) == 0ull) return;
        slot = (slot + 1) & G.intern_mask;
    }
}

// Bring rows whose state the store does not know (after the store was cleared, or after more bytes than
// a call carries) in from their host charts: every set of the packed chart becomes a state of its own,
// origins renamed from set indices to the new names.  One block per such row.
__global__ __launch_bounds__(256) void store_import_kernel(StoreView G, const RowChart *charts, const uint32_t *set_off, const Item *items, const uint32_t *group, uint32_t *import_root) {
    __shared__ uint32_t base[2];
    const uint32_t g = group[blockIdx.x];
    const RowChart rc = charts[blockIdx.x];
    if (threadIdx.x == 0) { base[0] = atomicAdd(&G.ctl[0], rc.n_sets); base[1] = atomicAdd(&G.ctl[1], rc.n_items); }
    __syncthreads();
    const uint32_t id0 = base[0], at0 = base[1];
    if (id0 > G.cap_states - rc.n_sets || id0 + rc.n_sets > G.cap_states || at0 > G.cap_items - rc.n_items || rc.n_items > G.cap_items) {
        if (threadIdx.x == 0) { atomicAdd(&G.ctl[2], 1u); import_root[g] = AT_FAIL; }   // the mask kernel, which starts from there, fails the call
        return;
    }
    const uint32_t *so = set_off + rc.set_base;
    const uint2 *it = reinterpret_cast<const uint2 *>(items) + rc.item_base;
    for (uint32_t k = threadIdx.x; k < rc.n_items; k += 256) { const uint2 x = it[k]; G.arena[at0 + k] = make_uint2(x.x, id0 + x.y); }
    for (uint32_t k = threadIdx.x; k < rc.n_sets; k += 256) G.hdr[id0 + k] = make_uint2(at0 + so[k], so[k + 1] - so[k]);
    if (threadIdx.x == 0) import_root[g] = id0 + rc.n_sets - 1;
}

}  // namespace

// the build of the kernel for a table mode and a kind of logits
typedef void (*StoreKernel)(StoreArgs, StoreInline);
static StoreKernel store_kernel(int mode, int apply) {
    static const StoreKernel k[3][3] = {{mask_store_kernel<0, 0>, mask_store_kernel<0, 1>, mask_store_kernel<0, 2>},
                                        {mask_store_kernel<1, 0>, mask_store_kernel<1, 1>, mask_store_kernel<1, 2>},
                                        {mask_store_kernel<2, 0>, mask_store_kernel<2, 1>, mask_store_kernel<2, 2>}};
    return k[mode < 0 ? 0 : (mode > 2 ? 2 : mode)][apply];
}

hipError_t prepare_store_kernels() {
    for (int m = 0; m < 3; m++)
        for (int p = 0; p < 3; p++) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(store_kernel(m, p)), hipFuncAttributeMaxDynamicSharedMemorySize, STORE_LDS_MAX);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

uint32_t store_lds_bytes(const DeviceTables &t, int mode, int scratch) {
    return TABLES_AT + table_bytes(t, mode) + 256 +
           STORE_WAVES * ((uint32_t)scratch * 8 + aut_hash_places((uint32_t)scratch) * 4);
}

// Blocks of the kernel one compute unit holds at once (registers and the LDS the call asks for decide; the builds differ little:
// the one with the most registers is asked about); asked of the runtime once per LDS size.
int store_blocks_per_cu(const DeviceTables &t, int mode, int scratch) {
    static thread_local uint32_t known_lds[3] = {0, 0, 0};
    static thread_local int known[3] = {0, 0, 0};
    const uint32_t lds = store_lds_bytes(t, mode, scratch);
    const int m = mode < 0 ? 0 : (mode > 2 ? 2 : mode);
    if (known[m] && known_lds[m] == lds) return known[m];
    int least = 1 << 30;
    for (int p = 0; p < 3; p++) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(store_kernel(m, p)), STORE_BLOCK, lds) != hipSuccess || n < 1) { (void)hipGetLastError(); n = 1; }
        least = n < least ? n : least;
    }
    known[m] = least; known_lds[m] = lds;
    return least;
}

hipError_t launch_mask_store(const StoreArgs &a, const StoreInline &in, uint32_t lds_bytes, hipStream_t s) {
    hipLaunchKernelGGL(store_kernel((int)a.tab_mode, a.dtype), dim3(a.n_blocks), dim3(STORE_BLOCK), lds_bytes, s, a, in);
    return hipGetLastError();
}

hipError_t launch_store_clear(const StoreView &G, uint32_t ncls, const void *root_items, uint32_t n_root, hipStream_t s) {
    hipLaunchKernelGGL(store_clear_kernel, dim3(2048), dim3(256), 0, s, G, ncls, (const uint2 *)root_items, n_root);
    return hipGetLastError();
}

hipError_t launch_store_adopt(const StoreView &G, uint32_t n_states, uint32_t n_items, hipStream_t s) {
    hipLaunchKernelGGL(store_adopt_kernel, dim3((n_states + 255) / 256), dim3(256), 0, s, G, n_states, n_items);
    return hipGetLastError();
}

hipError_t launch_store_import(const StoreView &G, const RowChart *charts, const uint32_t *set_off, const Item *items, const uint32_t *group,
                               uint32_t n, uint32_t *import_root, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(store_import_kernel, dim3(n), dim3(256), 0, s, G, charts, set_off, items, group, import_root);
    return hipGetLastError();
}

}  // namespace zf
