// Mask kernel for states whose vocabulary has been walked before (walk_mode 2): mask_look_kernel.
//
// The persistent automaton (zf_mask_store.hip) keeps every transition it has ever computed, so once the mask at a state has been
// computed -- or the automaton was explored to its end when the engine was compiled -- every transition that the vocabulary walk
// from that state can meet is in the table.  Such a state needs look-ups only: no Earley byte step, no grammar tables, no bytes
// to be fed first.  That is every call of a decode loop but the first visits of a state, and it is what this kernel is made for;
// mask_store_kernel takes the other calls.  (Without pruning, calls whose rows the token-mask cache decides: there is no string to walk.)
//
// What bounds it.  Not bandwidth (a launch moves a few MB) but the length of one wavefront: dependent trips to memory
// (arguments, cache words and the state's table row, strings, about 1 us each) and the instructions between them, which one
// wavefront issues at 4 to 5 cycles apiece.  mask_store_kernel, which this one was split from, carries both halves: 200 scalar registers
// put by in lanes of vector ones for the byte step's sake, 2.4 us from the group's record to its last request, 54 instructions
// per byte of a walk.  Here the record is a quarter shorter, the cache rows are read by uniform addresses, the table row is on its
// way before anything else, undecided tokens are listed by scattering (a few instructions per bit) instead of being searched
// for, and a byte of the walk takes 22 instructions, the whole wavefront together.
//
// The logits (zf_compute_mask_apply_async).  Memory has little to do while the masks are worked out, and a launch of its own behind this one
// pays for the gap (1.2 us), its ramp and the whole of the reading.  Masked by the wavefront that has worked their mask out they lengthen
// the chain (16 x 128,256 bf16 260 us per 16 steps, 237 in a launch of their own).  So wavefronts of their own take them along: blocks behind those
// of the mask in the grid, which request their logits at once, wait for the mask words, and store.  Against two launches, us per pass: 32 steps of one row x
// 32,000 fp32 324 -> 252, 16 of 16 x 128,256 bf16 196 -> 170, 16 of 64 x 128,256 bf16 288 -> 228, 16 of 64 x 152,064 fp32 422 -> 364,
// 8 of 130 x 40,037 bf16 173 -> 143, 8 of 256 x 128,256 bf16 262 -> 233, 4 of 1,024 x 128,256 495 -> 379.
//   Words travel as (call's number << 32 | word), one 8-byte store past the L2s each: whoever reads the number has the word, nothing is ordered
// and nothing is counted.  Blocks start in the order of the grid, so as a rule the mask's are at work while those with logits wait.  But each XCD takes
// up its share of a grid by itself, and two grids of the kind (two engines') can each fill an XCD with waiting blocks while a block of their mask
// has no place on it.  So a wavefront with logits looks for its words a limited number of times; then it leaves its unit to its group of blocks
// (those that report in one status word) and ends, and the block of the group that is done last masks what was left, however long the words take.  That
// leaves two blocks per XCD and call that wait for as long as it takes, of 160 places, and no block of the mask waits for another: all grids go on.
// (Calls of up to 64 blocks, eight per XCD, leave nothing to anybody.)
//   Where the cache rows leave no token undecided they are the mask: those wavefronts put it together themselves (STORE_ROW_DECIDED), wait for nobody and read no logit of which nothing
// comes: 16 steps of 64 x 128,256 bf16 of the query language 175 -> 158 us, 8 of 256 x 128,256 of the schema 222 -> 217, 16 of 16 x 128,256 133 -> 127,
// 16 of 64 x 152,064 fp32 293 -> 290 (176, 230, 132 and 292 with every logit read).  Of bf16 logits they store the group's mask rows too, and no others work it out: 161 -> 150 for the first.
#include "zf_kernel_common.h"
#include "zf_aut_step.h"

namespace zf {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
static const int LOOK_LC_BITS = 10;                      // the block's LDS cache of table entries: 1,024 of (key, state)
static const uint32_t LOOK_LC = 1u << LOOK_LC_BITS;
// A group's wavefronts store its mask words to every member's row, one member or a few at a time: a batch that stands in one state, 256 rows x 128,256,
// kept 63 wavefronts at it for 18 us.  With logits, those of groups of more members than these (in the argument block) leave it to the wavefronts that mask the
// logits, each for its unit.  It takes large groups to tell: of fp32 logits, 1,000 rows x 32,000 in a few states 82 -> 50 us a step (query language), 62 -> 52 (schema), 63 -> 57
// (expression grammar), 256 rows 26 -> 21.  Units of fp32 hold half as many words as those of bf16, and groups of a few dozen lose by it (16 steps of 64 x 152,064 312.8 us
// without, 315.2 from 32 members on, 317.0 from 16), hence 128.  Of bf16 logits the line matters little, since groups that the cache rows decide store their own rows
// (STORE_ROW_DECIDED): before they did, 8 steps of 130 x 40,037 109.1 -> 106.1 us from 16 members on, 108.9 from 32.
template <int DT> constexpr uint32_t look_members_max() { return DT == 2 ? 16u : 128u; }
static const uint32_t LOOK_STOP = 256;                   // beyond every class and mark: the walk of a lane has ended
// Where the groups' records are: one in the argument block, up to 64 there, or any number in device memory.  A build each, so that the records are asked
// for along with the other arguments and not after them.
enum { LOOK_ONE, LOOK_FEW, LOOK_MANY };
static const uint32_t LOOK_LIST = 512;                   // undecided tokens a wavefront lists at a time
static const int LOOK_RAW = 2;                           // token-mask cache rows that are asked for whether or not there are so many
static const uint32_t LOOK_POLLS_MAX = 1u << 24;         // how often a wavefront that can leave a unit to nobody looks for mask words before the call fails: tens of seconds
static_assert(LOOK_LIST >= 64u * STORE_WAVES, "the states one byte away are listed there, read by lane x wavefronts");
static const int LOOK_WARM = 6;                          // table rows one byte ahead that each wavefront of a block reads into the cache

// The compiler takes whatever does not change from one segment to the next out of the loop over them: 150 scalar instructions and 30 spills, half a
// microsecond in front of every wavefront's first segment, most of it for segments that follow (few wavefronts have more than one).  A value that went through here stays where it is used.
__device__ __forceinline__ uint32_t stay(uint32_t x) { asm volatile("" : "+s"(x)); return x; }

// A row of the table lies in neighbouring places: the states that a walk meets have neighbouring numbers (they were explored breadth first, or met
// one after the other), so their rows seldom share a place.  With places by a hash of the key two or three of a walk's four to nine rounds
// asked memory for entries that another lane had just put out (16 x 128,256 bf16 157 -> 151 us per 16 steps, 130 x 40,037 136 -> 129; 2,048 places: 153 and 127, and
// 4,096 leave room for three blocks).
__device__ __forceinline__ uint32_t look_slot(uint32_t key) { return key & (LOOK_LC - 1u); }
// The k-th row number, from device memory or from the argument block.  (Of two generic pointers the compiler makes one flat load, which waits for
// LDS as well as for memory: the one into device memory says so.)
__device__ __forceinline__ uint32_t member_row(const LookArgs &a, const LookInline &in, uint32_t k) {
    if (a.members) return ((const __attribute__((address_space(1))) uint16_t *)a.members)[k];
    return in.member[k];
}

// As hand_over_store, in one level: the block that draws the last ticket of its group of blocks tells the host, which looks at a word per
// group; there is nothing to tell but failed walks.  In two parts: what a block has left to do between the draw and its answer, the trip to
// memory hides.  A ticket: 1 | failed walks << 16 | has left units to the group << 48.
struct LookTicket { unsigned long long sum; uint32_t group, size; };
__device__ __forceinline__ uint32_t ticket_group_size(const LookArgs &a, uint32_t group) { return gridDim.x / a.done_groups + (group < gridDim.x % a.done_groups ? 1u : 0u); }
__device__ __forceinline__ LookTicket draw_ticket(const LookArgs &a, uint32_t failed, bool left) {
    LookTicket t;
    t.group = blockIdx.x % a.done_groups;
    t.size = ticket_group_size(a, t.group);
    const unsigned long long mine = 1ull | (unsigned long long)(failed < 4095u ? failed : 4095u) << 16 | (unsigned long long)(left ? 1u : 0u) << 48;
    t.sum = mine;
    if (t.size > 1u) t.sum += atomicAdd(&a.tickets[t.group * STORE_TICKET_STRIDE], mine);   // a block that is a group by itself has nobody to wait for
    return t;
}
__device__ __forceinline__ void tell_host(const LookArgs &a, const LookTicket &t) {
    if ((t.sum & 0xFFFFull) != t.size) return;
    const uint32_t failed = (uint32_t)(t.sum >> 16);
    __hip_atomic_store(&a.status[STORE_ST_ROW + t.group], ((unsigned long long)a.seq << 32) | (failed < 0xFFFFFFu ? failed : 0xFFFFFFu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Blocks that have left units: behind the mask words, a word for every block with logits, which travels as they do: call's number << 32 | a bit per wavefront.
__device__ __forceinline__ unsigned long long *left_units(const LookArgs &a) { return a.tagged + (size_t)a.n_groups * a.W; }

// A wavefront with logits: `unit_kb` KB of one row's.  It requests them, waits until the row's mask words for them are there, and stores them masked.
// Where the words are there at once -- a block that started late, most blocks of a large tensor -- pieces of which nothing is allowed are not read.
template <int DT> struct LookLogit { typedef uint32_t elem; static const int PER_PIECE = 4; static const uint32_t NEG_INF = 0xFF800000u; typedef u32x4 __attribute__((aligned(4))) piece; };
template <> struct LookLogit<2> { typedef uint16_t elem; static const int PER_PIECE = 8; static const uint32_t NEG_INF = 0xFF80u; typedef u32x4 __attribute__((aligned(2))) piece; };
// words_read(failed, left) is called when the mask words are in hand, before anything is stored, or when they were not there after `polls` looks: with
// LEAVE the unit is then left to the group, else the call fails.
template <int DT, int HOW, bool LEAVE, class WordsRead>
__device__ __forceinline__ void mask_logits(const LookArgs &a, const LookInline &in, uint32_t unit, uint32_t lane, uint32_t polls, WordsRead words_read) {
    typedef LookLogit<DT> L;
    typedef typename L::elem elem;
    typedef typename L::piece piece_t;
    constexpr uint32_t EPV = L::PER_PIECE, KB_WORDS = 64 * EPV / 32, WORDS = (LOOK_UNIT_KB * KB_WORDS + 63) / 64;   // mask words of a KB; of a unit, per lane
    const uint32_t m = unit / a.row_units, part = unit - m * a.row_units, nu = a.unit_kb, W = a.W;
    uint32_t group = 0, r[LOOK_WORDS];                        // the record of the row's group, where it is asked for
    r[3] = 0;
    if (HOW == LOOK_MANY) {
        group = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a.group_of[m]);
        r[1] = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.groups[group].w[1]); r[2] = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.groups[group].w[2]);
#pragma unroll
        for (int k = 4; k < LOOK_WORDS; k++) r[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.groups[group].w[k]);
    } else if (HOW == LOOK_ONE) {
#pragma unroll
        for (int k = 0; k < LOOK_WORDS; k++) r[k] = in.g[0].w[k];
    } else {
        uint32_t x[LOOK_WORDS];
#pragma unroll
        for (int k = 1; k < LOOK_WORDS; k++) x[k] = in.g[lane].w[k];
        group = (uint32_t)__popcll(__ballot(((x[3] & 0xFFFFu) <= m) & (lane < a.n_groups))) - 1u;
#pragma unroll
        for (int k = 1; k < LOOK_WORDS; k++) r[k] = (uint32_t)__builtin_amdgcn_readlane((int)x[k], (int)group);
    }
    const bool decided = (r[1] & ((uint32_t)STORE_ROW_DECIDED << 8)) != 0;
    const bool stores_row = (decided && r[2] >> 16 == 0) || (r[3] >> 16) > look_members_max<DT>();   // (a decided group without segments: nobody else does)
    const uint32_t row = (uint32_t)__builtin_amdgcn_readfirstlane((int)member_row(a, in, m));
    const unsigned long long *const words = a.tagged + (size_t)group * W;
    const uint32_t w0 = part * nu * KB_WORDS;
    unsigned long long t[WORDS];
    bool here = true;
    if (decided) {                                           // the cache rows are the mask: nothing is waited for, and no logit read of which nothing comes
        const uint32_t n_ent = r[1] & 0xFFu;
#pragma unroll
        for (uint32_t k = 0; k < WORDS; k++) {
            const uint32_t j = k * 64u + lane, w = w0 + j < W ? w0 + j : W - 1u;
            uint32_t v = 0, y[STORE_GROUP_ENT];
#pragma unroll
            for (uint32_t e = 0; e < (uint32_t)STORE_GROUP_ENT; e++) {
                y[e] = 0;
                if (e < n_ent) y[e] = a.cache[(size_t)((r[4 + ((e + 1) >> 1)] >> (((e + 1) & 1) * 16)) & 0xFFFFu) * W + w].x;
            }
#pragma unroll
            for (uint32_t e = 0; e < (uint32_t)STORE_GROUP_ENT; e++) v |= y[e];
            t[k] = (unsigned long long)a.seq << 32 | (j < nu * KB_WORDS && w0 + j < W ? v : 0u);
        }
    } else {
#pragma unroll
        for (uint32_t k = 0; k < WORDS; k++) {
            const uint32_t j = k * 64u + lane;
            t[k] = (unsigned long long)a.seq << 32;
            if (j < nu * KB_WORDS && w0 + j < W) t[k] = __hip_atomic_load(&words[w0 + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            here &= (uint32_t)(t[k] >> 32) == a.seq;
        }
    }
    const bool ready = __all(here);
    auto bits = [&](uint32_t u) __attribute__((always_inline)) -> uint32_t {   // of the lane's piece of KB u
        const uint32_t w = (uint32_t)__shfl((int)(uint32_t)t[u * KB_WORDS / 64u], (int)((u * KB_WORDS) % 64u + lane / (32u / EPV)));
        return (w >> ((lane % (32u / EPV)) * EPV)) & ((1u << EPV) - 1u);
    };
    const uint32_t n_vec = a.V / EPV, p0 = part * nu * 64u + lane, tail = a.V - n_vec * EPV;
    const elem *const src = (const elem *)a.logits + (size_t)row * a.stride;
    elem *const dst = (elem *)a.out + (size_t)row * a.stride;
    u32x4 x[LOOK_UNIT_KB];
#pragma unroll
    for (uint32_t u = 0; u < (uint32_t)LOOK_UNIT_KB; u++) {
        x[u] = u32x4{0, 0, 0, 0};
        if (u >= nu) continue;
        const bool wanted = !ready || bits(u);               // (all lanes: a lane's word may be with one beyond the row's end)
        if (wanted && p0 + u * 64u < n_vec) x[u] = __builtin_nontemporal_load(reinterpret_cast<const piece_t *>(src) + p0 + u * 64u);
    }
    const bool has_tail = tail && part + 1u == a.row_units && lane < tail;   // V is not a multiple of the piece: the row's last elements, one per lane
    elem last = 0;
    if (has_tail) last = src[n_vec * EPV + lane];
    if (!ready) {
        for (;;) {
            // few wavefronts look again at once, many stay out of the way (16 x 128,256 bf16 145.0 us per 16 steps with 8 here, 142.8 with 1, 146.5 with 16;
            // one row x 32,000 201.6, 198.4, 207.4; 64 x 152,064 fp32 342.7, 343.7 with 3, 341.2 with 16; 256 x 128,256 225.2, 227.5 with 3, 224.1: differences
            // of 1 to 4 %, where runs of one side differ by as much at one row and by 0.1 to 1 % at the others; where the line lies between them is not borne out)
            if (a.units <= 2048u) __builtin_amdgcn_s_sleep(1); else __builtin_amdgcn_s_sleep(16);
            here = true;
#pragma unroll
            for (uint32_t k = 0; k < WORDS; k++) {
                if ((uint32_t)(t[k] >> 32) != a.seq) t[k] = __hip_atomic_load(&words[w0 + k * 64u + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                here &= (uint32_t)(t[k] >> 32) == a.seq;
            }
            if (__all(here)) break;
            if (polls <= 1u) { words_read(LEAVE ? 0u : 1u, LEAVE); return; }
            polls--;
        }
    }
    words_read(0u, false);
    if (stores_row) {                                        // the row's mask words as well
#pragma unroll
        for (uint32_t k = 0; k < WORDS; k++) if (k * 64u + lane < nu * KB_WORDS && w0 + k * 64u + lane < W) a.out_mask[(size_t)row * W + w0 + k * 64u + lane] = (uint32_t)t[k];
    }
#pragma unroll
    for (uint32_t u = 0; u < (uint32_t)LOOK_UNIT_KB; u++) {
        if (u >= nu) continue;
        const uint32_t b = bits(u);
        elem *e = reinterpret_cast<elem *>(&x[u]);
#pragma unroll
        for (uint32_t k = 0; k < EPV; k++) if (!((b >> k) & 1u)) e[k] = (elem)L::NEG_INF;
        if (p0 + u * 64u < n_vec) __builtin_nontemporal_store(x[u], reinterpret_cast<piece_t *>(dst) + p0 + u * 64u);
    }
    if (tail && part + 1u == a.row_units) {
        const uint32_t v = n_vec * EPV + lane, j = v / 32u - w0;   // the words of the row's end are its unit's
        uint32_t w = 0;
#pragma unroll
        for (uint32_t k = 0; k < WORDS; k++) { const uint32_t y = (uint32_t)__shfl((int)(uint32_t)t[k], (int)(j & 63u)); w = j / 64u == k ? y : w; }
        if (has_tail) dst[v] = (w >> (v & 31u)) & 1u ? last : (elem)L::NEG_INF;
    }
}

// What blocks of a group have left, by the wavefront that has drawn the group's last ticket: `n` blocks' units.  Returns how many never got their words.
template <int DT, int HOW>
__device__ __forceinline__ uint32_t mask_left_units(const LookArgs &a, const LookInline &in, uint32_t group, uint32_t n, uint32_t lane) {
    uint32_t failed = 0, polls = LOOK_POLLS_MAX;
    unsigned long long *const left = left_units(a);
    const uint32_t blocks = gridDim.x - a.mask_blocks, stride = a.done_groups;
    uint32_t first = group;                                  // the group's first block with logits ...
    while (first < a.mask_blocks) first += stride;
    while (n) {                                              // (a word may be on its way still)
        for (uint32_t k = first - a.mask_blocks; n && k < blocks; k += stride) {
            const unsigned long long e = __hip_atomic_load(&left[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(e >> 32)) != a.seq) continue;
            if (lane == 0) __hip_atomic_store(&left[k], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            n--;
            for (uint32_t bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)e); bits; bits &= bits - 1u)
                mask_logits<DT, HOW, false>(a, in, k * STORE_WAVES + (uint32_t)__ffs((int)bits) - 1u, lane, LOOK_POLLS_MAX, [&](uint32_t f, bool) __attribute__((always_inline)) { failed += f; });
        }
        if (n && polls-- <= 1u) return failed + n;           // never: the call fails
    }
    return failed;
}

// Grid and groups as in mask_store_kernel: the blocks of all groups one after the other, a group = the rows of the call that
// stand in the same state, whose mask is worked out once, in token order.  A wavefront takes every n_units-th segment of `sw` mask words.
template <int DT, int HOW>   // of the logits masked along: 0 = none, 1 = fp32, 2 = bf16
__global__ __launch_bounds__(STORE_BLOCK, DT ? LOOK_BLOCKS_PER_CU + 2 : LOOK_BLOCKS_PER_CU) void mask_look_kernel(LookArgs a, LookInline in) {
    __shared__ unsigned long long lc[LOOK_LC];
    __shared__ uint32_t lists[STORE_WAVES][LOOK_LIST];
    __shared__ uint32_t vbufs[STORE_WAVES][64];
    __shared__ uint32_t blk_failed;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    if (blockIdx.x == 0 && wave == 0) clear_tickets(a.tickets_next, lane);
    // ---- the record of the block's group: one trip to the argument block (lane l asks for that of group l), or to device memory ----
    uint32_t r[LOOK_WORDS], part, parts, group = 0;
    // the block's ticket has been drawn, by lane 0 of this wavefront
    auto drawn = [&](LookTicket t) __attribute__((always_inline)) {
        if (DT) {
            const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)((t.sum & 0xFFFFull) == t.size ? (uint32_t)(t.sum >> 48) : 0u));
            if (__builtin_expect(n, 0)) {                    // (rare: the arguments are read anew, none is kept for it from the kernel's start)
                const void *at = (const void *)__builtin_amdgcn_kernarg_segment_ptr();
                asm volatile("" : "+s"(at));
                static_assert(sizeof(LookArgs) % alignof(LookInline) == 0, "the second argument follows the first");
                const LookArgs &a2 = *(const LookArgs *)at;
                const LookInline &in2 = *(const LookInline *)((const uint8_t *)at + sizeof(LookArgs));
                t.sum += (unsigned long long)mask_left_units<DT, HOW>(a2, in2, blockIdx.x % a2.done_groups, n, lane) << 16;
            }
        }
        if (lane == 0) tell_host(a, t);
    };
    if (DT && blockIdx.x >= a.mask_blocks) {
        if (tid == 0) blk_failed = 0;                        // wavefronts that have their words or have left their unit; who has, << 8; those that gave up << 16
        __syncthreads();
        const uint32_t block = blockIdx.x - a.mask_blocks, unit = block * STORE_WAVES + wave;
        LookTicket t{};
        bool drew = false;
        // nothing that belongs to the engine is read behind this: the ticket's trip to memory goes along with the stores
        auto words_read = [&](uint32_t f, bool left) __attribute__((always_inline)) {
            const uint32_t mine = 1u + (left ? 256u << wave : 0u) + (f << 16);
            const uint32_t sum = mine + (uint32_t)__builtin_amdgcn_readfirstlane((int)(lane == 0 ? atomicAdd(&blk_failed, mine) : 0u)), who = (sum >> 8) & 255u;
            drew = (sum & 255u) == STORE_WAVES;
            if (drew && lane == 0) {
                if (who) __hip_atomic_store(&left_units(a)[block], (unsigned long long)a.seq << 32 | who, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                t = draw_ticket(a, sum >> 16, who != 0);
            }
        };
        if (unit < a.units) mask_logits<DT, HOW, true>(a, in, unit, lane, a.polls, words_read);
        else words_read(0u, false);
        if (drew) drawn(t);
        return;
    }
    if (HOW == LOOK_MANY) {
        const uint32_t b0 = a.block_of[2u * blockIdx.x], b1 = a.block_of[2u * blockIdx.x + 1u];
        group = (uint32_t)__builtin_amdgcn_readfirstlane((int)b0);
        part = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b1 & 0xFFFFu));
        parts = (uint32_t)__builtin_amdgcn_readfirstlane((int)(b1 >> 16));
#pragma unroll
        for (int k = 0; k < LOOK_WORDS; k++) r[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.groups[group].w[k]);
    } else if (HOW == LOOK_ONE) {                           // one group: scalar loads, along with the other arguments
        part = blockIdx.x; parts = a.mask_blocks;
#pragma unroll
        for (int k = 0; k < LOOK_WORDS; k++) r[k] = in.g[0].w[k];
    } else {
        uint32_t x[LOOK_WORDS];                              // (the block holds 64 records, of which n_groups mean something: the loads need not wait for that number)
#pragma unroll
        for (int k = 0; k < LOOK_WORDS; k++) x[k] = in.g[lane].w[k];
        const uint32_t first = x[2] & 0xFFFFu;
        group = (uint32_t)__popcll(__ballot((blockIdx.x >= first) & (lane < a.n_groups))) - 1u;   // groups that start at or before this block
#pragma unroll
        for (int k = 0; k < LOOK_WORDS; k++) r[k] = (uint32_t)__builtin_amdgcn_readlane((int)x[k], (int)group);
        const uint32_t fb0 = r[2] & 0xFFFFu, fb1 = group + 1u < a.n_groups ? (uint32_t)__builtin_amdgcn_readlane((int)first, (int)(group + 1u)) : a.mask_blocks;
        part = blockIdx.x - fb0; parts = fb1 - fb0;
    }
#pragma unroll
    for (uint32_t k = 0; k < LOOK_LC / STORE_BLOCK; k++) lc[k * STORE_BLOCK + tid] = 0xFFFFFFFF00000000ull;
    if (tid == 0) blk_failed = 0;
    __syncthreads();
    const uint32_t start = r[0], n_ent = r[1] & 0xFFu, sw = ((r[1] >> 16) & 0xFFu) + 1u, n_seg = r[2] >> 16, member_at = r[3] & 0xFFFFu, n_members = r[3] >> 16;
    const uint32_t n_here = n_ent > (uint32_t)STORE_GROUP_ENT ? LOOK_ENT_OF_MORE : n_ent;   // cache rows in the record; the others are listed behind the members
    const uint32_t n_store = DT && HOW != LOOK_MANY && n_members > look_members_max<DT>() ? 0u : n_members;   // members whose mask rows the wavefronts without logits store
    const bool pooled = (r[1] & ((uint32_t)STORE_ROW_POOLED << 8)) != 0, keep = (r[1] & ((uint32_t)STORE_ROW_KEEP << 8)) != 0, use_cache = (r[1] & ((uint32_t)STORE_ROW_CACHE << 8)) != 0;
    const uint32_t unit = part * STORE_WAVES + wave, n_units = parts * STORE_WAVES, W = a.W, V = a.V, ncls = a.ncls;
    if (unit < n_seg) {
    uint32_t *const list = lists[wave], *const vbuf = vbufs[wave];
    const bool walks = !pooled && start < AT_FAIL;            // AT_SINK: the sentence is finished, no token can follow
    // ---- requests: the segment's cache words, the state's table row, members.  No lane is left out and nothing is asked for under a condition that
    // differs (lanes and rows too many ask again for what a neighbour asks for): the compiler then knows how many loads are on their way behind
    // each, and waits for the one it needs; where it does not know, it waits for all of them ----
    struct Words { uint2 x[LOOK_RAW], y[STORE_GROUP_ENT - LOOK_RAW]; };
    auto request = [&](uint32_t g, Words &q) __attribute__((always_inline)) {
        const uint32_t w = g * sw + lane < W ? g * sw + lane : W - 1u;
        const uint32_t rows[5] = {stay(r[4]), stay(r[5]), stay(r[6]), stay(r[7]), stay(r[8])};
        auto ent = [&](int j) -> uint32_t { return (rows[(j + 1) >> 1] >> (((j + 1) & 1) * 16)) & 0xFFFFu; };
        if (pooled) {
            q.x[0] = make_uint2(a.pool[(size_t)start * W + w], 0);
#pragma unroll
            for (int j = 1; j < LOOK_RAW; j++) q.x[j] = make_uint2(0, 0);
            return;
        }
        if (n_here > (uint32_t)LOOK_RAW) {
#pragma unroll
            for (int j = LOOK_RAW; j < STORE_GROUP_ENT; j++) q.y[j - LOOK_RAW] = a.cache[(size_t)((uint32_t)j < n_here ? ent(j) : ent(0)) * W + w];
        }
#pragma unroll
        for (int j = 0; j < LOOK_RAW; j++) q.x[j] = a.cache[(size_t)((uint32_t)j < n_here ? ent(j) : ent(0)) * W + w];   // (without a row: row 0, not looked at)
    };
    Words x;
#pragma unroll
    for (int j = 0; j < STORE_GROUP_ENT - LOOK_RAW; j++) x.y[j] = make_uint2(0, 0);
    request(unit, x);
    const uint32_t known = walks ? start : 0u, column = lane < ncls ? lane : 0u;
    // (the table takes 128 MB at most: an offset of 32 bits)
    auto table = [&](uint32_t st) __attribute__((always_inline)) -> uint32_t { return *(const uint32_t *)((const uint8_t *)a.trans + (size_t)((st * ncls + column) * 4u)); };
    uint32_t t_root = table(known);
    auto members_from = [&](uint32_t m0) __attribute__((always_inline)) -> uint32_t {   // lane l: the l-th of the 64 rows in hand
        const uint32_t k = member_at + m0 + lane;
        return m0 + lane < n_members ? member_row(a, in, k) : 0u;
    };
    const uint32_t member_k = member_at + (lane < n_members ? lane : 0u);
    uint32_t members = member_row(a, in, member_k);
    if (!walks || lane >= ncls) t_root = AT_NONE;
    // ---- the block's LDS cache: the state's row, and the rows of the states one byte away, shared out among the wavefronts ----
    auto into_cache = [&](uint32_t st, uint32_t t) __attribute__((always_inline)) {
        if (lane < ncls) { const uint32_t key = st * ncls + lane; __hip_atomic_store(&lc[look_slot(key)], ((unsigned long long)key << 32) | t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
    };
    uint32_t ahead[LOOK_WARM], t_ahead[LOOK_WARM], n_ahead = 0;
    into_cache(start, t_root);
    {
        // a lane per state one byte away: of lanes with the same state one is left (by whose number stays in a common place; different states may
        // share a place, one of them is not read ahead then), the wavefront takes every STORE_WAVES-th of them
        const bool live = t_root < AT_FAIL && t_root != start;
        uint32_t *const place = &list[t_root % LOOK_LIST];
        if (live) lds_store(place, lane);
        const bool mine = live && lds_load(place) == lane;
        const unsigned long long owners = __ballot(mine);
        const uint32_t rank = (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(owners >> 32), (uint32_t)__builtin_amdgcn_mbcnt_lo((uint32_t)owners, 0)), n = (uint32_t)__popcll(owners);
        if (mine) lds_store(&list[rank], t_root);
        n_ahead = n > wave ? (n - wave + STORE_WAVES - 1u) / STORE_WAVES : 0u;
        const uint32_t at_rank = lds_load(&list[lane * STORE_WAVES + wave]);   // lane k: the wavefront's k-th
#pragma unroll
        for (int k = 0; k < LOOK_WARM; k++) {
            const uint32_t nx = (uint32_t)__builtin_amdgcn_readlane((int)at_rank, k);
            ahead[k] = (uint32_t)k < n_ahead ? nx : known;
            t_ahead[k] = table(ahead[k]);
        }
    }
    uint32_t failed = 0;
    bool first = true;
    for (uint32_t g = unit; g < n_seg; g += n_units) {
        const uint32_t w = lane < sw ? g * sw + lane : 0xFFFFFFFFu;   // the lane's mask word
        uint32_t v = 0, c = 0;
#pragma unroll
        for (int j = 0; j < LOOK_RAW; j++) { v |= x.x[j].x; c |= x.x[j].y; }
#pragma unroll
        for (int j = 0; j < STORE_GROUP_ENT - LOOK_RAW; j++) { v |= x.y[j].x; c |= x.y[j].y; }
        const uint32_t n_rows = stay(n_ent);
        if (__builtin_expect(n_rows > (uint32_t)STORE_GROUP_ENT, 0)) {   // a state of many items: the rest of its cache rows, four at a time
            const uint32_t more_at = stay(r[8]) >> 16, n_more = n_rows - LOOK_ENT_OF_MORE, wc = g * sw + lane < W ? g * sw + lane : W - 1u;
#pragma unroll 1
            for (uint32_t k0 = 0; k0 < n_more; k0 += 64) {
                const uint32_t n = n_more - k0 < 64u ? n_more - k0 : 64u, ent = member_row(a, in, more_at + k0 + (lane < n ? lane : 0u));
#pragma unroll 1
                for (uint32_t j = 0; j < n; j += 4) {
                    uint2 y[4];
#pragma unroll
                    for (uint32_t i = 0; i < 4; i++) y[i] = a.cache[(size_t)(uint32_t)__builtin_amdgcn_readlane((int)ent, (int)(j + i < n ? j + i : j)) * W + wc];
#pragma unroll
                    for (uint32_t i = 0; i < 4; i++) { v |= y[i].x; c |= y[i].y; }
                }
            }
        }
        if (!n_ent) { v = pooled ? v : 0u; c = pooled || use_cache ? 0u : 0xFFFFFFFFu; }
        if (g + n_units < n_seg) request(g + n_units, x);    // the next segment's words travel while this one's tokens are checked
        uint32_t want = c & ~v;
        {
            const uint32_t t0 = w * 32u;
            if (w >= W || t0 >= V || !walks) want = 0;
            else if (V - t0 < 32u) want &= (1u << (V - t0)) - 1u;
        }
        if (!walks && !pooled) v = 0;
        // ---- the undecided tokens, listed: running sums of the words' bit counts (data-parallel-primitive moves), then every lane
        // writes the numbers of its word's tokens where they belong ----
        const uint32_t cnt = (uint32_t)__popc(want);
        uint32_t incl = cnt;
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x111, 0xF, 0xF, true);    // row_shr:1
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x112, 0xF, 0xF, true);    // row_shr:2
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x114, 0xF, 0xF, true);    // row_shr:4
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x118, 0xF, 0xF, true);    // row_shr:8
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
        incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (lane < sw) lds_store(&vbuf[lane], 0u);
        for (uint32_t base = 0; base < total; base += LOOK_LIST) {
            {
                uint32_t at = incl - cnt - base, bits = want;   // (wraps below the window: not listed)
                while (bits) {
                    const uint32_t b = (uint32_t)__ffs((int)bits) - 1u;
                    bits &= bits - 1u;
                    if (at < LOOK_LIST) lds_store(&list[at], lane * 32u + b);
                    at++;
                }
            }
            const uint32_t n = total - base < LOOK_LIST ? total - base : LOOK_LIST;
            struct Tok { uint32_t at; u32x4 s; };
            auto fetch = [&](uint32_t b0) __attribute__((always_inline)) -> Tok {   // requested here, looked at a batch later
                Tok k;
                k.at = lds_load(&list[b0 + lane < n ? b0 + lane : 0u]);
                k.s = *reinterpret_cast<const u32x4 *>(&a.tok16[g * sw * 32u + k.at]);
                return k;
            };
            Tok nxt = fetch(0);
            if (first) {                                     // the rows one byte ahead have arrived meanwhile
#pragma unroll
                for (int k = 0; k < LOOK_WARM; k++) if ((uint32_t)k < n_ahead) into_cache(stay(ahead[k]), t_ahead[k]);
                first = false;
            }
            for (uint32_t b0 = 0; b0 < n; b0 += 64) {
                const Tok cur = nxt;
                nxt = fetch(b0 + 64);                        // (behind the last batch: the list's first token again)
                // One lane per token: it follows its string through the table for as long as there is a state and a next byte.  The
                // classes at hand are a shift register; a mark ends them.  All lanes take every round; those that are done keep what they
                // hold: 22 instructions a round, where lanes that leave the loop one by one cost twice as many, in execution masks (16 x 128,256 bf16
                // 150 -> 143 us per 16 steps, 130 x 40,037 129 -> 122 per 8, one row x 32,000 fp32 212 -> 204 per 32).  Strings that go on are seen to between the rounds.
                uint32_t w0 = cur.s[0], w1 = cur.s[1], w2 = cur.s[2], w3 = cur.s[3], passed = 0;
                uint32_t c = b0 + lane < n ? w0 & 0xFFu : TOK_END;         // the next class, or what ended the walk: a mark, or LOOK_STOP + the class or mark behind the last step
                uint32_t t = c == TOK_END ? AT_DEAD : start;               // the state or the entry that ended the walk; an empty token is never allowed
                for (;;) {
                    do {
                        const bool on = c < TOK_MORE;
                        const uint32_t key = __umul24(t, ncls) + c;        // a state has at most 18 bits, a class 8
                        const uint32_t slot = look_slot(key);
                        const unsigned long long e = __hip_atomic_load(&lc[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        uint32_t to = (uint32_t)e;
                        if (on & ((uint32_t)(e >> 32) != key)) {
                            to = __hip_atomic_load((const uint32_t *)((const uint8_t *)a.trans + (size_t)(key * 4u)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                            __hip_atomic_store(&lc[slot], ((unsigned long long)key << 32) | to, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                        w0 = __builtin_amdgcn_alignbyte(w1, w0, 1); w1 = __builtin_amdgcn_alignbyte(w2, w1, 1); w2 = __builtin_amdgcn_alignbyte(w3, w2, 1); w3 >>= 8;
                        const uint32_t next = (w0 & 0xFFu) | (to < AT_FAIL ? 0u : LOOK_STOP);
                        t = on ? to : t;
                        c = on ? next : c;
                    } while (__ballot(c < TOK_MORE));
                    if (!__ballot(c == TOK_MORE)) break;
                    if (c == TOK_MORE) {                     // a string beyond the bytes at hand: its next fifteen classes
                        const DeviceTables &D = a.konst->tab;
                        const uint32_t rank = D.rank_of[g * sw * 32u + cur.at], from = D.str_off[rank], len = D.str_off[rank + 1] - from;
                        passed += TOK_AT_HAND;
                        const uint32_t left = len - passed, m = left < TOK_AT_HAND ? left : TOK_AT_HAND;   // left >= 1: the mark says that the string goes on
                        uint32_t nw[4] = {0, 0, 0, 0};
                        for (uint32_t k = 0; k <= m; k++) {
                            const uint32_t b = (k < m ? (uint32_t)D.str_cls[from + passed + k] : (left > TOK_AT_HAND ? TOK_MORE : TOK_END)) << ((k & 3u) * 8u);
                            nw[0] |= k < 4u ? b : 0u; nw[1] |= (k >> 2) == 1u ? b : 0u; nw[2] |= (k >> 2) == 2u ? b : 0u; nw[3] |= (k >> 2) == 3u ? b : 0u;
                        }
                        w0 = nw[0]; w1 = nw[1]; w2 = nw[2]; w3 = nw[3];
                        c = w0 & 0xFFu;
                    }
                }
                if ((c & 0xFFu) == TOK_END && (t < AT_FAIL || t == AT_SINK)) atomicOr(&vbuf[cur.at >> 5], 1u << (cur.at & 31u));
                // an entry that is not there, or stands for no room: the host was wrong about the state, the call fails
                failed += (uint32_t)__popcll(__ballot(t == AT_NONE || t == AT_BUSY || t == AT_FAIL));
            }
        }
        if (total) v |= lane < sw ? lds_load(&vbuf[lane]) : 0u;   // LDS serves one wavefront's accesses in issue order
        if (DT && w < W) __hip_atomic_store(&a.tagged[(size_t)group * W + w], (unsigned long long)a.seq << 32 | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // ---- the segment's words go to every member's mask row (and to the state cache) ----
        for (uint32_t m0 = 0; m0 < n_store; m0 += 64) {
            if (n_store > 64u) members = members_from(m0);
            const uint32_t n = n_store - m0 < 64u ? n_store - m0 : 64u;
            if (n < 4u || sw > 32u) {
                for (uint32_t k = 0; k < n; k++) {
                    uint32_t *dst = a.out_mask + (size_t)(uint32_t)__builtin_amdgcn_readlane((int)members, (int)k) * W + w;
                    if (w < W) put_word(dst, v, a.complete);
                }
            } else {                                         // several members per store: the lanes hold the segment 2, 4, 8 or 16 times over
                const uint32_t s = stay(sw), lg = s <= 4u ? 2u : s <= 8u ? 3u : s <= 16u ? 4u : 5u, word = lane & ((1u << lg) - 1u), w2 = g * sw + word;
                const uint32_t v2 = (uint32_t)__shfl((int)v, (int)word);
                for (uint32_t k0 = 0; k0 < n; k0 += 64u >> lg) {
                    const uint32_t k = k0 + (lane >> lg);
                    uint32_t *dst = a.out_mask + (size_t)(uint32_t)__shfl((int)members, (int)(k & 63u)) * W + w2;
                    if (k < n && word < sw && w2 < W) put_word(dst, v2, a.complete);
                }
            }
        }
        if (keep && w < W) put_word(&a.pool[(size_t)(r[4] & 0xFFFFu) * W + w], v, a.complete);
        if (n_store > 64u) members = members_from(0);
    }
    if (lane == 0 && failed) atomicAdd(&blk_failed, failed);
    }
    if (a.complete) stores_arrived();                        // every word this wavefront wrote has reached memory before the block's ticket is drawn
    __syncthreads();
    if (wave == 0) {
        LookTicket t{};
        if (lane == 0) t = draw_ticket(a, lds_load(&blk_failed), false);
        drawn(t);
    }
}

}  // namespace

// Blocks of the kernel one compute unit holds at once.
int look_blocks_per_cu() {
    static const int blocks = [] {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(mask_look_kernel<0, LOOK_FEW>), STORE_BLOCK, 0) != hipSuccess || n < 1) { (void)hipGetLastError(); n = 1; }
        return n < LOOK_BLOCKS_PER_CU ? n : LOOK_BLOCKS_PER_CU;
    }();
    return blocks;
}

hipError_t launch_mask_look(const LookArgs &a, const LookInline &in, hipStream_t s) {
    const dim3 grid(look_grid(a)), block(STORE_BLOCK);
    const int dt = a.units ? (int)a.dtype : 0, how = a.groups ? LOOK_MANY : a.n_groups == 1u ? LOOK_ONE : LOOK_FEW;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, a, in); };
#define LOOK_HOW(DT) (how == LOOK_MANY ? launch(mask_look_kernel<DT, LOOK_MANY>) : how == LOOK_ONE ? launch(mask_look_kernel<DT, LOOK_ONE>) : launch(mask_look_kernel<DT, LOOK_FEW>))
    if (dt == 0) LOOK_HOW(0);
    else if (dt == 1) LOOK_HOW(1);
    else LOOK_HOW(2);
#undef LOOK_HOW
    return hipGetLastError();
}

}  // namespace zf
