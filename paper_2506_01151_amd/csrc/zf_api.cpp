// The C boundary: argument checks, engine / state life cycle, advance, chart packing and
// upload, kernel launches.
#include <hip/hip_runtime_api.h>
#include <unistd.h>
#include <algorithm>
#include <chrono>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <system_error>
#include <thread>
#include <unordered_map>
#include "zf_internal.h"
#include "zf_host_automaton.h"
#include "zf_launch.h"

using namespace zf;

namespace zf {
static thread_local std::string g_err;
void set_error(const std::string &m) { g_err = m; }
// Bring the state's chart up to date: the bytes fed through the host automaton since it last was, one zf_advance call at
// a time (Scan -> Complete -> Compact -> Predict, as feed_token_bytes does without the automaton).
static void catch_up(zf_state *s) {
    if (s->lag.empty()) return;
    const Tables &t = s->eng->tab;
    Chart &c = s->chart;
    int64_t created = 0;
    size_t at = 0;
    for (uint32_t cut : s->lag_cut) {
        for (; at < cut; at++) (void)earley_step(t, c, s->lag[at], false, &created);
        chart_compact(t, c);
    }
    s->items_created += created;
    s->lag.clear(); s->lag_cut.clear();
}
const Chart &chart_of(const zf_state *s) {
    catch_up(const_cast<zf_state *>(s));
    return s->chart;
}

}  // namespace zf

// Device-side resources of an engine.
struct DeviceSide {
    int device = 0;
    DeviceTables tab{};
    // What an engine keeps in device memory for its whole life is carved out of a few large allocations: a schema that a request
    // brings along is compiled and thrown away again, and hipFree costs about 0.1 ms apiece (so does hipHostFree).  The first is made for
    // all that the engine is going to ask for.
    static const size_t SLAB_BYTES = (size_t)16 << 20;
    std::vector<void *> slabs;
    uint8_t *slab_next = nullptr; size_t slab_left = 0;
    // per-call buffers, grown on demand
    void *d_chart = nullptr; size_t chart_cap = 0;
    static const int N_SLOTS = 4;                    // calls that may be in flight before zf_mask_wait
    void *h_block = nullptr;                         // pinned: the status words, and the room that every slot has from the start
    void *h_stage[N_SLOTS] = {nullptr, nullptr, nullptr, nullptr}; size_t stage_cap[N_SLOTS] = {0, 0, 0, 0};   // pinned: a piece of h_block, or ...
    bool stage_own[N_SLOTS] = {false, false, false, false};   // ... grown, an allocation of its own
    uint32_t *h_status = nullptr;                    // pinned, [N_SLOTS][8]: counters [0..3] and the call's number [4], written by each call's last kernel
    uint32_t call_seq = 0, last_seq = 0, last_slot = 0; // number of the newest call in flight and its slot
    uint32_t next_slot = 0, pending = 0;
    uint32_t occ_lds = 0;                            // LDS size the cached occupancy answer belongs to
    int occ_blocks = 1;
    // State cache (paper Section 5.2): finished token-order mask rows keyed by the row's packed chart.
    struct CacheEntry { uint64_t hash = 0; std::vector<uint32_t> key; uint32_t stamp = 0; bool used = false; };
    std::vector<CacheEntry> cache;                   // one per pool slot
    std::unordered_multimap<uint64_t, uint32_t> cache_index;
    uint32_t *d_pool = nullptr;                      // [cache.size()][W]
    uint32_t cache_victim = 0, cache_call = 0;
    uint32_t *d_rank_mask = nullptr; size_t rank_cap = 0;
    uint4 *d_overflow = nullptr; size_t overflow_cap = 0;
    uint4 *d_work = nullptr;
    int cus = 256;
    int mode = 2;
    bool lanes_call[N_SLOTS] = {false, false, false, false};   // the call ran the per-block automaton's AUT_STEP_LANES build
    // The status of a call through the closing kernel is final when that kernel starts, and zf_mask_wait returns with the kernel at work on the engine's
    // buffers (d_rank_mask, d_chart): a call on another stream goes behind this event.
    hipEvent_t closing_done = nullptr;
    hipStream_t closing_stream = nullptr;            // the newest stream that is behind it
    bool closing_open = false;                       // it stands behind the last call through the closing kernel (which was not a waiting one)
    bool lanes_outgrown = false;                     // such a call left strings to the fallback pass: AUT_STEP_WIDE from then on
    uint32_t *d_counters = nullptr;
    uint2 *d_fb_items = nullptr;
    uint32_t *d_fb_ss = nullptr;
    uint8_t *scratch = nullptr;          // this device's copy of the static array behind zf_compute_mask_noalloc
    // The persistent automaton (walk_mode 2).
    StoreView store{};
    void *d_root_items = nullptr; uint32_t n_root = 0;
    uint32_t *d_import_root = nullptr;               // [MAX_BATCH]
    volatile uint64_t *h_store_status = nullptr;     // pinned, [N_SLOTS][STORE_STATUS_WORDS]: see STORE_ST_DONE
    unsigned long long *d_tickets = nullptr;         // [2][STORE_TICKETS]
    uint32_t ticket_set = 0;                         // the one the next kernel draws from
    unsigned long long *d_tagged = nullptr; size_t tagged_cap = 0;   // LookArgs::tagged (words)
    uint32_t look_polls = LOOK_POLLS;
    StoreConst *d_konst = nullptr;
    const uint32_t *no_trans = nullptr;     // engine without a persistent automaton: the row of the table that mask_look_kernel reads of a state without transitions
    uint32_t store_epoch = 1;                        // bumped whenever the store is cleared
    uint32_t store_states = 0, store_items = 0;      // as of the last call that reported back
    bool store_dirty = true;                         // the store must be cleared before its next use
    // What sizes a call's grid: the tokens a state's token-mask cache rows leave to the parser.  The host keeps the token-order
    // rows and counts the union for every set of cache rows it meets, once (the sets repeat all the time).
    std::vector<uint2> h_ci_tok;                     // [Q + N][W]
    std::vector<uint32_t> ci_undecided;              // [Q + N] what a row leaves undecided by itself
    VocabRows voc{};                                 // the DFAs as the kernels that make cache rows read them, and where the token-order rows go
    std::unordered_map<uint64_t, uint32_t> undecided_of;   // signature of a list of several cache rows -> undecided tokens
    uint32_t store_backoff = 0, store_backoff_next = 8;   // after a call the store had no room for: calls that take the per-block automaton instead
    // A call through the persistent automaton until zf_mask_wait has seen its status: the groups whose state the kernel reports,
    // and their rows.  (Groups the host knows the state of need no note.)
    struct CallRecord {
        bool active = false;
        uint32_t seq = 0, epoch = 0;
        struct Group { uint32_t group, host_id, first, n; uint64_t hop; };   // host_id: the state's name in the host automaton (0 = none); hop: the (state, token) pair the kernel walks (0 = none)
        struct Row { std::shared_ptr<StateLink> st; uint32_t gen; uint64_t upto; };
        std::vector<Group> groups;
        std::vector<Row> rows;
        uint32_t host_epoch = 0;                     // epoch of the host automaton the names belong to
        int64_t undecided = 0;                       // for the report
        bool sure = false;                           // look-ups only, over transitions that have been reported to be there: nothing in the call is expected to fail
        uint32_t done_groups = 0;                    // words the call reports in (mask_look_kernel); 0: in STORE_ST_DONE
        uint32_t debug_failed = 0;                   // added to what the call reports
        bool lazy = false;                           // such a call that zf_mask_wait has let go of: its kernels may still be at work with the slot
    } rec[N_SLOTS];
    uint32_t n_lazy = 0;                             // how many slots are
    hipStream_t lazy_stream = nullptr;               // the stream these calls are on
    uint32_t late_failed = 0;                        // walks that failed in them all the same: an error that the next call that waits reports (report_late)
    uint32_t debug_failed = 0;                       // zf_debug_fail_look_ups
    // State cache (Section 5.2) on this path: the pool's slot of a state by its name in the host automaton.  A name says all there
    // is to say about a set, so nothing is packed or compared.
    std::vector<uint32_t> slot_of_host;              // slot + 1; 0 = none
    std::vector<uint32_t> host_of_slot, slot_stamp;
    uint32_t pool_victim = 0, pool_epoch = 0, pool_call = 0;
    // The device's name of a state of the host automaton, as the mask kernel has reported it for a row that stood there.  The two
    // automata hold the same sets under different names; once a state's device name is known, a row that arrives in it is sent
    // with that name and no bytes to walk, whatever token took it there.  Valid while neither automaton has been emptied.
    std::vector<uint32_t> name_of_host;
    uint32_t name_host_epoch = 0, name_store_epoch = 0;
    uint32_t closed_states = 0, closed_epoch = 0;    // in that epoch of the store every transition out of the states below closed_states is in it
    uint32_t name_find(uint32_t host_id, uint32_t host_epoch, uint32_t st_epoch) const {   // 0 = unknown
        return host_epoch == name_host_epoch && st_epoch == name_store_epoch && host_id < name_of_host.size() ? name_of_host[host_id] : 0u;
    }
    void name_note(uint32_t host_id, uint32_t host_epoch, uint32_t st_epoch, uint32_t dev) {
        if (host_epoch != name_host_epoch || st_epoch != name_store_epoch) { name_of_host.clear(); name_host_epoch = host_epoch; name_store_epoch = st_epoch; }
        if (host_id >= (1u << 22)) return;
        if (host_id >= name_of_host.size()) name_of_host.resize(std::max<size_t>(host_id + 1, name_of_host.size() * 2), 0u);
        name_of_host[host_id] = dev;
    }
    // Where a token leads from a state of the persistent automaton, as the mask kernel has reported it: (state << 32 | token + 1)
    // -> state.  Names are stable while the store is not cleared, so a row that is fed a token in a state some row was fed it in
    // before is sent with the state it arrives in and no bytes to walk.  Open addressing, exact keys, emptied with the store.
    std::vector<uint64_t> hop_key; std::vector<uint32_t> hop_val;
    uint32_t hop_used = 0, hop_epoch = 0;
    static const uint32_t HOP_SLOTS = 1u << 16;
    uint32_t hop_find(uint64_t key) const {          // 0 = unknown
        if (hop_key.empty()) return 0;
        for (uint32_t i = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 48);; i = (i + 1) & (HOP_SLOTS - 1)) {
            if (hop_key[i] == key) return hop_val[i];
            if (hop_key[i] == 0) return 0;
        }
    }
    void hop_note(uint64_t key, uint32_t val) {
        if (hop_key.empty()) { hop_key.assign(HOP_SLOTS, 0); hop_val.assign(HOP_SLOTS, 0); }
        if (hop_used >= HOP_SLOTS / 2) { std::fill(hop_key.begin(), hop_key.end(), 0); hop_used = 0; }
        for (uint32_t i = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> 48);; i = (i + 1) & (HOP_SLOTS - 1)) {
            if (hop_key[i] == key) return;
            if (hop_key[i] == 0) { hop_key[i] = key; hop_val[i] = val; hop_used++; return; }
        }
    }
    zf_mask_report report{};
    uint32_t call_parity = 0;            // which of the two counter sets the next call uses
    bool profiling = false;
    bool closing_kernel = true;          // the last call enqueued a kernel behind its mask kernel (closing kernel or gather)
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
};

namespace {

const int MAX_BATCH = 4096;   // rows per zf_compute_mask call
const size_t STORE_STATUS_WORDS = STORE_ST_ROW + MAX_BATCH;
const uint32_t STORE_ROOT_ID = 1;

int fail(int code, const std::string &m) { set_error(m); return code; }
#define HIP_TRY(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) return fail(ZF_ERR_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); } while (0)

// Device memory that lives as long as the engine.
template <class Tv>
int engine_alloc(DeviceSide *d, size_t bytes, Tv **out) {
    bytes = (std::max<size_t>(bytes, 16) + 255) & ~(size_t)255;
    if (bytes > d->slab_left) {
        uint8_t *p = nullptr;
        const bool own = bytes >= DeviceSide::SLAB_BYTES;   // an allocation of its own: the slab in use stays in use
        HIP_TRY(hipMalloc((void **)&p, own ? bytes : DeviceSide::SLAB_BYTES));
        d->slabs.push_back(p);
        if (own) { *out = (Tv *)p; return ZF_OK; }
        d->slab_next = p; d->slab_left = DeviceSide::SLAB_BYTES;
    }
    *out = (Tv *)d->slab_next;
    d->slab_next += bytes; d->slab_left -= bytes;
    return ZF_OK;
}

int engine_reserve(DeviceSide *d, size_t bytes) {
    HIP_TRY(hipMalloc((void **)&d->slab_next, bytes));
    d->slabs.push_back(d->slab_next);
    d->slab_left = bytes;
    return ZF_OK;
}
// Pinned staging room of a slot, grown (the slot is free: its last call has been waited for).
int grow_stage(DeviceSide *d, uint32_t slot, size_t cap) {
    if (d->stage_own[slot]) (void)hipHostFree(d->h_stage[slot]);
    d->h_stage[slot] = nullptr; d->stage_cap[slot] = 0; d->stage_own[slot] = false;
    HIP_TRY(hipHostMalloc(&d->h_stage[slot], cap, hipHostMallocDefault));
    d->stage_cap[slot] = cap; d->stage_own[slot] = true;
    return ZF_OK;
}

template <class Tv>
int upload(DeviceSide *d, const std::vector<Tv> &v, const Tv **out, uint32_t *bytes_out = nullptr) {
    // padded to a multiple of 16 bytes (zero filled) so that blocks can stage it with 16-byte copies
    uint8_t *p = nullptr;
    const size_t have = v.size() * sizeof(Tv), bytes = (std::max<size_t>(have, 16) + 15) & ~(size_t)15;
    const int rc = engine_alloc(d, bytes, &p);
    if (rc != ZF_OK) return rc;
    if (have < bytes) HIP_TRY(hipMemset(p + have, 0, bytes - have));
    if (have) HIP_TRY(hipMemcpy(p, v.data(), have, hipMemcpyHostToDevice));
    *out = (const Tv *)p;
    if (bytes_out) *bytes_out = (uint32_t)bytes;
    return ZF_OK;
}

void free_device(DeviceSide *d) {
    if (!d) return;
    (void)hipSetDevice(d->device);
    if (d->d_tagged) (void)hipFree(d->d_tagged);
    for (void *p : d->slabs) (void)hipFree(p);
    if (d->d_chart) (void)hipFree(d->d_chart);
    for (int k = 0; k < DeviceSide::N_SLOTS; k++) if (d->stage_own[k]) (void)hipHostFree(d->h_stage[k]);
    if (d->h_block) (void)hipHostFree(d->h_block);
    if (d->d_rank_mask) (void)hipFree(d->d_rank_mask);
    if (d->d_overflow) (void)hipFree(d->d_overflow);
    if (d->d_work) (void)hipFree(d->d_work);
    if (d->d_fb_items) (void)hipFree(d->d_fb_items);
    if (d->d_fb_ss) (void)hipFree(d->d_fb_ss);
    for (auto &ev : d->ev) if (ev) (void)hipEventDestroy(ev);
    if (d->closing_done) (void)hipEventDestroy(d->closing_done);
    delete d;
}

const uint32_t STORE_CAP_ITEMS = 1u << 22;
uint32_t store_cap_states(int n_cls) {
    uint32_t cap = 1u << 18;
    while (cap > 4096 && (size_t)cap * (size_t)std::max(n_cls, 1) * 4 > ((size_t)128 << 20)) cap >>= 1;
    return cap;
}

// The arenas of the fallback pass (256 MB).
int alloc_fallback(DeviceSide *d) {
    if (!d->d_fb_items) HIP_TRY(hipMalloc((void **)&d->d_fb_items, (size_t)FB_ITEMS_PER_WAVE * FB_WAVES * sizeof(uint2)));
    if (!d->d_fb_ss) HIP_TRY(hipMalloc((void **)&d->d_fb_ss, (size_t)(FB_DEPTH_MAX + 2) * FB_WAVES * sizeof(uint32_t)));
    return ZF_OK;
}

// Tokens that the cache rows `ent` together leave to the parser: the bits of any row's second words that are in no row's first words.
// A stretch of words at a time, so that every loop is a plain one over neighbours.
uint32_t undecided_tokens(const std::vector<uint2> &ci_tok, size_t W, const uint32_t *ent, uint32_t n) {
    static const size_t STRETCH = 512;
    uint64_t both[STRETCH];
    uint32_t left[STRETCH], cnt = 0;
    for (size_t w0 = 0; w0 < W; w0 += STRETCH) {
        const size_t m = std::min(STRETCH, W - w0);
        std::fill(both, both + m, 0);
        for (uint32_t k = 0; k < n; k++) {
            const uint2 *row = ci_tok.data() + ent[k] * W + w0;
            for (size_t j = 0; j < m; j++) both[j] |= (uint64_t)row[j].y << 32 | row[j].x;
        }
        for (size_t j = 0; j < m; j++) left[j] = (uint32_t)(both[j] >> 32) & ~(uint32_t)both[j];
        for (size_t j = 0; j < m; j++) cnt += (uint32_t)__builtin_popcount(left[j]);
    }
    return cnt;
}

// The device's part of an engine, in two: what needs the grammar's tables and the vocabulary as it came -- the cache rows in token order are
// on their way when this returns --, and, when the vocabulary has been sorted (setup_device), the rest.
size_t engine_bytes(const zf_engine *e);
int begin_device(zf_engine *e) {
    DeviceSide *d = new (std::nothrow) DeviceSide();
    if (!d) return fail(ZF_ERR_OOM, "out of memory");
    e->dev = d;
    d->device = e->opt.device;
    HIP_TRY(hipSetDevice(d->device));
    const Tables &t = e->tab;
    DeviceTables &T = d->tab;
    T.V = e->V; T.W = e->W;
    int rc = engine_reserve(d, engine_bytes(e));
    if (rc != ZF_OK) return rc;
    std::vector<uint8_t> cls(t.cls, t.cls + 256);
    {   // the grammar tables in one allocation, in the order the kernels lay them out in LDS, each padded
        // to 16 bytes: a block stages whatever prefix fits with one flat copy
        std::vector<uint8_t> blob;
        size_t at[8];
        auto add = [&](const void *p, size_t bytes, uint32_t *padded, int k) {
            at[k] = blob.size();
            const size_t pad = (std::max<size_t>(bytes, 16) + 15) & ~(size_t)15;
            blob.resize(blob.size() + pad, 0);
            if (bytes) memcpy(blob.data() + at[k], p, bytes);
            *padded = (uint32_t)pad;
        };
        add(t.advpq.data(), t.advpq.size() * 4, &T.small_bytes[0], 0); add(cls.data(), cls.size(), &T.small_bytes[1], 1);
        add(t.qinfo.data(), t.qinfo.size() * 4, &T.small_bytes[2], 2); add(t.scan_off.data(), t.scan_off.size() * 4, &T.small_bytes[3], 3);
        add(t.comp_off.data(), t.comp_off.size() * 4, &T.small_bytes[4], 4);
        add(t.delta_dense.data(), t.delta_dense.size() * 4, &T.big_bytes[0], 5); add(t.dev_scan_list.data(), t.dev_scan_list.size() * 4, &T.big_bytes[1], 6);
        add(t.dev_comp_list.data(), t.dev_comp_list.size() * 4, &T.big_bytes[2], 7);
        const uint8_t *dev = nullptr;
        if ((rc = upload(d, blob, &dev)) != ZF_OK) return rc;
        T.table_blob = dev;
        T.advpq = (const uint32_t *)(dev + at[0]); T.cls = dev + at[1]; T.qinfo = (const uint32_t *)(dev + at[2]);
        T.scan_off = (const uint32_t *)(dev + at[3]); T.comp_off = (const uint32_t *)(dev + at[4]); T.delta = (const uint32_t *)(dev + at[5]);
        T.scan_list = (const uint32_t *)(dev + at[6]); T.comp_list = (const uint32_t *)(dev + at[7]);
    }
    {   // the DFAs as the kernels that make cache rows read them
        VocabRows &r = d->voc;
        std::vector<uint32_t> first_off(1, 0), first_state;
        for (int Y = 0; Y < t.N; Y++) {
            for (uint16_t term : t.first_terms[Y]) first_state.push_back(t.term_start[term]);
            first_off.push_back((uint32_t)first_state.size());
        }
        if ((rc = upload(d, t.delta, &r.delta)) != ZF_OK || (rc = upload(d, t.qflags, &r.qflags)) != ZF_OK || (rc = upload(d, first_off, &r.first_off)) != ZF_OK ||
            (rc = upload(d, first_state, &r.first_state)) != ZF_OK || (rc = upload(d, e->follow.behind, &r.behind)) != ZF_OK || (rc = upload(d, e->follow.next, &r.follow)) != ZF_OK ||
            (rc = upload(d, e->follow.sure_behind, &r.sure_behind)) != ZF_OK || (rc = upload(d, e->follow.sure_next, &r.sure_next)) != ZF_OK) return rc;
        r.cls = T.cls; r.Q = (uint32_t)t.Q; r.N = (uint32_t)t.N; r.n_cls = (uint32_t)t.n_cls;
    }
    if (e->rows_on) {
        // The mask kernels over the persistent automaton, and mask_look_kernel for calls that leave nothing to any, work in token order: every token's string as byte classes, and the
        // rows of the token-mask cache with one bit per token.
        const size_t V = (size_t)e->V, W = (size_t)e->W, n_rows = (size_t)(t.Q + t.N);   // a row each, of a vocabulary without a string too: the kernels read them
        const int64_t *off = nullptr;
        VocabRows &r = d->voc;
        Str16 *tok16 = nullptr;
        if ((rc = upload(d, e->voc_off, &off)) != ZF_OK || (rc = upload(d, e->voc_bytes, &r.bytes)) != ZF_OK || (rc = engine_alloc(d, V * sizeof(Str16), &tok16)) != ZF_OK ||
            (rc = engine_alloc(d, n_rows * W * sizeof(uint2), &r.both)) != ZF_OK || (rc = engine_alloc(d, n_rows * 4, &r.counts)) != ZF_OK) return rc;
        r.n = (uint32_t)V; r.words = (uint32_t)W;
        HIP_TRY(hipMemsetAsync(r.counts, 0, n_rows * 4, nullptr));
        HIP_TRY(launch_vocab_tokens(off, r.bytes, r.cls, r.n, tok16, nullptr));
        HIP_TRY(launch_vocab_rows(r, off, nullptr));
        T.tok16 = tok16; T.ci_tok = r.both;
    }
    return ZF_OK;
}

// Device memory that the engine is going to ask for, rather too much than too little (the trie has at most a node per byte of the vocabulary).
size_t engine_bytes(const zf_engine *e) {
    const Tables &t = e->tab;
    const size_t V = (size_t)e->V, W = (size_t)e->W + 1, n_rows = (size_t)(t.Q + t.N), text = e->voc_bytes.size(), cap = store_cap_states(t.n_cls), ncls = (size_t)std::max(t.n_cls, 1);
    size_t n = ((size_t)1 << 20) + 4 * (t.advpq.size() + t.qinfo.size() + t.scan_off.size() + t.comp_off.size() + t.delta_dense.size() + t.dev_scan_list.size() + t.dev_comp_list.size()) + 2 * (t.delta.size() + e->follow.behind.size() + e->follow.next.size() + e->follow.sure_behind.size() + e->follow.sure_next.size());
    n += text * (sizeof(TrieNode) + 4 + 2) + (V / (size_t)e->opt.chunk_strings + 1) * (8 + CHUNK_ANC * sizeof(TrieNode)) + V * (4 + 4 + sizeof(Str16)) + n_rows * W * 8;
    if (e->rows_on) n += V * (8 + sizeof(Str16)) + text + n_rows * (W * 8 + 4);
    if (e->store_on) n += cap * (sizeof(uint2) + ncls * 4 + 16) + STORE_CAP_ITEMS * sizeof(uint2) + (size_t)MAX_BATCH * 4;
    if (e->opt.state_cache_entries > 0) n += (size_t)e->opt.state_cache_entries * W * 4;
    return n;
}

// The host's copy of the rows in token order, and their counts, when the kernels have made them.
int fetch_rows(zf_engine *e) {
    DeviceSide *d = e->dev;
    const size_t n_rows = (size_t)(e->tab.Q + e->tab.N), W = (size_t)e->W;
    HIP_TRY(hipSetDevice(d->device));
    d->ci_undecided.assign(std::max<size_t>(n_rows, 1), 0);
    if (e->store_on) d->h_ci_tok.resize(std::max<size_t>(n_rows * W, 1));
    if (n_rows) HIP_TRY(hipMemcpy(d->ci_undecided.data(), d->voc.counts, n_rows * 4, hipMemcpyDeviceToHost));
    if (e->store_on && n_rows * W) HIP_TRY(hipMemcpy(d->h_ci_tok.data(), d->voc.both, n_rows * W * sizeof(uint2), hipMemcpyDeviceToHost));
    return ZF_OK;
}

int setup_device(zf_engine *e) {
    DeviceSide *d = e->dev;
    const Tables &t = e->tab;
    const Trie &tr = e->trie;
    DeviceTables &T = d->tab;
    int rc;
#define UP(field, vec, bytes) if ((rc = upload(d, vec, &T.field, bytes)) != ZF_OK) return rc
    UP(nodes, tr.nodes, nullptr); UP(parent, tr.parent, nullptr); UP(chunk_begin, tr.chunk_begin, nullptr); UP(chunk_end, tr.chunk_end, nullptr);
    UP(chunk_anc, tr.chunk_anc, nullptr); UP(rank_of, tr.rank_of, nullptr);
    {   // in rank order, for the per-block automaton and the trie walk: the distinct strings as class strings, and the cache rows
        std::vector<uint8_t> rep(std::max(t.n_cls, 1), 0);
        for (int b = 255; b >= 0; b--) rep[t.cls[b]] = (uint8_t)b;
        UP(str_off, tr.str_off, nullptr); UP(cls_rep, rep, nullptr);
        const size_t n = (size_t)tr.n_strings, words = (size_t)(t.Q + t.N) * (size_t)tr.Wr;
        VocabRows r = d->voc;
        uint8_t *str_cls = nullptr;
        Str16 *str16 = nullptr;
        if ((rc = upload(d, tr.str_bytes, &r.bytes)) != ZF_OK || (rc = engine_alloc(d, tr.str_bytes.size(), &str_cls)) != ZF_OK || (rc = engine_alloc(d, n * sizeof(Str16), &str16)) != ZF_OK ||
            (rc = engine_alloc(d, words * 4, &r.valid)) != ZF_OK || (rc = engine_alloc(d, words * 4, &r.undecided)) != ZF_OK) return rc;
        r.both = nullptr; r.counts = nullptr; r.n = (uint32_t)n; r.words = (uint32_t)tr.Wr;
        HIP_TRY(launch_vocab_strings(T.str_off, r.bytes, r.cls, r.n, str_cls, str16, nullptr));
        HIP_TRY(launch_vocab_rows(r, T.str_off, nullptr));
        T.str_cls = str_cls; T.str16 = str16; T.ci_valid = r.valid; T.ci_cd = r.undecided;
    }
    T.Q = t.Q;
#undef UP
    T.N = t.N; T.n_cls = t.n_cls; T.end_base = t.end_base; T.n_nodes = (int)tr.nodes.size(); T.n_chunks = (int)tr.chunk_begin.size();
    T.n_strings = tr.n_strings; T.chunk_ranks = tr.chunk_ranks;
    T.Wr = tr.Wr;
    d->mode = choose_table_mode(T);
    HIP_TRY(prepare_kernels());
    HIP_TRY(hipDeviceGetAttribute(&d->cus, hipDeviceAttributeMultiprocessorCount, d->device));
    if (e->opt.state_cache_entries > 0 && e->W > 0) {
        d->cache.resize(e->opt.state_cache_entries);
        if ((rc = engine_alloc(d, (size_t)e->opt.state_cache_entries * e->W * 4, &d->d_pool)) != ZF_OK) return rc;
    }
    if (walk_lds_bytes(T, d->mode, e->opt.lane_item_cap) > 160u * 1024u)
        return fail(ZF_ERR_INVALID_ARG, "lane_item_cap and the grammar tables do not fit the 160 KB of LDS");
    if ((rc = engine_alloc(d, 2 * COUNTER_SET_WORDS * 4, &d->d_counters)) != ZF_OK) return rc;     // two sets of counters (see MaskArgs::counters)
    HIP_TRY(hipMemset(d->d_counters, 0, 2 * COUNTER_SET_WORDS * 4));
    {   // staging room every engine has from the start (zf_compute_mask_noalloc never grows it), and status words
        const size_t status = 32 * DeviceSide::N_SLOTS, store_status = e->rows_on ? DeviceSide::N_SLOTS * STORE_STATUS_WORDS * 8 : 0;
        HIP_TRY(hipHostMalloc(&d->h_block, DeviceSide::N_SLOTS * NOALLOC_STAGE_BYTES + status + store_status, hipHostMallocDefault));
        uint8_t *at = (uint8_t *)d->h_block;
        for (int k = 0; k < DeviceSide::N_SLOTS; k++, at += NOALLOC_STAGE_BYTES) { d->h_stage[k] = at; d->stage_cap[k] = NOALLOC_STAGE_BYTES; }
        memset(at, 0, status + store_status);
        d->h_status = (uint32_t *)at;
        if (e->rows_on) d->h_store_status = (volatile uint64_t *)(at + status);
    }
    if (e->rows_on) {
        if ((rc = engine_alloc(d, 2 * STORE_TICKETS * 8, &d->d_tickets)) != ZF_OK) return rc;
        HIP_TRY(hipMemset(d->d_tickets, 0, 2 * STORE_TICKETS * 8));
        if (!e->store_on && (rc = upload(d, std::vector<uint32_t>((size_t)std::max(t.n_cls, 1), HostAutomaton::NONE), &d->no_trans)) != ZF_OK) return rc;
    }
    if (e->store_on) {
        // Room of the persistent automaton: states x byte classes transition words (at most 128 MB), 4 M items, a hash table of
        // twice as many slots as states.  The host clears the store when it is half full (see enqueue_mask_impl).
        StoreView &G = d->store;
        const uint32_t cap = store_cap_states(t.n_cls);
        G.cap_states = cap; G.cap_items = STORE_CAP_ITEMS; G.intern_mask = 2 * cap - 1;
        if ((rc = engine_alloc(d, (size_t)G.cap_states * sizeof(uint2), &G.hdr)) != ZF_OK) return rc;
        if ((rc = engine_alloc(d, (size_t)G.cap_items * sizeof(uint2), &G.arena)) != ZF_OK) return rc;
        if ((rc = engine_alloc(d, (size_t)G.cap_states * std::max(t.n_cls, 1) * 4, &G.trans)) != ZF_OK) return rc;
        if ((rc = engine_alloc(d, ((size_t)G.intern_mask + 1) * 8, &G.intern)) != ZF_OK) return rc;
        if ((rc = engine_alloc(d, 64, &G.ctl)) != ZF_OK) return rc;
        if ((rc = engine_alloc(d, (size_t)MAX_BATCH * 4, &d->d_import_root)) != ZF_OK) return rc;
        {
            const StoreConst k{d->tab, G};
            if ((rc = engine_alloc(d, sizeof k, &d->d_konst)) != ZF_OK) return rc;
            HIP_TRY(hipMemcpy(d->d_konst, &k, sizeof k, hipMemcpyHostToDevice));
        }
        Chart c0;                                        // the empty prefix's set, completed items dropped, as device item words
        chart_init(t, c0);
        std::vector<uint32_t> root;
        for (const Item &it : c0.items) {
            if ((t.sym[it.p] >> SYM_KIND_SHIFT) == SYM_END) continue;
            const uint32_t aw = t.advpq[it.p];
            root.push_back((aw & IW_TERM) ? ((aw & 0xFFFFu) | ((uint32_t)it.q << 16)) : aw);
            root.push_back(0);
        }
        d->n_root = (uint32_t)root.size() / 2;
        if ((rc = engine_alloc(d, root.size() * 4, (uint32_t **)&d->d_root_items)) != ZF_OK) return rc;
        if (!root.empty()) HIP_TRY(hipMemcpy(d->d_root_items, root.data(), root.size() * 4, hipMemcpyHostToDevice));
        d->store_dirty = true;
    }
    HIP_TRY(scratch_init(d->device));                    // once per device, with that device current
    d->scratch = (uint8_t *)scratch_ptr(d->device);
    if (!d->scratch) return fail(ZF_ERR_DEVICE, "the device address of the static scratch array is unknown");
    if (!e->store_on) return alloc_fallback(d);          // an engine with a persistent automaton may never need it: on first use
    return ZF_OK;
}

// Rows of the token-mask cache that the items of the current set select: the DFA state of an
// item that stands inside (or before) a terminal, Q + Y for an item that waits for nonterminal Y.
uint32_t current_set_entries(const Tables &t, const Item *items, uint32_t n_items, uint32_t *out) {
    uint32_t n = 0;
    for (uint32_t i = 0; i < n_items; i++) {
        uint16_t code = t.sym[items[i].p];
        uint32_t row;
        if ((code >> SYM_KIND_SHIFT) == SYM_TERM) row = items[i].q;
        else if ((code >> SYM_KIND_SHIFT) == SYM_NT) row = (uint32_t)t.Q + (code & SYM_ID_MASK_NT);
        else continue;
        bool dup = false;
        for (uint32_t k = 0; k < n && !dup; k++) dup = out[k] == row;
        if (!dup) out[n++] = row;
    }
    return n;
}
uint32_t current_set_entries(const Tables &t, const Chart &c, uint32_t *out) {
    const uint32_t lo = c.set_off[c.n_sets() - 1];
    return current_set_entries(t, c.items.data() + lo, c.set_off[c.n_sets()] - lo, out);
}

static const size_t HOST_LAG_MAX = 1u << 16;          // bytes a chart may lag behind before it is brought up to date anyway
static const int64_t HOST_AUT_ITEMS_MAX = 1 << 25;    // the host automaton is emptied when it is full or holds more items than this

// The state's place in the host automaton (the caller holds the engine's lock).
uint32_t host_place(zf_state *s) {
    zf_engine *e = s->eng;
    if (s->host_id == HostAutomaton::ROOT || s->host_id_epoch == e->host_epoch) return s->host_id;
    const uint32_t at = e->host_aut->import(chart_of(s));   // the automaton was emptied since: the chart says where the state stands
    if (at == 0) return 0;                             // no room
    s->host_id = at; s->host_id_epoch = e->host_epoch;
    return s->host_id;
}

// The items of the state's current set and the size of the largest set its chart holds -- from the host automaton when the
// engine has one (the caller holds its lock; the chart may lag behind), else from the chart.
struct CurrentSet { const Item *items; uint32_t n, biggest; };
CurrentSet current_set(zf_state *s) {
    zf_engine *e = s->eng;
    if (e->host_aut) {
        const uint32_t at = host_place(s);
        if (at == HostAutomaton::SINK) return CurrentSet{nullptr, 0, 0};
        if (at == 0) {                                     // the automaton has no room for the state's chart: the chart itself, then
            const Chart &c = chart_of(s);
            uint32_t biggest = 0;
            for (uint32_t k = 0; k < c.n_sets(); k++) biggest = std::max(biggest, c.set_off[k + 1] - c.set_off[k]);
            const uint32_t lo = c.set_off[c.n_sets() - 1];
            return CurrentSet{c.items.data() + lo, c.set_off[c.n_sets()] - lo, biggest};
        }
        const HostAutomaton &A = *e->host_aut;
        const HostAutomaton::State &hs = A.st(at);
        return CurrentSet{hs.items, hs.n_items, hs.widest};
    }
    const Chart &c = s->chart;
    uint32_t biggest = 0;
    for (uint32_t k = 0; k < c.n_sets(); k++) biggest = std::max(biggest, c.set_off[k + 1] - c.set_off[k]);
    const uint32_t lo = c.set_off[c.n_sets() - 1];
    return CurrentSet{c.items.data() + lo, c.set_off[c.n_sets()] - lo, biggest};
}

int feed_token_bytes(zf_state *s, const uint8_t *bytes, int64_t n) {
    if (n <= 0) return fail(ZF_ERR_REJECTED, "an empty token is never allowed");
    const Tables &t = s->eng->tab;
    const bool pruning = s->eng->opt.pruning != 0;
    if (s->eng->host_aut) {
        // Through the host automaton: a look-up per byte once the transition is known (Sections 4.4, 5.2: nothing is parsed
        // twice), an Earley byte step the first time -- run without the lock (the sets it reads do not change), so
        // that the rows of a batch can be fed by several threads.  All or nothing, as below.
        zf_engine *e = s->eng;
        HostAutomaton &A = *e->host_aut;
        std::unique_lock<std::mutex> lk(e->host_mu);
        while (A.full() || A.n_items > HOST_AUT_ITEMS_MAX) {   // start over; the states find their way back through their charts
            if (e->host_walkers == 0) { A.clear(); e->host_epoch++; break; }
            lk.unlock();                                  // somebody is at work on a transition (and waits for nobody): let them finish
            std::this_thread::yield();
            lk.lock();
        }
        if (s->host_id != HostAutomaton::ROOT && s->host_id_epoch != e->host_epoch) {
            lk.unlock();
            const Chart &c = chart_of(s);                 // the automaton was emptied since: the chart says where the state stands
            lk.lock();
            const uint32_t at = A.import(c);
            if (at == 0) return fail(ZF_ERR_OOM, "the chart is too large for the host automaton");
            s->host_id = at; s->host_id_epoch = e->host_epoch;
        }
        const uint32_t epoch = e->host_epoch;             // cannot change while this thread is a walker or holds the lock
        uint32_t at = s->host_id;
        bool accepted = false;
        for (int64_t i = 0; i < n; i++) {
            if (at == HostAutomaton::SINK) at = HostAutomaton::DEAD;
            else {
                const int cl = t.cls[bytes[i]];
                if (A.st(at).trans[cl] == HostAutomaton::NONE) {
                    static thread_local HostAutomaton::Work w;
                    e->host_walkers++;
                    lk.unlock();
                    A.look_ahead(at, cl, w);
                    lk.lock();
                    e->host_walkers--;
                    if (A.st(at).trans[cl] == HostAutomaton::NONE) A.record(at, cl, w);   // else somebody else has made it meanwhile
                }
                accepted = A.st(at).acc[cl] != 0;
                at = A.st(at).trans[cl];
            }
            if (at == HostAutomaton::DEAD || (at == HostAutomaton::SINK && i + 1 < n))
                return fail(ZF_ERR_REJECTED, "byte " + std::to_string(i) + " of the input cannot extend the prefix");
        }
        s->host_id = at; s->host_id_epoch = epoch;
        s->accepting = accepted;
        lk.unlock();
        s->bytes_fed += n;
        s->lag.insert(s->lag.end(), bytes, bytes + n);
        s->lag_cut.push_back((uint32_t)s->lag.size());
        if (s->lag.size() > HOST_LAG_MAX) catch_up(s);
    } else {
        Chart &c = s->chart;
        const uint32_t keep = c.n_sets();
        int64_t created = 0;
        bool accepted = false;
        for (int64_t i = 0; i < n; i++) {
            StepResult r = earley_step(t, c, bytes[i], !pruning, &created);
            accepted = r.accepted;
            // a byte is rejected when its set is empty; a completed sentence that cannot be extended
            // is still fine as the last byte
            if (!r.alive || (!r.kernel_nonempty && i + 1 < n)) {
                c.truncate(keep);
                return fail(ZF_ERR_REJECTED, "byte " + std::to_string(i) + " of the input cannot extend the prefix");
            }
        }
        s->accepting = accepted;
        s->items_created += created;
        s->bytes_fed += n;
        if (pruning) chart_compact(t, c);   // Compact: after Complete, before the next Predict
    }
    if (s->eng->store_on) {                               // the device walks the same bytes at the next mask call
        for (int64_t i = 0; i < n; i++) s->pending.push_back(t.cls[bytes[i]]);
        s->fed_total += (uint64_t)n;
        s->pending_token = -1;                            // zf_advance knows better
        if (s->pending.size() > (size_t)STORE_PENDING_MAX) {   // too far behind: the row comes in through its chart again
            s->pending.clear(); s->pending_base = s->fed_total; s->dev_id = 0; s->dev_epoch = 0;
        }
    }
    return ZF_OK;
}

}  // namespace

// Poll a word that a call's last kernel writes into pinned memory instead of synchronising the stream (which also waits for
// whatever the caller queued behind the mask kernels, apply_mask for one, and wakes up microseconds later).  Bounded: after
// two seconds `synchronise` is called, which also surfaces a device error.
template <class Arrived, class Sync>
static int await_status(Arrived arrived, Sync synchronise) {
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t spins = 0; !arrived(); spins++) {
        __builtin_ia32_pause();
        if ((spins & 0xFFFu) == 0xFFFu && std::chrono::steady_clock::now() - t0 > std::chrono::seconds(2)) {
            HIP_TRY(synchronise());
            if (!arrived()) return fail(ZF_ERR_DEVICE, "the mask kernels did not report back");
            break;
        }
    }
    std::atomic_thread_fence(std::memory_order_acquire);
    return ZF_OK;
}
// The words in which a call through mask_look_kernel reports.
static bool look_done(const volatile uint64_t *status, const DeviceSide::CallRecord &rec) {
    for (uint32_t g = 0; g < rec.done_groups; g++) if ((uint32_t)(status[STORE_ST_ROW + g] >> 32) != rec.seq) return false;
    return true;
}
static uint32_t look_failed(const volatile uint64_t *status, const DeviceSide::CallRecord &rec) {
    uint32_t n = rec.debug_failed;
    for (uint32_t g = 0; g < rec.done_groups; g++) n += (uint32_t)status[STORE_ST_ROW + g] & 0xFFFFFFu;
    return n;
}
// A call that zf_mask_wait has let go of ends before its slot is used again, before a call of the engine comes on another stream and
// before the store is touched by anything but a kernel behind it on its stream.  (After two seconds the device is synchronised: the
// call's stream may be gone by then.)
static void forget_cached_masks(DeviceSide *d);
static int settle_call(DeviceSide *d, uint32_t k) {
    DeviceSide::CallRecord &rec = d->rec[k];
    if (!rec.lazy) return ZF_OK;
    rec.lazy = false; d->n_lazy--;
    const volatile uint64_t *out = d->h_store_status + k * STORE_STATUS_WORDS;
    const int rc = await_status([&]() { return look_done(out, rec); }, [] { return hipDeviceSynchronize(); });
    if (rc != ZF_OK) return rc;
    const uint32_t failed = look_failed(out, rec);
    if (failed) { d->late_failed += failed; d->store_dirty = true; forget_cached_masks(d); }
    return ZF_OK;
}
// The failure of a call that zf_mask_wait has let go of, by a call that waits and has itself ended well.
static int report_late(DeviceSide *d) {
    if (!d->late_failed) return ZF_OK;
    const uint32_t n = d->late_failed;
    d->late_failed = 0;
    return fail(ZF_ERR_OVERFLOW, std::to_string(n) + " walks failed in a call of look-ups that zf_mask_wait had let go of: its mask is not valid (the one of the call that reports it is)");
}
static hipError_t next_call_number(DeviceSide *d, hipStream_t stream) {
    if (++d->call_seq != 0) return hipSuccess;
    d->call_seq = 1;                                      // numbers start over: no mask word lies about with one that comes again
    return d->d_tagged ? launch_clear_words((uint32_t *)d->d_tagged, (uint32_t)(d->tagged_cap * 2), stream) : hipSuccess;
}
// Whether work on `now` is behind what was enqueued on `then`.  (The handle of a thread's own stream is the same in every thread.)
static bool same_stream(hipStream_t now, hipStream_t then) { return now == then && now != hipStreamPerThread; }
static int settle_calls(DeviceSide *d) {
    int rc = ZF_OK;
    for (int k = 0; d->n_lazy && k < DeviceSide::N_SLOTS; k++) { const int r = settle_call(d, (uint32_t)k); if (rc == ZF_OK) rc = r; }
    return rc;
}

extern "C" {

const char *zf_strerror(int code) {
    switch (code) {
    case ZF_OK: return "ok";
    case ZF_ERR_INVALID_ARG: return "invalid argument";
    case ZF_ERR_GRAMMAR: return "invalid grammar";
    case ZF_ERR_REJECTED: return "input rejected by the grammar";
    case ZF_ERR_RANGE: return "token id out of range";
    case ZF_ERR_DEVICE: return "device error";
    case ZF_ERR_OOM: return "out of memory";
    case ZF_ERR_OVERFLOW: return "Earley set exceeded the fallback arena";
    }
    return "unknown error";
}
const char *zf_last_error(void) { return g_err.c_str(); }

static bool wants_exploration(const zf_engine *e);
static bool explore_host(zf_engine *e, size_t cap_states, size_t cap_items, std::unique_lock<std::mutex> *lk);
static void store_adopt(zf_engine *e, bool whole, std::unique_lock<std::mutex> *lk);
static std::vector<std::vector<uint32_t>> explored_entries(const zf_engine *e);
static void count_lists(zf_engine *e, const std::vector<std::vector<uint32_t>> &lists);

int zf_compile(const zf_grammar_desc *g, const zf_vocab_desc *v, const zf_options *opt, zf_engine **out) {
    if (!g || !v || !out || v->V < 0 || (v->V && !v->off)) return fail(ZF_ERR_INVALID_ARG, "null argument");
    for (int i = 0; i < v->V; i++) {
        int64_t n = v->off[i + 1] - v->off[i];
        if (n < 0 || n > MAX_TOKEN_LEN_ON_DEVICE) return fail(ZF_ERR_INVALID_ARG, "token " + std::to_string(i) + ": length must be 0..255");
    }
    zf_engine *e = new (std::nothrow) zf_engine();
    if (!e) return fail(ZF_ERR_OOM, "out of memory");
    e->opt = opt ? *opt : zf_options{1, 0, 0, 0, 0, 0, 0, 0, 0};
    e->lane_cap_auto = e->opt.lane_item_cap <= 0;
    if (e->opt.lane_item_cap <= 0) e->opt.lane_item_cap = LANE_CAP_DEFAULT;
    if (e->opt.lane_item_cap > LANE_CAP_MAX) e->opt.lane_item_cap = LANE_CAP_MAX;
    if (e->opt.fallback_item_cap <= 0 || e->opt.fallback_item_cap > FB_ITEMS_PER_WAVE) e->opt.fallback_item_cap = FB_ITEMS_PER_WAVE;
    if (e->opt.state_cache_entries == 0) e->opt.state_cache_entries = 2048;
    if (e->opt.state_cache_entries < 0) e->opt.state_cache_entries = 0;
    if (e->opt.state_cache_entries > 65536) e->opt.state_cache_entries = 65536;
    if (e->opt.chunk_strings != 8 && e->opt.chunk_strings != 16 && e->opt.chunk_strings != 32) e->opt.chunk_strings = 8;
    if (e->opt.precompute_states == 0) e->opt.precompute_states = 65536;
    if (e->opt.precompute_states < 0) e->opt.precompute_states = 0;
    // The exploration needs the grammar tables only: it runs beside everything else.  While the tables go to the device, its thread
    // counts what the explored states' lists of cache rows leave undecided.
    struct Explorer {
        std::thread thread;
        std::mutex mu;
        std::condition_variable cv;
        bool whole = false, explored = false, rows_made = false, stop = false;   // whole: explore_host's answer
        void tell(bool &what) { { std::lock_guard<std::mutex> lk(mu); what = true; } cv.notify_all(); }
        void await(const bool &what) { std::unique_lock<std::mutex> lk(mu); cv.wait(lk, [&]() { return what || stop; }); }
        void end() { if (thread.joinable()) { tell(stop); thread.join(); } }
        ~Explorer() { end(); }
    } explorer;
    struct Fetcher {                                      // brings the rows in token order back while the vocabulary is being sorted
        std::thread thread;
        int rc = ZF_OK;
        std::string error;
        void end() { if (thread.joinable()) thread.join(); }
        ~Fetcher() { end(); }
    } fetcher;
    auto give_up = [&](int rc) { explorer.end(); fetcher.end(); free_device(e->dev); delete e->host_aut; delete e; return rc; };
    try {
        if (!build_tables(g, e->tab)) { delete e; return ZF_ERR_GRAMMAR; }
        e->V = v->V; e->W = (v->V + 31) / 32;
        e->store_on = e->opt.device >= 0 && e->opt.walk_mode == 2 && e->opt.pruning != 0 && e->tab.n_cls <= (int)TOK_MORE;   // (a byte class for nearly every byte: the per-block automaton's records hold any class)
        e->rows_on = e->store_on || (e->opt.device >= 0 && e->opt.walk_mode == 2 && !e->opt.disable_token_mask_cache && e->lane_cap_auto && e->tab.n_cls <= (int)TOK_MORE);
        if (e->opt.walk_mode == 2 && e->opt.pruning != 0) e->host_aut = new HostAutomaton(e->tab);
        if (wants_exploration(e))
            explorer.thread = std::thread([e, &explorer]() {
                try { explorer.whole = explore_host(e, store_cap_states(e->tab.n_cls), STORE_CAP_ITEMS, nullptr); } catch (const std::bad_alloc &) {}   // what was learnt by then stands
                explorer.tell(explorer.explored);
                if (e->opt.disable_token_mask_cache) return;
                try {
                    const std::vector<std::vector<uint32_t>> lists = explored_entries(e);
                    explorer.await(explorer.rows_made);
                    if (explorer.rows_made) count_lists(e, lists);
                } catch (const std::bad_alloc &) {}       // the mask calls count, then
            });
        e->voc_off.assign(v->off, v->off + v->V + 1);
        e->voc_bytes.assign(v->bytes, v->bytes + v->off[v->V]);
        // an explicit item budget is there to see sets outgrow it: every string that a terminal leaves open is walked
        if (!e->lane_cap_auto || e->opt.disable_token_mask_cache) follow_everything(e->tab, e->follow);
        else if (e->opt.device >= 0) { build_follow(e->tab, e->follow); build_sure(e->tab, e->follow); }
        if (e->opt.device >= 0) {
            const int rc = begin_device(e);
            if (rc != ZF_OK) return give_up(rc);
        }
        if (e->rows_on)
            fetcher.thread = std::thread([e, &explorer, &fetcher]() {
                try { fetcher.rc = fetch_rows(e); } catch (const std::bad_alloc &) { fetcher.rc = fail(ZF_ERR_OOM, "out of memory"); }
                if (fetcher.rc == ZF_OK) explorer.tell(explorer.rows_made);
                else fetcher.error = zf_last_error();
            });
        build_trie(v, e->opt.chunk_strings, e->tab.cls, e->trie);
    } catch (const std::bad_alloc &) { return give_up(fail(ZF_ERR_OOM, "out of memory")); }
    catch (const std::system_error &) { return give_up(fail(ZF_ERR_OOM, "no thread to be had")); }
    if (e->opt.device >= 0) {
        int rc = setup_device(e);
        fetcher.end();
        if (rc == ZF_OK && fetcher.rc != ZF_OK) rc = fail(fetcher.rc, fetcher.error);
        if (rc != ZF_OK) return give_up(rc);
    }
    if (explorer.thread.joinable()) {
        explorer.await(explorer.explored);
        try { store_adopt(e, explorer.whole, nullptr); } catch (const std::bad_alloc &) {}   // the store starts empty, then
        explorer.thread.join();
    }
    // The kernels that make the strings and the cache rows are on the null stream, for which the caller's need not wait: what they write is there when
    // this returns.  (An engine without a persistent automaton has nothing behind them that waits; behind store_adopt the stream is idle.)
    if (e->dev) {
        const hipError_t rc = hipStreamSynchronize(nullptr);
        if (rc != hipSuccess) return give_up(fail(ZF_ERR_DEVICE, std::string("the tables' kernels: ") + hipGetErrorString(rc)));
    }
    *out = e;
    return ZF_OK;
}

void zf_engine_destroy(zf_engine *e) {
    if (!e) return;
    if (e->dev) { (void)hipSetDevice(e->dev->device); (void)settle_calls(e->dev); }
    free_device(e->dev);
    delete e->host_aut;
    delete e;
}

int zf_engine_get_info(const zf_engine *e, zf_engine_info *o) {
    if (!e || !o) return fail(ZF_ERR_INVALID_ARG, "null argument");
    o->V = e->V; o->W = e->W; o->n_nonterminals = e->tab.N; o->n_rules = e->tab.n_rules_kept; o->n_positions = e->tab.P;
    o->n_dfa_states = e->tab.Q; o->n_byte_classes = e->tab.n_cls; o->n_trie_nodes = (int)e->trie.nodes.size();
    o->n_strings = e->trie.n_strings; o->lane_item_cap = e->opt.lane_item_cap; o->device = e->opt.device;
    o->table_lds_mode = e->dev ? e->dev->mode : -1;
    return ZF_OK;
}

int zf_state_new(zf_engine *e, zf_state **out) {
    if (!e || !out) return fail(ZF_ERR_INVALID_ARG, "null argument");
    zf_state *s = new (std::nothrow) zf_state();
    if (!s) return fail(ZF_ERR_OOM, "out of memory");
    s->eng = e;
    s->link = std::make_shared<StateLink>(StateLink{s});
    *out = s;
    return zf_state_reset(s);
}

int zf_state_reset(zf_state *s) {
    if (!s) return fail(ZF_ERR_INVALID_ARG, "null argument");
    const Tables &t = s->eng->tab;
    chart_init(t, s->chart);
    // the empty prefix is a sentence iff the start symbol is nullable: then the initial set holds
    // the completed start rule; drop completed items as every later set does (pruning on)
    s->accepting = false;
    Chart &c = s->chart;
    size_t w = 0;
    for (size_t i = 0; i < c.items.size(); i++) {
        bool done = (t.sym[c.items[i].p] >> SYM_KIND_SHIFT) == SYM_END;
        if (done) s->accepting = true;
        if (!done || !s->eng->opt.pruning) c.items[w++] = c.items[i];
    }
    c.items.resize(w);
    c.set_off[1] = (uint32_t)w;
    s->items_created = 0; s->bytes_fed = 0;
    s->dev_id = STORE_ROOT_ID; s->dev_epoch = 0; s->generation++;
    s->pending.clear(); s->pending_base = s->fed_total; s->pending_token = -1;
    s->lag.clear(); s->lag_cut.clear();
    s->host_id = HostAutomaton::ROOT; s->host_id_epoch = 0;
    return ZF_OK;
}

int zf_state_clone(const zf_state *s, zf_state **out) {
    if (!s || !out) return fail(ZF_ERR_INVALID_ARG, "null argument");
    zf_state *c = new (std::nothrow) zf_state(*s);
    if (!c) return fail(ZF_ERR_OOM, "out of memory");
    c->link = std::make_shared<StateLink>(StateLink{c});
    *out = c;
    return ZF_OK;
}

void zf_state_destroy(zf_state *s) {
    if (s && s->link) s->link->s = nullptr;               // calls in flight must not write to a state that is gone (the engine may be gone already)
    delete s;
}

int zf_advance(zf_state *s, int32_t token) {
    if (!s) return fail(ZF_ERR_INVALID_ARG, "null argument");
    const zf_engine *e = s->eng;
    if (token < 0 || token >= e->V) return fail(ZF_ERR_RANGE, "token id out of range");
    const bool fresh = s->pending.empty();
    const int rc = feed_token_bytes(s, e->voc_bytes.data() + e->voc_off[token], e->voc_off[token + 1] - e->voc_off[token]);
    if (rc == ZF_OK && fresh && !s->pending.empty()) s->pending_token = token;   // the device will walk exactly this token from the state it knows
    return rc;
}

// Rows of a batch are independent (one state = one query).  A byte step of an ambiguous grammar
// costs O(set size squared) on the host, so a batch of wide charts is dealt to a few worker
// threads; batches of small charts (the common case: a pruned chart's sets hold a handful of
// items, Section 4.2) are fed by the caller's thread, where waking anybody would cost more than
// the work.
namespace {

struct AdvanceJob {
    zf_state *const *states;
    const int32_t *ids;          // null: the job is to bring the rows' charts up to date
    int32_t n;
    int32_t *rc;                 // [n]
    std::string *err;            // [n] the error text of a row that failed
    std::atomic<int32_t> next{0}, done{0};
};

int advance_one(zf_state *s, int32_t id) { return id < 0 ? zf_state_reset(s) : zf_advance(s, id); }

bool advance_rows(AdvanceJob &j) {   // takes rows until none is left; true if it fed any
    bool any = false;
    for (;;) {
        const int32_t b = j.next.fetch_add(1, std::memory_order_relaxed);
        if (b >= j.n) return any;
        if (j.ids) j.rc[b] = advance_one(j.states[b], j.ids[b]);
        else { (void)chart_of(j.states[b]); j.rc[b] = ZF_OK; }
        if (j.rc[b] != ZF_OK) j.err[b] = zf_last_error();   // the text lives in the worker's thread: hand it over
        j.done.fetch_add(1, std::memory_order_release);
        any = true;
    }
}

class AdvancePool {              // created on first use, never destroyed: its threads sleep until the process ends
  public:
    explicit AdvancePool(int n_workers) : n_workers_(n_workers), pid_(getpid()) {
        for (int i = 0; i < n_workers; i++) std::thread([this] { loop(); }).detach();
    }
    bool usable() const { return n_workers_ > 0 && pid_ == getpid(); }   // a forked child has the object but not the threads
    // The caller feeds rows too and returns when every row is done; a worker that wakes up late finds
    // no row left and never touches the caller's arrays (the job object itself is shared).
    void run(const std::shared_ptr<AdvanceJob> &j) {
        {
            std::lock_guard<std::mutex> lk(m_);
            job_ = j; epoch_++;
        }
        cv_work_.notify_all();
        advance_rows(*j);
        std::unique_lock<std::mutex> lk(m_);
        cv_done_.wait(lk, [&] { return j->done.load(std::memory_order_acquire) == j->n; });
        job_.reset();
    }

  private:
    void loop() {
        uint64_t seen = 0;
        for (;;) {
            std::shared_ptr<AdvanceJob> j;
            {
                std::unique_lock<std::mutex> lk(m_);
                cv_work_.wait(lk, [&] { return epoch_ != seen; });
                seen = epoch_;
                j = job_;
            }
            if (j && advance_rows(*j)) {
                { std::lock_guard<std::mutex> lk(m_); }     // the caller is either before its check or already waiting
                cv_done_.notify_one();
            }
        }
    }
    std::mutex m_;
    std::condition_variable cv_work_, cv_done_;
    std::shared_ptr<AdvanceJob> job_;
    uint64_t epoch_ = 0;
    int n_workers_ = 0;
    pid_t pid_;
};

std::mutex g_pool_mutex;         // one batch at a time through the pool; a second caller feeds its rows itself
AdvancePool *g_pool = nullptr;

// Host cost of feeding the rows' tokens, in item visits: Scan reads the current set once per byte,
// Complete of an ambiguous grammar pairs its items with each other, Compact sweeps the chart.
const int64_t ADVANCE_PARALLEL_FROM = 12000;   // about 0.1 ms of one core: below that the hand-over costs more than it saves
int64_t advance_cost(zf_state *const *states, const int32_t *ids, int32_t n) {
    int64_t cost = 0;
    for (int32_t b = 0; b < n; b++) {
        const zf_state *s = states[b];
        if (!s || ids[b] < 0 || ids[b] >= s->eng->V) continue;
        if (s->eng->host_aut) {
            // a walk through the host automaton costs nothing unless it meets a transition nobody has taken: then one Earley
            // byte step per byte from there on is the likely cost
            zf_engine *e = s->eng;
            std::lock_guard<std::mutex> rl(e->host_mu);
            const HostAutomaton &A = *e->host_aut;
            const bool placed = s->host_id == HostAutomaton::ROOT || s->host_id_epoch == e->host_epoch;
            if (placed && s->host_id == HostAutomaton::SINK) continue;
            const uint8_t first = e->voc_bytes[(size_t)e->voc_off[ids[b]]];
            const bool has_bytes = e->voc_off[ids[b] + 1] > e->voc_off[ids[b]];
            if (placed && has_bytes && A.st(s->host_id).trans[e->tab.cls[first]] != HostAutomaton::NONE) continue;
            const int64_t last = placed ? (int64_t)A.st(s->host_id).n_items : 64, all = placed ? 8 * (int64_t)A.st(s->host_id).widest : 4096;
            cost += (e->voc_off[ids[b] + 1] - e->voc_off[ids[b]]) * (last + last * last / 16 + all);
            continue;
        }
        const Chart &c = chart_of(s);
        const int64_t last = c.set_off[c.n_sets()] - c.set_off[c.n_sets() - 1];
        cost += (s->eng->voc_off[ids[b] + 1] - s->eng->voc_off[ids[b]]) * (last + last * last / 16) + (int64_t)c.items.size();
    }
    return cost;
}

}  // namespace

// Bring the charts of a call's rows up to date (those fed through the host automaton lag behind): the same work as feeding
// them, so a batch of wide charts is dealt to the worker threads here as it is there.
static void catch_up_batch(zf_state *const *states, int32_t n) {
    int64_t cost = 0;
    int32_t lagging = 0;
    for (int32_t b = 0; b < n; b++) {
        const zf_state *s = states[b];
        if (!s || s->lag.empty()) continue;
        const Chart &c = s->chart;
        const int64_t last = c.set_off[c.n_sets()] - c.set_off[c.n_sets() - 1];
        cost += (int64_t)s->lag.size() * (last + last * last / 16) + (int64_t)c.items.size() * (int64_t)s->lag_cut.size();
        lagging++;
    }
    bool parallel = lagging >= 4 && cost >= ADVANCE_PARALLEL_FROM;
    if (parallel) {
        std::vector<const zf_state *> seen(states, states + n);
        std::sort(seen.begin(), seen.end());
        parallel = std::adjacent_find(seen.begin(), seen.end()) == seen.end();
    }
    std::unique_lock<std::mutex> pool_lock(g_pool_mutex, std::defer_lock);
    if (parallel) parallel = pool_lock.try_lock();
    if (parallel) {
        if (!g_pool) {
            const unsigned hw = std::thread::hardware_concurrency();
            g_pool = new AdvancePool((int)std::min(15u, std::max(1u, hw) - 1u));
        }
        parallel = g_pool->usable();
    }
    if (!parallel) {
        for (int32_t b = 0; b < n; b++) if (states[b]) (void)chart_of(states[b]);
        return;
    }
    std::vector<int32_t> rc((size_t)n, ZF_OK);
    std::vector<std::string> errs((size_t)n);
    auto job = std::make_shared<AdvanceJob>();
    job->states = states; job->ids = nullptr; job->n = n; job->rc = rc.data(); job->err = errs.data();
    g_pool->run(job);
}

int zf_advance_batch(zf_state *const *states, const int32_t *token_ids, int32_t n, int32_t *status) {
    if (!states || !token_ids || n < 0) return fail(ZF_ERR_INVALID_ARG, "null argument");
    for (int32_t b = 0; b < n; b++) if (!states[b]) return fail(ZF_ERR_INVALID_ARG, "null state");
    int first = ZF_OK;
    bool parallel = n >= 4 && advance_cost(states, token_ids, n) >= ADVANCE_PARALLEL_FROM;
    if (parallel) {                                       // every state at most once: a state named twice is fed twice, in order
        std::vector<const zf_state *> seen(states, states + n);
        std::sort(seen.begin(), seen.end());
        parallel = std::adjacent_find(seen.begin(), seen.end()) == seen.end();
    }
    std::unique_lock<std::mutex> pool_lock(g_pool_mutex, std::defer_lock);
    if (parallel) parallel = pool_lock.try_lock();
    if (parallel) {
        if (!g_pool) {
            const unsigned hw = std::thread::hardware_concurrency();
            g_pool = new AdvancePool((int)std::min(15u, std::max(1u, hw) - 1u));
        }
        parallel = g_pool->usable();
    }
    if (!parallel) {
        std::string first_err;
        for (int32_t b = 0; b < n; b++) {
            const int rc = advance_one(states[b], token_ids[b]);
            if (status) status[b] = rc;
            if (rc != ZF_OK && first == ZF_OK) { first = rc; first_err = zf_last_error(); }
        }
        if (first != ZF_OK) set_error(first_err);        // the caller sees the first failing row's text
        return first;
    }
    std::vector<int32_t> rc_store;
    if (!status) { rc_store.assign((size_t)n, ZF_OK); status = rc_store.data(); }
    std::vector<std::string> errs((size_t)n);
    auto job = std::make_shared<AdvanceJob>();
    job->states = states; job->ids = token_ids; job->n = n; job->rc = status; job->err = errs.data();
    g_pool->run(job);
    for (int32_t b = n - 1; b >= 0; b--)
        if (status[b] != ZF_OK) { first = status[b]; set_error(errs[b]); }
    return first;
}

int zf_advance_bytes(zf_state *s, const uint8_t *bytes, int64_t n) {
    if (!s || (n > 0 && !bytes) || n < 0) return fail(ZF_ERR_INVALID_ARG, "null argument");
    if (n == 0) return ZF_OK;
    return feed_token_bytes(s, bytes, n);
}

int zf_is_accepting(const zf_state *s, int32_t *out) {
    if (!s || !out) return fail(ZF_ERR_INVALID_ARG, "null argument");
    *out = s->accepting;
    return ZF_OK;
}

int zf_state_stats(const zf_state *s, zf_stats *o) {
    if (!s || !o) return fail(ZF_ERR_INVALID_ARG, "null argument");
    o->n_sets = chart_of(s).n_sets(); o->n_items = (int64_t)chart_of(s).items.size();
    o->items_created = s->items_created; o->bytes_fed = s->bytes_fed; o->accepting = s->accepting;
    return ZF_OK;
}

int zf_state_chart(const zf_state *s, int32_t *items, int64_t *set_off) {
    if (!s) return fail(ZF_ERR_INVALID_ARG, "null argument");
    if (items) for (size_t i = 0; i < chart_of(s).items.size(); i++) {
        items[3 * i] = chart_of(s).items[i].p; items[3 * i + 1] = (int32_t)chart_of(s).items[i].o; items[3 * i + 2] = chart_of(s).items[i].q;
    }
    if (set_off) for (size_t k = 0; k < chart_of(s).set_off.size(); k++) set_off[k] = chart_of(s).set_off[k];
    return ZF_OK;
}

int zf_position_info(const zf_engine *e, int32_t p, int32_t *lhs, int32_t *rule, int32_t *dot) {
    if (!e || p < 0 || p >= e->tab.P) return fail(ZF_ERR_INVALID_ARG, "bad position");
    if (lhs) *lhs = e->tab.pos_lhs_orig[p];
    if (rule) *rule = e->tab.pos_rule[p];
    if (dot) *dot = e->tab.pos_dot[p];
    return ZF_OK;
}

int zf_debug_host_mask(zf_engine *e, const zf_state *s, uint32_t *mask) { return zf_debug_host_mask_stats(e, s, mask, nullptr); }

int zf_debug_fail_look_ups(zf_engine *e, uint32_t walks) {
    if (!e || !e->dev) return fail(ZF_ERR_INVALID_ARG, "bad argument");
    e->dev->debug_failed = walks;
    return ZF_OK;
}

int zf_debug_look_polls(zf_engine *e, uint32_t polls) {
    if (!e || !e->dev) return fail(ZF_ERR_INVALID_ARG, "bad argument");
    e->dev->look_polls = polls;
    return ZF_OK;
}

int zf_debug_host_mask_cached(zf_engine *e, const zf_state *s, uint32_t *mask, int64_t *stats) {
    if (!e || !s || !mask || s->eng != e) return fail(ZF_ERR_INVALID_ARG, "bad argument");
    const Tables &t = e->tab;
    host_token_mask_cache(t, e->follow, e->trie);
    const Trie &tr = e->trie;
    Chart c = chart_of(s);
    const uint32_t m0 = c.n_sets();
    std::vector<uint32_t> ents(c.set_off[m0] - c.set_off[m0 - 1] + 1);
    const uint32_t n_ent = current_set_entries(t, c, ents.data());
    std::vector<uint32_t> valid(tr.Wr, 0), want(tr.Wr, 0);
    for (uint32_t k = 0; k < n_ent; k++)
        for (int w = 0; w < tr.Wr; w++) { valid[w] |= tr.ci_valid[(size_t)ents[k] * tr.Wr + w]; want[w] |= tr.ci_cd[(size_t)ents[k] * tr.Wr + w]; }
    for (int w = 0; w < tr.Wr; w++) want[w] &= ~valid[w];
    auto any_in = [&](uint32_t lo, uint32_t hi) { for (uint32_t r = lo; r < hi; r++) if ((want[r >> 5] >> (r & 31)) & 1) return true; return false; };
    int64_t n_steps = 0, n_wanted = 0, n_replay = 0, n_queued = 0;
    for (int w = 0; w < tr.Wr; w++) n_wanted += __builtin_popcount(want[w]);
    size_t chunk = 0;
    int64_t last_counted = -1;
    for (uint32_t i = 0; i < tr.nodes.size();) {
        const TrieNode &nd = tr.nodes[i];
        if (!any_in(nd.rank, nd.rank + nd.n_sub)) { i = nd.skip; continue; }
        while (chunk + 1 < tr.chunk_begin.size() && tr.chunk_end[chunk] <= i) chunk++;
        if ((int64_t)chunk != last_counted) {    // the kernel walks chunk by chunk and replays the path above each chunk's first node
            last_counted = (int64_t)chunk; n_queued++;
            n_replay += tr.nodes[tr.chunk_begin[chunk]].depth - 1;
        }
        c.truncate(m0 + nd.depth - 1);
        StepResult r = earley_step(t, c, nd.byte, false, nullptr);
        n_steps++;
        if (nd.has_string && r.alive && ((want[nd.rank >> 5] >> (nd.rank & 31)) & 1)) valid[nd.rank >> 5] |= 1u << (nd.rank & 31);
        i = r.kernel_nonempty ? i + 1 : nd.skip;
    }
    memset(mask, 0, sizeof(uint32_t) * e->W);
    for (int v = 0; v < e->V; v++) {
        uint32_t r = tr.rank_of[v];
        if (r != 0xFFFFFFFFu && ((valid[r >> 5] >> (r & 31)) & 1)) mask[v >> 5] |= 1u << (v & 31);
    }
    if (stats) { stats[0] = n_steps; stats[1] = n_wanted; stats[2] = n_ent; stats[3] = n_replay; stats[4] = n_queued; }
    return ZF_OK;
}

int zf_debug_host_mask_stats(zf_engine *e, const zf_state *s, uint32_t *mask, int64_t *stats) {
    if (!e || !s || !mask || s->eng != e) return fail(ZF_ERR_INVALID_ARG, "bad argument");
    int64_t n_steps = 0, n_alive = 0, max_path = 0, max_set = 0, chunks_over = 0;
    const int CHUNK_RANKS = e->trie.chunk_ranks;
    std::vector<uint8_t> chunk_over((e->trie.n_strings + CHUNK_RANKS - 1) / CHUNK_RANKS + 1, 0);
    const Tables &t = e->tab;
    const Trie &tr = e->trie;
    Chart c = chart_of(s);
    const uint32_t m0 = c.n_sets();
    std::vector<uint8_t> ok(tr.n_strings, 0);
    for (uint32_t i = 0; i < tr.nodes.size();) {
        const TrieNode &nd = tr.nodes[i];
        c.truncate(m0 + nd.depth - 1);
        StepResult r = earley_step(t, c, nd.byte, false, nullptr);
        if (nd.has_string && r.alive) ok[nd.rank] = 1;
        n_steps++; n_alive += r.alive;
        int64_t path = (int64_t)c.items.size() - c.set_off[m0];
        int64_t last = (int64_t)c.items.size() - c.set_off[c.n_sets() - 1];
        if (path > max_path) max_path = path;
        if (last > max_set) max_set = last;
        if (path > e->opt.lane_item_cap && !chunk_over[nd.rank / CHUNK_RANKS]) { chunk_over[nd.rank / CHUNK_RANKS] = 1; chunks_over++; }
        i = r.kernel_nonempty ? i + 1 : nd.skip;
    }
    if (stats) { stats[0] = n_steps; stats[1] = n_alive; stats[2] = max_path; stats[3] = max_set; stats[4] = chunks_over; }
    memset(mask, 0, sizeof(uint32_t) * e->W);
    for (int v = 0; v < e->V; v++) {
        uint32_t r = tr.rank_of[v];
        if (r != 0xFFFFFFFFu && ok[r]) mask[v >> 5] |= 1u << (v & 31);
    }
    return ZF_OK;
}

// The packed form of a chart: [n_sets][set offsets][item word, origin]...; what the kernels read, and the state cache's key.
static void pack_chart(const Tables &t, const Chart &c, std::vector<uint32_t> &k) {
    k.clear();
    k.push_back(c.n_sets());
    k.insert(k.end(), c.set_off.begin(), c.set_off.end());
    for (const Item &it : c.items) {   // host item -> device item word + origin
        const uint32_t aw = t.advpq[it.p];
        k.push_back((aw & IW_TERM) ? ((aw & 0xFFFFu) | ((uint32_t)it.q << 16)) : aw);
        k.push_back(it.o);
    }
}

// State cache (Section 5.2): find every row's pool slot by its packed chart; rows seen for the first time get a slot
// (round-robin victim, never one handed out in the same call) and are listed in miss_rows.  Returns the number of hits.
static int state_cache_lookup(DeviceSide *d, const std::vector<std::vector<uint32_t>> &packed, int32_t batch,
                              std::vector<uint32_t> &row_slot, std::vector<uint32_t> &miss_rows) {
    int n_hits = 0;
    const uint32_t call = ++d->cache_call;
    for (int b = 0; b < batch; b++) {
        const std::vector<uint32_t> &k = packed[b];
        uint64_t h = 0xCBF29CE484222325ull;
        for (uint32_t w : k) { h ^= w; h *= 0x100000001B3ull; h ^= h >> 29; }
        uint32_t found = 0xFFFFFFFFu;
        auto range = d->cache_index.equal_range(h);
        for (auto it = range.first; it != range.second; ++it) if (d->cache[it->second].key == k) { found = it->second; break; }
        if (found == 0xFFFFFFFFu) {
            while (d->cache[d->cache_victim].used && d->cache[d->cache_victim].stamp == call) d->cache_victim = (d->cache_victim + 1) % d->cache.size();
            found = d->cache_victim;
            d->cache_victim = (d->cache_victim + 1) % d->cache.size();
            DeviceSide::CacheEntry &ce = d->cache[found];
            if (ce.used) {   // evict
                auto r2 = d->cache_index.equal_range(ce.hash);
                for (auto it = r2.first; it != r2.second; ++it) if (it->second == found) { d->cache_index.erase(it); break; }
            }
            ce.hash = h; ce.key = k; ce.used = true;
            d->cache_index.emplace(h, found);
            miss_rows.push_back((uint32_t)b);
        } else n_hits++;
        d->cache[found].stamp = call;
        row_slot[b] = found;
    }
    return n_hits;
}

static int enqueue_store_impl(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, void *hip_stream, bool wait, bool noalloc, uint32_t slot);
static int enqueue_decided(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, hipStream_t stream, bool wait, uint32_t slot);
static int wait_for_calls(zf_engine *e, void *hip_stream);
static const int STORE_NO_ROOM = 1;                       // enqueue_store_impl: the call does not fit the memory at hand (noalloc); nothing was enqueued
// zf_compute_mask_apply_async: the logits the call's mask is to be applied to.  The mask kernel over the persistent automaton
// takes them along when it can (fused = true); whoever set the request launches the logit-masking kernel otherwise.
struct ApplyRequest { const void *logits = nullptr; void *out = nullptr; int64_t stride = 0; int32_t dtype = 0; bool fused = false; };
static thread_local ApplyRequest g_apply;

// Pack and upload the charts and enqueue the kernels of one compute_mask call: upload, mask kernel,
// closing kernel (fallback pass for what the mask kernel listed + permutation into token order),
// gather when the state cache is on.  wait = true: also wait and return the final status.
// noalloc = true (zf_compute_mask_noalloc): the state cache is passed by and nothing is allocated.  The persistent automaton has
// its memory since zf_compile (a step of 16 rows of a JSON schema takes 29 us through it, 61 through the per-block automaton, to
// which such calls went before); on the other paths every per-call device buffer is a slice of the device's static scratch array,
// and a call that does not fit the array or the staging room is refused.
static int enqueue_mask_impl(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, void *hip_stream, bool wait, bool noalloc, bool per_block) {
    if (!e || !states || batch <= 0 || batch > MAX_BATCH || !d_mask) return fail(ZF_ERR_INVALID_ARG, "bad argument (batch must be 1..4096)");
    DeviceSide *d = e->dev;
    if (!d) return fail(ZF_ERR_DEVICE, "engine was compiled without a device (device = -1)");
    hipStream_t stream = (hipStream_t)hip_stream;
    HIP_TRY(hipSetDevice(d->device));
    if (d->pending >= (uint32_t)DeviceSide::N_SLOTS) return fail(ZF_ERR_INVALID_ARG, "too many asynchronous mask calls in flight: call zf_mask_wait");
    const uint32_t slot = d->next_slot;
    // (no event marks the slot free: at most N_SLOTS calls are in flight between two zf_mask_wait calls, so the call that used it before has been waited for, or is now)
    if (d->n_lazy) {
        const int rc = same_stream(stream, d->lazy_stream) ? settle_call(d, slot) : settle_calls(d);
        if (rc != ZF_OK) return rc;
    }
    if (d->closing_open && !same_stream(stream, d->closing_stream)) {
        HIP_TRY(hipStreamWaitEvent(stream, d->closing_done, 0));
        d->closing_stream = stream;                       // which is behind it now
    }
    for (int b = 0; b < batch; b++)
        if (!states[b] || states[b]->eng != e) return fail(ZF_ERR_INVALID_ARG, "state " + std::to_string(b) + " is null or belongs to another engine");
    // (noalloc with an explicit item budget: the budget is one of the per-block automaton's wavefronts)
    if (e->store_on && !per_block && !(noalloc && !e->lane_cap_auto)) {
        const int rc = enqueue_store_impl(e, states, batch, d_mask, hip_stream, wait, noalloc, slot);
        if (rc != STORE_NO_ROOM) return rc;
    }
    catch_up_batch(states, batch);                        // these paths send the charts
    if (e->rows_on && !e->store_on && !noalloc && d->cache.empty()) {
        const int rc = enqueue_decided(e, states, batch, d_mask, stream, wait, slot);
        if (rc != STORE_NO_ROOM) return rc;
    }
    // ---- the packed form of every row: [n_sets][set offsets][item word, origin]... (also the cache key) ----
    static thread_local std::vector<std::vector<uint32_t>> packed;
    if ((int)packed.size() < batch) packed.resize(batch);
    for (int b = 0; b < batch; b++) pack_chart(e->tab, chart_of(states[b]), packed[b]);
    // ---- state cache: rows whose chart has been seen before only need their finished mask copied ----
    // (an engine with a persistent automaton keeps its finished rows by its names: a call that comes here instead serves none)
    const bool sc_asked = !noalloc && !d->cache.empty() && (size_t)batch * 2 <= d->cache.size(), sc = sc_asked && !e->store_on;
    static thread_local std::vector<uint32_t> row_slot, miss_rows;
    row_slot.assign(batch, 0);
    miss_rows.clear();
    int n_hits = 0;
    if (sc) n_hits = state_cache_lookup(d, packed, batch, row_slot, miss_rows);
    else for (int b = 0; b < batch; b++) miss_rows.push_back((uint32_t)b);
    // trie walk: rows with a wide current set first: their chunks are the expensive ones, and work that starts early does
    // not end up as the kernel's tail (the mask automaton gives every row its own blocks: the order does not matter there)
    if (e->opt.walk_mode == 1) std::stable_sort(miss_rows.begin(), miss_rows.end(), [&](uint32_t x, uint32_t y) {
        const Chart &cx = chart_of(states[x]), &cy = chart_of(states[y]);
        return cx.set_off[cx.n_sets()] - cx.set_off[cx.n_sets() - 1] > cy.set_off[cy.n_sets()] - cy.set_off[cy.n_sets() - 1];
    });
    const int nb = (int)miss_rows.size();                // rows that go through the kernels
    d->report.cache_hits = n_hits; d->report.cache_misses = sc_asked ? nb : 0;
    // ---- upload: [RowChart x nb][set offsets][items][cache rows of the token-mask cache][dst slot x nb][row slot x batch] ----
    size_t n_off = 0, n_items = 0, n_ent = 0, max_off = 0, max_items = 0, max_ent = 0;
    const bool use_cache = !e->opt.disable_token_mask_cache;
    for (int r = 0; r < nb; r++) {
        const Chart &c = chart_of(states[miss_rows[r]]);
        const size_t last = c.set_off[c.n_sets()] - c.set_off[c.n_sets() - 1];
        n_off += c.set_off.size();
        n_items += c.items.size();
        if (use_cache) n_ent += last;
        max_off = std::max(max_off, c.set_off.size()); max_items = std::max(max_items, c.items.size());
        if (use_cache) max_ent = std::max(max_ent, last);
    }
    // Mask automaton: when the rows' charts are of similar size each row's sections get the same room, so that a block
    // can request its row's sets, items and cache rows without waiting for the row's header (one memory round trip
    // instead of two; the round trip is over PCIe when the kernels read the staging slot directly).
    const bool uniform = e->opt.walk_mode != 1 && nb > 0 &&
                         (size_t)nb * (4 * max_off + 8 * max_items + 4 * max_ent) <= 2 * (4 * n_off + 8 * n_items + 4 * n_ent) + 4096;
    if (uniform) { n_off = (size_t)nb * max_off; n_items = (size_t)nb * max_items; n_ent = (size_t)nb * max_ent; }
    auto align16 = [](size_t x) { return (x + 15) & ~(size_t)15; };
    const size_t off_rows = 0, off_so = align16(sizeof(RowChart) * nb), off_items = align16(off_so + 4 * n_off);
    const size_t off_ent = align16(off_items + sizeof(Item) * n_items);
    const size_t off_dst = align16(off_ent + 4 * n_ent), off_rowslot = align16(off_dst + 4 * (size_t)nb);
    const size_t total = off_rowslot + 4 * (size_t)batch + 16;
    if (noalloc && total > d->stage_cap[slot])
        return fail(ZF_ERR_INVALID_ARG, "zf_compute_mask_noalloc: the packed charts (" + std::to_string(total) + " bytes) exceed the staging room of " +
                                        std::to_string(d->stage_cap[slot]) + " bytes");
    if (total > d->stage_cap[slot]) {
        const int rc = grow_stage(d, slot, total * 2 + 4096);
        if (rc != ZF_OK) return rc;
    }
    if (!noalloc && total > d->chart_cap) {
        HIP_TRY(hipStreamSynchronize(stream));            // earlier calls may still read the old buffer
        if (d->d_chart) (void)hipFree(d->d_chart);
        d->d_chart = nullptr; d->chart_cap = 0;
        size_t cap = total * 2 + 4096;
        HIP_TRY(hipMalloc(&d->d_chart, cap));
        d->chart_cap = cap;
    }
    uint32_t n_cache_rows = 0;                            // distinct rows of the token-mask cache, summed over the rows of the call
    {
        uint8_t *h = (uint8_t *)d->h_stage[slot];
        RowChart *rows = (RowChart *)(h + off_rows);
        uint32_t *so = (uint32_t *)(h + off_so);
        uint32_t *dev_items = (uint32_t *)(h + off_items);
        uint32_t *ents = (uint32_t *)(h + off_ent);
        uint32_t *dst = (uint32_t *)(h + off_dst);
        memcpy(h + off_rowslot, row_slot.data(), 4 * (size_t)batch);
        uint32_t so_at = 0, it_at = 0, en_at = 0;
        for (int r = 0; r < nb; r++) {
            const Chart &c = chart_of(states[miss_rows[r]]);
            const std::vector<uint32_t> &k = packed[miss_rows[r]];
            if (uniform) { so_at = (uint32_t)(r * max_off); it_at = (uint32_t)(r * max_items); en_at = (uint32_t)(r * max_ent); }
            rows[r] = RowChart{c.n_sets(), so_at, it_at, en_at, 0, (uint32_t)c.items.size(), {0, 0}};
            if (use_cache) rows[r].n_ent = current_set_entries(e->tab, c, ents + en_at);
            n_cache_rows += rows[r].n_ent;
            en_at += rows[r].n_ent;
            memcpy(so + so_at, k.data() + 1, 4 * c.set_off.size());
            memcpy(dev_items + 2 * (size_t)it_at, k.data() + 1 + c.set_off.size(), 8 * c.items.size());
            so_at += (uint32_t)c.set_off.size(); it_at += (uint32_t)c.items.size();
            dst[r] = sc ? row_slot[miss_rows[r]] : miss_rows[r];
        }
    }
    // ---- per-call device buffers ----
    const size_t need_rank = (size_t)std::max(nb, 1) * d->tab.Wr, need_ovf = 2 * (size_t)std::max(nb, 1) * d->tab.n_chunks;   // the automaton kernel may name a chunk in two entries
    // zf_compute_mask_noalloc: the same buffers as slices of the static array: [counters: 64 words][fallback set starts][fallback
    // arenas][rank-ordered verdict words][device copy of the charts (trie walk)][the trie walk's queue][fallback list: what is left]
    uint8_t *const scr = d->scratch;
    size_t scr_ss = 0, scr_fb = 0, scr_rank = 0, scr_chart = 0, scr_work = 0, scr_ovf = 0, scr_ovf_cap = 0;
    if (noalloc) {
        auto align256 = [](size_t x) { return (x + 255) & ~(size_t)255; };
        scr_ss = 1024;
        scr_fb = align256(scr_ss + (size_t)(FB_DEPTH_MAX + 2) * NOALLOC_FB_WAVES * 4);
        scr_rank = align256(scr_fb + (size_t)NOALLOC_FB_WAVES * NOALLOC_FB_ITEMS_PER_WAVE * sizeof(uint2));
        scr_chart = align256(scr_rank + need_rank * 4 + 16);
        scr_work = align256(scr_chart + (e->opt.walk_mode == 1 ? total + 16 : 0));
        scr_ovf = align256(scr_work + (e->opt.walk_mode == 1 ? (size_t)std::max(nb, 1) * d->tab.n_chunks * sizeof(uint4) + 16 : 0));
        if (scr_ovf + 4096 * sizeof(uint4) > NOALLOC_SCRATCH_BYTES)
            return fail(ZF_ERR_INVALID_ARG, "zf_compute_mask_noalloc: batch x vocabulary needs " + std::to_string(scr_ovf + 4096 * sizeof(uint4)) +
                                            " bytes of scratch memory, the static array holds " + std::to_string(NOALLOC_SCRATCH_BYTES));
        scr_ovf_cap = std::min(need_ovf, (NOALLOC_SCRATCH_BYTES - scr_ovf) / sizeof(uint4));   // a longer list fails the call loudly (ZF_ERR_OVERFLOW)
    } else if (need_rank > d->rank_cap || need_ovf > d->overflow_cap) {
        HIP_TRY(hipStreamSynchronize(stream));
        if (d->d_rank_mask) (void)hipFree(d->d_rank_mask);
        if (d->d_overflow) (void)hipFree(d->d_overflow);
        if (d->d_work) (void)hipFree(d->d_work);
        d->d_rank_mask = nullptr; d->d_overflow = nullptr; d->d_work = nullptr; d->rank_cap = d->overflow_cap = 0;
        HIP_TRY(hipMalloc((void **)&d->d_rank_mask, need_rank * 4 + 16));
        HIP_TRY(hipMalloc((void **)&d->d_overflow, need_ovf * sizeof(uint4) + 16));
        HIP_TRY(hipMalloc((void **)&d->d_work, need_ovf * sizeof(uint4) + 16));
        d->rank_cap = need_rank; d->overflow_cap = need_ovf;
    }
    if (!noalloc) { const int rc = alloc_fallback(d); if (rc != ZF_OK) return rc; }
    MaskArgs a{};
    a.tab = d->tab;
    // Where the kernels read the packed charts: with the mask automaton and the state cache off, straight from the pinned
    // staging slot (a block needs a few hundred bytes once; the copy to device memory would be a kernel of its own at the
    // head of the call); else from the device copy that upload_kernel makes.
    const bool direct = e->opt.walk_mode != 1 && !sc;
    uint8_t *chart_base = direct ? (uint8_t *)d->h_stage[slot] : (noalloc ? scr + scr_chart : (uint8_t *)d->d_chart);
    a.rows = (const RowChart *)(chart_base + off_rows);
    a.set_off = (const uint32_t *)(chart_base + off_so);
    a.items = (const Item *)(chart_base + off_items);
    a.entries = (const uint32_t *)(chart_base + off_ent);
    a.rank_mask = noalloc ? (uint32_t *)(scr + scr_rank) : d->d_rank_mask;
    a.out_mask = sc ? d->d_pool : d_mask;                 // with the state cache the rows are finished in their pool slots
    a.dst_row = direct ? nullptr : (const uint32_t *)(chart_base + off_dst);   // null: row r of the launch is row r of the output (no state cache: every row runs)
    a.row_slot = (const uint32_t *)(chart_base + off_rowslot);
    a.so_stride = uniform ? (uint32_t)max_off : 0u; a.it_stride = uniform ? (uint32_t)max_items : 0u; a.ent_stride = uniform ? (uint32_t)max_ent : 0u;
    a.user_mask = d_mask;
    a.user_batch = batch;
    a.handoff_in_permute = sc ? 0 : 1;
    if (noalloc) {                                        // cleared at the head of the call; counters_next is a spare set
        a.counters = (uint32_t *)scr; a.counters_next = (uint32_t *)scr + COUNTER_SET_WORDS;
    } else {
        a.counters = d->d_counters + COUNTER_SET_WORDS * d->call_parity;
        a.counters_next = d->d_counters + COUNTER_SET_WORDS * (d->call_parity ^ 1u);
        d->call_parity ^= 1u;
    }
    a.work = noalloc ? (uint4 *)(scr + scr_work) : d->d_work;
    a.host_status = d->h_status + 8 * slot;
    HIP_TRY(next_call_number(d, stream));
    a.seq = d->call_seq;
    a.overflow_list = noalloc ? (uint4 *)(scr + scr_ovf) : d->d_overflow;
    a.overflow_cap = (uint32_t)(noalloc ? scr_ovf_cap : d->overflow_cap);
    a.fb_items = noalloc ? (uint2 *)(scr + scr_fb) : d->d_fb_items;
    a.fb_set_start = noalloc ? (uint32_t *)(scr + scr_ss) : d->d_fb_ss;
    a.fb_waves = noalloc ? NOALLOC_FB_WAVES : FB_WAVES;
    a.fb_stride = noalloc ? NOALLOC_FB_ITEMS_PER_WAVE : FB_ITEMS_PER_WAVE;
    a.batch = nb;
    // Item budget of a walking wavefront: the configured one, raised for this call when the rows'
    // current sets are large (ambiguous grammars) so that such rows do not all end in the fallback.
    a.lane_cap = e->opt.lane_item_cap;
    if (e->lane_cap_auto) {
        size_t widest = 0;
        for (int r = 0; r < nb; r++) {
            const Chart &c = chart_of(states[miss_rows[r]]);
            widest = std::max<size_t>(widest, c.set_off[c.n_sets()] - c.set_off[c.n_sets() - 1]);
        }
        size_t want_cap = (8 * widest + 64 + 31) / 32 * 32;
        while (want_cap > (size_t)a.lane_cap && walk_lds_bytes(d->tab, d->mode, (int)std::min<size_t>(want_cap, LANE_CAP_MAX)) > 160u * 1024u) want_cap -= 32;
        if (want_cap > (size_t)a.lane_cap) a.lane_cap = (int)std::min<size_t>(want_cap, LANE_CAP_MAX);
    }
    {   // the persistent walk grid: as many blocks as the chip holds at once (LDS is the limit)
        const uint32_t lds = walk_lds_bytes(d->tab, d->mode, a.lane_cap);
        if (lds != d->occ_lds) {                          // ask the runtime once per LDS size
            HIP_TRY(walk_blocks_per_cu(d->mode, lds, &d->occ_blocks));
            d->occ_lds = lds;
        }
        // half as many blocks again as the chip holds at once: the surplus blocks take the places of
        // blocks whose share of the queue was light (measured: exactly-resident grids are ~10 % slower,
        // larger surpluses bring nothing more)
        a.walk_blocks = std::max(1, d->cus) * d->occ_blocks * 3 / 2;
    }
    a.fb_cap = (int32_t)std::min<uint32_t>((uint32_t)e->opt.fallback_item_cap, a.fb_stride);
    a.mode = d->mode;
    const bool automaton = e->opt.walk_mode != 1;
    if (automaton) {
        // LDS budgets of one block's automaton.  The set under construction gets the configured item
        // budget (tests set it tiny to force the fallback pass), else room for sets a few times as wide
        // as the widest current set; states and the item arena share what the tables leave of 160 KB.
        size_t widest = 0, most_sets = 0, most_items = 0, biggest_set = 0;
        for (int r = 0; r < nb; r++) {
            const Chart &c = chart_of(states[miss_rows[r]]);
            widest = std::max<size_t>(widest, c.set_off[c.n_sets()] - c.set_off[c.n_sets() - 1]);
            most_sets = std::max<size_t>(most_sets, c.n_sets());
            most_items = std::max<size_t>(most_items, c.set_off[c.n_sets()]);
            for (uint32_t k = 0; k < c.n_sets(); k++) biggest_set = std::max<size_t>(biggest_set, c.set_off[k + 1] - c.set_off[k]);
        }
        int scratch = 0, n_states = 0, arena = 0, base_sets = 0, base_items = 0, waves = nb <= d->cus ? AUT_WAVES : AUT_WAVES_MANY_ROWS;
        // The build without the wide byte step also takes the chart from LDS only (its pointers are then
        // known to be LDS addresses): it serves calls whose sets are all small and whose charts all fit.
        // AUT_STEP_LANES holds sets of 64 items, which a byte or a long token can take a dozen items beyond: the strings behind such a set
        // then cost the fallback pass more than the build saves (7 %), and the short list of a call that allocates nothing
        // might not hold them.  So that call never takes the build, and an engine whose strings have outgrown it once takes the wide one.
        // Where every operand completes all operations before it, the sets of the strings outgrow a narrow step's, however small the charts' are.
        const bool lanes = !noalloc && !d->lanes_outgrown;
        int step = biggest_set <= (size_t)AUT_NARROW_SET_MAX ? (e->tab.operators && lanes ? AUT_STEP_LANES : AUT_STEP_NARROW)
                 : biggest_set <= (size_t)AUT_LANES_SET_MAX && lanes ? AUT_STEP_LANES : AUT_STEP_WIDE;
        const uint32_t lds_max = 160u * 1024u;
        for (;;) {
            scratch = e->lane_cap_auto ? (int)std::min<size_t>(LANE_CAP_MAX, (4 * widest + 128 + 31) / 32 * 32) : e->opt.lane_item_cap;
            auto room_for = [&](int n) { n_states = n; arena = std::max(AUT_ARENA_PER_STATE * n, 8 * scratch); };
            room_for(AUT_STATES_DEFAULT);
            base_sets = BASE_SETS_LDS; base_items = BASE_ITEMS_LDS;
            auto lds_now = [&]() { return automaton_lds_bytes(d->tab, d->mode, n_states, arena, scratch, base_sets, base_items, step == AUT_STEP_WIDE, waves); };
            if (lds_now() > lds_max) waves = AUT_WAVES_MANY_ROWS;
            if (waves == AUT_WAVES_MANY_ROWS && lds_now() > lds_max / 2) room_for(AUT_STATES_TIGHT);
            while (lds_now() > lds_max && arena > 2 * scratch) arena /= 2;
            while (lds_now() > lds_max && n_states > 8) n_states /= 2;
            while (lds_now() > lds_max && scratch > 32) { scratch /= 2; arena = std::max(arena / 2, 2 * scratch); }
            if (lds_now() > lds_max) return fail(ZF_ERR_INVALID_ARG, "the grammar tables leave no LDS for the mask automaton");
            // the rows' charts are read over and over by Complete: keep them in LDS too when the longest one fits in what is left
            if (most_sets > (size_t)BASE_SETS_LDS || most_items > (size_t)BASE_ITEMS_LDS) {
                const int want_sets = (int)std::max<size_t>(BASE_SETS_LDS, (most_sets + 32) / 32 * 32 - 1);
                const int want_items = (int)std::max<size_t>(BASE_ITEMS_LDS, (most_items + 63) / 64 * 64);
                if (want_sets <= AUT_BASE_SETS_MAX && want_items <= AUT_BASE_ITEMS_MAX &&
                    automaton_lds_bytes(d->tab, d->mode, n_states, arena, scratch, want_sets, want_items, step == AUT_STEP_WIDE, waves) <= lds_max) {
                    base_sets = want_sets; base_items = want_items;
                }
            }
            const bool chart_fits = most_sets <= (size_t)base_sets && most_items <= (size_t)base_items;
            if (!chart_fits && waves == AUT_WAVES) { waves = AUT_WAVES_MANY_ROWS; continue; }   // smaller blocks leave more of it
            if (step == AUT_STEP_WIDE || chart_fits) break;
            step = AUT_STEP_WIDE;                         // some chart stays in global memory: the other build
        }
        a.aut_states = n_states; a.aut_arena = arena; a.aut_scratch = scratch;
        a.aut_base_sets = base_sets; a.aut_base_items = base_items;
        a.aut_step = step; a.aut_waves = waves;
        d->lanes_call[slot] = step == AUT_STEP_LANES;
        // blocks per row: as many as the chip holds at once -- of 16 wavefronts one per compute unit, of 8 at most two --, at most one per AUT_PART_WORDS words.
        // (Every block works its row's automaton out from the start: a second round of blocks, where the wide byte step's scratch
        // leaves room for one block per compute unit, took as long as the first.)
        const int n_sub = (d->tab.Wr + AUT_PART_WORDS - 1) / AUT_PART_WORDS, most = waves == AUT_WAVES ? 1 : 2;
        const int resident = std::min(most, automaton_blocks_per_cu(a)) * std::max(1, d->cus);
        a.aut_parts = std::max(1, std::min(n_sub, resident == 2 * d->cus ? (resident + std::max(nb, 1) - 1) / std::max(nb, 1) : resident / std::max(nb, 1)));
    }
    const bool prof = d->profiling;
    d->report.chart_bytes = (int64_t)total;
    d->report.cache_rows = (int32_t)n_cache_rows;
    d->report.main_ms = d->report.fallback_ms = d->report.permute_ms = 0.f;
    d->report.overflow_chunks = d->report.walk_chunks = d->report.parser_steps = 0;
    // everything the host has to work out is done: enqueue the upload and the kernels back to back
    if (noalloc) HIP_TRY(launch_clear_words((uint32_t *)scr, 2 * COUNTER_SET_WORDS, stream));   // the array keeps the last call's counters
    if (!direct) HIP_TRY(launch_upload(d->h_stage[slot], chart_base, total, stream));
    const bool run_kernels = nb > 0;
    if (run_kernels && d->tab.n_chunks > 0 && !automaton) HIP_TRY(launch_cache_merge(a, stream));
    if (prof) HIP_TRY(hipEventRecord(d->ev[0], stream));
    if (run_kernels && d->tab.n_chunks > 0) HIP_TRY(automaton ? launch_mask_automaton(a, stream) : launch_mask_walk(a, stream));
    if (prof) HIP_TRY(hipEventRecord(d->ev[1], stream));
    d->closing_kernel = true;
    if (g_apply.out && !a.dst_row && run_kernels) {       // the closing kernel of all of the caller's rows, in their order, masks their logits along
        const size_t esz = g_apply.dtype == 0 ? 4 : 2;
        if ((uintptr_t)g_apply.logits % esz == 0 && (uintptr_t)g_apply.out % esz == 0) {
            a.logits = g_apply.logits; a.logits_out = g_apply.out; a.logit_stride = g_apply.stride; a.logit_dtype = g_apply.dtype + 1;
            g_apply.fused = true;
        }
    }
    if (run_kernels) HIP_TRY(launch_finish(a, d->cus, stream));   // fallback pass (if anything was listed) + permutation; also hands the counters to the host and clears the next call's
    if (sc) HIP_TRY(launch_gather(a, stream));            // every row's finished mask from its pool slot to the caller's tensor
    if (prof) HIP_TRY(hipEventRecord(d->ev[3], stream));
    d->next_slot = (slot + 1) % DeviceSide::N_SLOTS;
    d->pending++;
    d->last_seq = a.seq; d->last_slot = slot;
    d->closing_open = !wait;
    if (!wait) {
        // (without the fences that show memory to the host and other devices: what waits for it only has to come later, on this device)
        if (!d->closing_done) HIP_TRY(hipEventCreateWithFlags(&d->closing_done, hipEventDisableTiming | hipEventDisableSystemFence));
        HIP_TRY(hipEventRecord(d->closing_done, stream));
        d->closing_stream = stream;
        return ZF_OK;
    }
    HIP_TRY(hipStreamSynchronize(stream));               // the waiting call returns with the mask complete, not only its status known
    return wait_for_calls(e, hip_stream);
}

static void forget_cached_masks(DeviceSide *d) {
    d->cache_index.clear();
    for (auto &ce : d->cache) ce.used = false;
    d->slot_of_host.clear();
    std::fill(d->host_of_slot.begin(), d->host_of_slot.end(), 0u);
}

// ---- the same call through the persistent automaton (walk_mode 2) ----
// Rows that stand in the same state -- the host automaton's name says so -- have the same mask: they form a group, which the
// kernel works out once and stores to all of them (the rows of a batch are queries under one grammar, most of them inside a
// string, a number or an identifier: 256 rows of a JSON schema stand in about 20 states).  What a group sends is the name of
// the state on the device and nothing else when the device has reported it before; else the state its rows were last known
// to be in and the byte classes fed since, which the kernel walks, reporting the state it arrives at (pinned memory), which
// zf_mask_wait notes in the rows' zf_states.  States the store does not know -- after it was cleared, or too far behind --
// bring a packed chart along and are made states of by the import kernel first.

// The state's name in the host automaton, when it has a current one there (the caller holds the host automaton's lock) ...
static bool host_name_valid(const zf_engine *e, const zf_state *st) {
    return e->host_aut && st->host_id != HostAutomaton::ROOT && st->host_id_epoch == e->host_epoch && st->host_id < HostAutomaton::SINK && st->host_id != 0;
}
// ... and the device's name of that state, 0 when the device has not reported one
static uint32_t device_name_of(const zf_engine *e, const zf_state *st) {
    return host_name_valid(e, st) ? e->dev->name_find(st->host_id, e->host_epoch, e->dev->store_epoch) : 0u;
}
static bool device_knows(const DeviceSide *d, const zf_state *st) { return st->dev_id == STORE_ROOT_ID || (st->dev_id != 0 && st->dev_epoch == d->store_epoch); }
// The row stands in device state `dev`, everything fed so far included.
static void note_device_state(const DeviceSide *d, zf_state *st, uint32_t dev) {
    st->dev_id = dev; st->dev_epoch = d->store_epoch;
    st->pending.clear(); st->pending_base = st->fed_total; st->pending_token = -1;
}

// Tokens that a list of token-mask cache rows leaves to the parser.
static uint64_t entries_signature(const uint32_t *ent, uint32_t n) {
    uint64_t sig = 0xCBF29CE484222325ull ^ n;
    for (uint32_t k = 0; k < n; k++) sig = (sig ^ ent[k]) * 0x100000001B3ull;
    return sig;
}
static int64_t count_undecided(DeviceSide *d, const uint32_t *ent, uint32_t n) {
    if (n == 1) return d->ci_undecided[ent[0]];
    const uint64_t sig = entries_signature(ent, n);
    auto it = d->undecided_of.find(sig);
    if (it == d->undecided_of.end()) {
        if (d->undecided_of.size() > 65536) d->undecided_of.clear();
        it = d->undecided_of.emplace(sig, undecided_tokens(d->h_ci_tok, (size_t)d->tab.W, ent, n)).first;
    }
    return it->second;
}

namespace {
struct RowGroup {
    zf_state *lead;                // the row whose knowledge the group sends
    uint32_t at;                   // name in the host automaton (0: none, the row is a group of its own)
    uint32_t dev;                  // name on the device (0: the kernel walks the lead's pending bytes, or imports its chart)
    int32_t last, n;               // rows: the last one (a chain through next_row), how many
    const Item *items; uint32_t n_items;
    const uint32_t *ents; uint32_t n_ent;
    double undecided;
    uint32_t slot;                 // row of the state cache's pool
    uint8_t pooled, keep, known, decided, alone;   // decided: its cache rows, all in a record, leave nothing undecided; alone: the wavefronts with logits do all there is to do
    int32_t seg_w, parts;          // launch shape
};
struct StoreCall {                 // one call's working memory, kept per thread
    std::vector<RowGroup> g;
    std::vector<int32_t> next_row; // chain of the rows of a group
    std::vector<uint32_t> table;   // open addressing: host name -> group + 1
    std::vector<uint32_t> ents_at; // entries of groups outside the host automaton
    std::vector<uint32_t> spare_ents;
    std::vector<zf_state *> unknown;
    std::vector<uint32_t> imports; // groups that bring their charts along
    std::vector<std::vector<uint32_t>> packed;
    StoreInline in;
    LookInline look;
};
}  // namespace

// Launch shape: mask words a wavefront takes per pass and blocks, per group; returns the blocks of the grid.  A wavefront takes a
// group's mask words in segments and the undecided tokens among them 64 at a time; groups differ by orders of magnitude in how
// many tokens their token-mask cache rows leave undecided, which was counted once per list of cache rows.  The grid is never
// larger than what the chip holds at once: a block that had to wait for a place would start from nothing (LDS cache, the
// group's state) when the others are nearly done, which costs more than a few more passes of the wavefronts that are there.
static int store_launch_shape(std::vector<RowGroup> &g, int W, int V, int budget, int logit_bytes, int member_words) {
    const int n = (int)g.size();
    static thread_local std::vector<double> inv_cost;
    static thread_local std::vector<int> segs, passes;
    inv_cost.resize(n); segs.resize(n); passes.resize(n);
    double lo = 1e30;
    const double apply_us_per_word = 0.25 * 32 * logit_bytes * 2 / 1024;
    for (int r = 0; r < n; r++) {
        // words per segment: as many as are expected to hold 40 undecided tokens, at most 64 (a batch is 64: the
        // tokens are spread unevenly, and a second, nearly empty batch costs as much as a full one)
        const double und = g[r].undecided;
        int sw = g[r].pooled ? 16 : (int)std::max(1.0, std::min<double>(STORE_SEG_WORDS_MAX, 40.0 * std::max(1, V) / (32.0 * std::max(und, 1.0))));
        // where the logits are masked too: no more words than the logits a wavefront requests ahead for all rows of the group
        // (two pieces of 16 bytes per lane), so that nothing is waited for at the end while there are wavefronts to spare
        if (logit_bytes) sw = std::min(sw, std::max(1, STORE_AHEAD_BYTES / (32 * logit_bytes * g[r].n)));
        // nor, in a call of look-ups, more words than its wavefront stores to all its rows in a few stores (256 rows x 128,256 in some 20 states, 8 waiting calls: 241 -> 213 us;
        // 64 rows of the query language, 16 calls: 274 -> 258; with half as many words 216 and 254).  First visits, all of whose rows stand in a state or two, have no
        // wavefronts to spare for that: 256 x 128,256 of the schema 56.5 us a step, 65 so.
        if (member_words) sw = std::min(sw, std::max(1, member_words / g[r].n));
        else if (g[r].alone) sw = W;                      // (nothing to do: a block that reports)
        segs[r] = std::max(1, (W + sw - 1) / sw);
        g[r].seg_w = sw;
        // what a pass costs a wavefront (microseconds, measured): an empty segment 2.8, a segment with a batch 3.7, each further
        // batch 3; storing and masking a member's share of it on top
        const double per_seg = und / segs[r];
        const double walk = g[r].pooled ? 1.5 : (per_seg < 1.0 ? 2.8 + 0.9 * per_seg : 3.7 + 3.0 * std::max(0.0, per_seg / 64.0 - 0.75));
        const double cost = walk + g[r].n * (0.03 + apply_us_per_word * sw);
        inv_cost[r] = 1.0 / cost;
        lo = std::min(lo, cost);
    }
    // Every wavefront of a group takes the same number of passes (a group is as slow as its slowest wavefront).  The
    // smallest time T is looked for in which every group, taking as many passes as fit into T, leaves the grid within
    // what the chip holds; groups are then given passes back while blocks are left.
    auto blocks_for = [&](int r, int n_pass) { return std::max(1, (segs[r] + n_pass * STORE_WAVES - 1) / (n_pass * STORE_WAVES)); };
    auto need = [&](double T) {
        int tot = 0;
        for (int r = 0; r < n; r++) tot += blocks_for(r, std::max(1, (int)(T * inv_cost[r])));
        return tot;
    };
    double hi = lo;
    if (need(hi) > budget) {
        while (need(hi) > budget && hi < 1e9) { lo = hi; hi *= 2; }
        for (int it = 0; it < 6; it++) { const double mid = 0.5 * (lo + hi); if (need(mid) <= budget) hi = mid; else lo = mid; }   // to 2 %: the blocks left over go back to the groups below
    }
    int all = 0;
    for (int r = 0; r < n; r++) { passes[r] = std::max(1, (int)(hi * inv_cost[r])); g[r].parts = blocks_for(r, passes[r]); all += g[r].parts; }
    for (int r = 0; r < n && all < budget; r++) {
        if (passes[r] <= 1) continue;
        const int p = blocks_for(r, passes[r] - 1);
        if (p - g[r].parts <= budget - all) { all += p - g[r].parts; g[r].parts = p; passes[r]--; }
    }
    // Blocks are dealt to the eight XCDs in turn, and every XCD has an L2 of its own.  When groups start at multiples of eight,
    // the blocks that take the same stretch of the vocabulary for different groups run on the same XCD and find each other's
    // strings and cache rows in its L2.  So groups of eight blocks or more are rounded UP to a multiple of eight while blocks are
    // left over (never down: fewer blocks would mean more passes); a block beyond the group's segments leaves at once.
    for (int r = 0; r < n; r++) {
        const int up = (8 - (g[r].parts & 7)) & 7;
        if (g[r].parts >= 8 && up && all + up <= budget) { g[r].parts += up; all += up; }
    }
    for (int r = 0; r < n; r++) {
        // A wavefront that has several segments to take takes them as fewer, wider ones (up to 64 words): the strings of a
        // segment's first batch are waited for, those of its further batches travel while the batch before is checked.
        if (passes[r] > 1 && g[r].seg_w < STORE_SEG_WORDS_MAX) {
            const int words_per_wave = (W + g[r].parts * STORE_WAVES - 1) / (g[r].parts * STORE_WAVES);
            const int n_pass = (words_per_wave + STORE_SEG_WORDS_MAX - 1) / STORE_SEG_WORDS_MAX;
            g[r].seg_w = std::max(g[r].seg_w, std::min<int>(STORE_SEG_WORDS_MAX, (words_per_wave + n_pass - 1) / n_pass));
        }
    }
    return all;
}

// A call of look-ups only, whose groups are in c.g: its shape, its records and its launch.  n_more: cache rows that the groups' records do not hold.
static int enqueue_look(zf_engine *e, StoreCall &c, zf_state *const *states, int32_t batch, uint32_t *d_mask, hipStream_t stream, bool wait, bool noalloc, uint32_t slot,
                        size_t n_more, uint32_t n_cache_rows, std::unique_lock<std::mutex> &host_lk) {
    DeviceSide *d = e->dev;
    DeviceSide::CallRecord &rec = d->rec[slot];
    const int ng = (int)c.g.size();
    const bool use_cache = !e->opt.disable_token_mask_cache;
    const size_t n_members = (size_t)batch + n_more;      // behind the members: the cache rows that the records do not hold
    const bool big = ng > STORE_INLINE_GROUPS;            // records and members travel in device memory instead of the argument block
    auto align16 = [](size_t x) { return (x + 15) & ~(size_t)15; };
    // staging: [group records][blocks][members][groups of the members] (uploaded when big)
    const int max_blocks = std::max(ng, STORE_BLOCKS_PER_CU * std::max(1, d->cus)) + 8 * ng;
    const size_t off_block = align16(big ? sizeof(LookGroup) * ng : 0), off_mem = align16(off_block + (big ? 8 * (size_t)max_blocks : 0));
    const size_t off_gof = align16(off_mem + 2 * n_members), up_bytes = align16(off_gof + (big && g_apply.out ? 2 * (size_t)batch : 0)), total = up_bytes + 16;
    if (noalloc && (total > d->stage_cap[slot] || (big && up_bytes > NOALLOC_SCRATCH_BYTES))) return STORE_NO_ROOM;
    if (total > d->stage_cap[slot]) {
        const int rc = grow_stage(d, slot, total * 2 + 4096);
        if (rc != ZF_OK) return rc;
    }
    if (big && !noalloc && up_bytes > d->chart_cap) {
        HIP_TRY(hipStreamSynchronize(stream));
        if (d->d_chart) (void)hipFree(d->d_chart);
        d->d_chart = nullptr; d->chart_cap = 0;
        const size_t cap = up_bytes * 2 + 4096;
        HIP_TRY(hipMalloc(&d->d_chart, cap));
        d->chart_cap = cap;
    }
    LookArgs k{};
    const size_t esz = g_apply.dtype == 0 ? 4 : 2;
    const bool whole = g_apply.out && (uintptr_t)g_apply.logits % esz == 0 && (uintptr_t)g_apply.out % esz == 0;
    // mask_look_kernel masks the logits with wavefronts of their own, whatever their size: they read them while the others work the masks out.  The
    // logits are dealt out in units of as many KB as make 2,048 wavefronts, 4 at most (units of 2 / 4 / 6 / 8 KB, us per pass: 16 steps of 16 x 128,256
    // bf16 171 / 176 / 184 / 186, of 64 x 152,064 fp32 - / 361 / 371 / 379, 8 steps of 130 x 40,037 bf16 148 / 144 / 149 / 151; 256 x 128,256 - / 235 / 229 / 239).
    const uint32_t row_kb = (uint32_t)(((uint64_t)e->V * esz + 1023) / 1024);
    const uint64_t kb = (uint64_t)row_kb * (uint64_t)batch;
    const uint32_t unit_kb = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(LOOK_UNIT_KB, (kb + 2047) / 2048)), row_units = (row_kb + unit_kb - 1) / unit_kb;
    if (whole && e->V > 0 && (uint64_t)batch * (uint64_t)e->V < (1ull << 32) && (uint64_t)row_units * (uint64_t)batch <= LOOK_UNITS_MAX) {
        static_assert(LOOK_UNITS_MAX / STORE_WAVES + 9 * MAX_BATCH + 4096 <= 16 * 65535, "with the mask's (max_blocks) the blocks of a group fit their count");
        k.unit_kb = unit_kb;
        k.row_units = row_units;
        k.units = k.row_units * (uint32_t)batch;
        const size_t words = (size_t)ng * (size_t)d->tab.W + (k.units + STORE_WAVES - 1) / STORE_WAVES;
        if (words > d->tagged_cap) {
            const int rc = settle_calls(d);
            if (rc != ZF_OK) return rc;
            HIP_TRY(hipStreamSynchronize(stream));
            if (d->d_tagged) (void)hipFree(d->d_tagged);
            d->d_tagged = nullptr; d->tagged_cap = 0;
            const size_t cap = std::max(words * 2, (size_t)STORE_INLINE_GROUPS * (size_t)d->tab.W);
            HIP_TRY(hipMalloc((void **)&d->d_tagged, cap * 8));
            d->tagged_cap = cap;
            HIP_TRY(launch_clear_words((uint32_t *)d->d_tagged, (uint32_t)(cap * 2), stream));
        }
        k.polls = d->look_polls;
        k.tagged = d->d_tagged; k.logits = g_apply.logits; k.out = g_apply.out; k.stride = g_apply.stride; k.dtype = (uint32_t)g_apply.dtype + 1;
        g_apply.fused = true;
    }
    for (RowGroup &g : c.g) {
        g.decided = use_cache && !g.pooled && g.undecided == 0 && g.n_ent <= (uint32_t)STORE_GROUP_ENT;
        // Where the wavefronts with logits make a group's mask they may as well store it, and no others work it out: 16 steps of 64 x 128,256 bf16 of the query language 161 -> 150 us
        // (from four rows a group on 160), 8 of 130 x 40,037 103.1 -> 102.3.  Not with fp32, whose units hold half as many words: 16 of 64 x 152,064 288 -> 294, a step of 256 x 128,256
        // of the expression grammar 52.1 -> 53.7, of the query language 43.3 -> 43.0; 16 rows and 1,000 x 32,000 the same either way.
        g.alone = k.units && g.decided && !g.keep && k.dtype == 2;
    }
    const int budget = std::max(ng, look_blocks_per_cu() * std::max(1, d->cus));
    k.mask_blocks = (uint32_t)store_launch_shape(c.g, d->tab.W, e->V, budget, 0, k.units ? 0 : LOOK_MEMBER_WORDS);
    // ---- the records ----
    {
        uint8_t *h = (uint8_t *)d->h_stage[slot];
        LookGroup *gr = big ? (LookGroup *)h : c.look.g;
        uint32_t *blk = (uint32_t *)(h + off_block);
        const bool members_apart = big || n_members > (size_t)STORE_INLINE_ROWS;
        uint16_t *mem = members_apart ? (uint16_t *)(h + off_mem) : c.look.member, *gof = (uint16_t *)(h + off_gof);
        uint32_t mem_at = 0, blk_at = 0, more_at = (uint32_t)batch;
        for (int r = 0; r < ng; r++) {
            const RowGroup &g = c.g[r];
            LookGroup &m = gr[r];
            const uint32_t flags = g.pooled ? STORE_ROW_POOLED : (use_cache ? STORE_ROW_CACHE : 0u) | (g.keep ? STORE_ROW_KEEP : 0u) | (g.decided ? STORE_ROW_DECIDED : 0u);
            m.w[0] = g.pooled ? g.slot : g.dev;
            m.w[1] = g.n_ent | flags << 8 | (g.alone ? 0u : (uint32_t)(g.seg_w - 1) << 16);
            m.w[2] = (blk_at & 0xFFFFu) | (g.alone ? 0u : (uint32_t)((d->tab.W + g.seg_w - 1) / g.seg_w) << 16);
            m.w[3] = mem_at | (uint32_t)g.n << 16;
            m.w[4] = g.slot & 0xFFFFu;
            for (int j = 5; j < LOOK_WORDS; j++) m.w[j] = 0;
            const uint32_t n_here = g.n_ent > (uint32_t)STORE_GROUP_ENT ? LOOK_ENT_OF_MORE : g.n_ent;
            for (uint32_t j = 0; j < n_here; j++) m.w[4 + ((j + 1) >> 1)] |= g.ents[j] << (((j + 1) & 1u) * 16u);
            if (n_here < g.n_ent) {
                m.w[4 + ((n_here + 1) >> 1)] |= more_at << (((n_here + 1) & 1u) * 16u);
                for (uint32_t j = n_here; j < g.n_ent; j++) mem[more_at++] = (uint16_t)g.ents[j];
            }
            for (int32_t b = g.last; b >= 0; b = c.next_row[b]) {
                if (big && k.units) gof[mem_at] = (uint16_t)r;
                mem[mem_at++] = (uint16_t)b;
                if (g.dev) note_device_state(d, states[b], g.dev);
            }
            if (big) for (int p = 0; p < g.parts; p++) { blk[2 * blk_at] = (uint32_t)r; blk[2 * blk_at + 1] = (uint32_t)p | (uint32_t)g.parts << 16; blk_at++; }
            else blk_at += (uint32_t)g.parts;
        }
        const uint8_t *up = noalloc ? d->scratch : (const uint8_t *)d->d_chart;
        k.trans = e->store_on ? d->store.trans : d->no_trans; k.cache = d->tab.ci_tok; k.tok16 = d->tab.tok16; k.out_mask = d_mask; k.pool = d->d_pool;
        k.konst = d->d_konst;
        if (big) { k.groups = (const LookGroup *)up; k.block_of = (const uint32_t *)(up + off_block); k.members = (const uint16_t *)(up + off_mem); k.group_of = (const uint16_t *)(up + off_gof); }
        else if (members_apart) k.members = (const uint16_t *)(h + off_mem);
        k.V = (uint32_t)e->V; k.W = (uint32_t)d->tab.W; k.ncls = (uint32_t)d->tab.n_cls; k.n_groups = (uint32_t)ng;
    }
    k.tickets = d->d_tickets + d->ticket_set * STORE_TICKETS; k.tickets_next = d->d_tickets + (d->ticket_set ^ 1u) * STORE_TICKETS;
    k.status = (unsigned long long *)d->h_store_status + slot * STORE_STATUS_WORDS;
    HIP_TRY(next_call_number(d, stream));
    k.seq = rec.seq = d->call_seq;
    k.complete = wait ? 1 : 0;
    const bool prof = d->profiling;
    d->report.chart_bytes = (int64_t)(total + (big ? 0 : sizeof(LookGroup) * ng));
    d->report.cache_rows = (int32_t)n_cache_rows;
    d->report.main_ms = d->report.fallback_ms = d->report.permute_ms = 0.f;
    d->report.overflow_chunks = d->report.walk_chunks = d->report.parser_steps = 0;
    if (big) HIP_TRY(launch_upload(d->h_stage[slot], noalloc ? d->scratch : (uint8_t *)d->d_chart, up_bytes, stream));
    if (prof) HIP_TRY(hipEventRecord(d->ev[0], stream));
    d->closing_kernel = false;
    rec.debug_failed = d->debug_failed; d->debug_failed = 0;
    const uint32_t grid = look_grid(k);
    // Up to 64 blocks each have a status word of their own, and nobody draws a ticket (one row x 32,000 223 -> 214 us per 32 steps); more share 16 (16 x 128,256, eight waiting calls: 139; with 64 words to look at 143, in two levels 139).
    k.done_groups = rec.done_groups = grid <= (uint32_t)STORE_TICKET_GROUPS ? grid : 16u;
    HIP_TRY(launch_mask_look(k, c.look, stream));
    d->ticket_set ^= 1u;
    if (prof) { HIP_TRY(hipEventRecord(d->ev[1], stream)); HIP_TRY(hipEventRecord(d->ev[3], stream)); }
    d->next_slot = (slot + 1) % DeviceSide::N_SLOTS;
    d->pending++;
    d->last_seq = k.seq; d->last_slot = slot;
    rec.active = true;
    // Nothing in the call is expected to fail: its states' transitions are in the table for certain, no call in flight is still to say so.  zf_mask_wait
    // then has nothing to wait for, and the host gets the next step ready while this one is at work (a step of one row x 32,000: 13.6 us
    // waited for, 10.1 not; 16 x 128,256 bf16 14.4 and 12.3; 130 x 40,037 bf16 26.1 and 21.6).
    // (Not one that leaves rows in the state cache's pool: later calls are served those.)
    rec.sure = !wait && !prof && !(e->store_on && d->store_dirty);
    for (const RowGroup &g : c.g) rec.sure &= g.pooled || !g.keep;
    uint32_t in_store = 0;                                // calls in flight that went through the store; the others have flags that zf_mask_wait has to await
    for (const DeviceSide::CallRecord &other : d->rec) if (other.active) { in_store++; if (!other.sure) rec.sure &= &other == &rec; }
    rec.sure &= in_store == d->pending;
    if (rec.sure) d->lazy_stream = stream;
    host_lk.unlock();
    // the waiting call returns with the mask complete: the kernel wrote it through to memory before it drew its tickets
    return wait ? wait_for_calls(e, (void *)stream) : ZF_OK;
}

// An engine without a persistent automaton (pruning off): a call all of whose rows select token-mask cache rows that leave no token to the parser is one of look-ups
// too, without any to make.  Rows with the same list are a group.  STORE_NO_ROOM: some row leaves something, or does not fit a record; nothing was enqueued.
// (64 rows x 152,064 of the expression grammar, 8 steps: 262 us through the per-block automaton and its closing kernel, 144 so.  A call of which the last row alone is
// undecided is enqueued as fast as without the look: 6.6 us of 16 rows, 17.8 of 256.  Calls with a state cache or
// without allocations keep to the per-block automaton: it is what knows the one, and fits the static array.)
static int enqueue_decided(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, hipStream_t stream, bool wait, uint32_t slot) {
    DeviceSide *d = e->dev;
    static thread_local StoreCall c;
    std::unique_lock<std::mutex> host_lk(e->host_mu);
    c.g.clear(); c.spare_ents.clear(); c.next_row.resize(batch);
    static thread_local std::unordered_multimap<uint64_t, uint32_t> by_list;
    static thread_local std::vector<size_t> at_of;        // of each group: where its list begins
    by_list.clear(); at_of.clear();
    size_t n_more = 0;
    uint32_t n_cache_rows = 0;
    for (int32_t b = 0; b < batch; b++) {
        const Chart &ch = chart_of(states[b]);
        const uint32_t lo = ch.set_off[ch.n_sets() - 1], n_items = ch.set_off[ch.n_sets()] - lo;
        const size_t at = c.spare_ents.size();
        c.spare_ents.resize(at + n_items);
        const uint32_t n = current_set_entries(e->tab, ch.items.data() + lo, n_items, c.spare_ents.data() + at);
        const uint32_t *ents = c.spare_ents.data() + at;
        if (n > LOOK_ENT_MAX) return STORE_NO_ROOM;
        for (uint32_t k = 0; k < n; k++) if (ents[k] >= 65536u || d->ci_undecided[ents[k]] != 0) return STORE_NO_ROOM;
        const uint64_t sig = entries_signature(ents, n);
        c.next_row[b] = -1;
        RowGroup *g = nullptr;
        for (auto range = by_list.equal_range(sig); range.first != range.second && !g; ++range.first) {
            RowGroup &x = c.g[range.first->second];
            if (x.n_ent == n && std::equal(ents, ents + n, c.spare_ents.data() + at_of[range.first->second])) g = &x;
        }
        if (g) {
            c.next_row[b] = g->last; g->last = b; g->n++;
            c.spare_ents.resize(at);
            continue;
        }
        c.spare_ents.resize(at + n);
        RowGroup x{};
        x.lead = states[b]; x.last = b; x.n = 1; x.n_ent = n;
        if (n > (uint32_t)STORE_GROUP_ENT) n_more += n - LOOK_ENT_OF_MORE;
        n_cache_rows += n;
        by_list.emplace(sig, (uint32_t)c.g.size());
        c.g.push_back(x); at_of.push_back(at);
    }
    if (d->tab.W > 65535 || (size_t)batch + n_more > 65535) return STORE_NO_ROOM;
    for (size_t r = 0; r < c.g.size(); r++) c.g[r].ents = c.spare_ents.data() + at_of[r];
    d->report.cache_hits = 0; d->report.cache_misses = 0;
    DeviceSide::CallRecord &rec = d->rec[slot];
    rec.epoch = d->store_epoch; rec.host_epoch = e->host_epoch;
    rec.groups.clear(); rec.rows.clear(); rec.undecided = 0;
    return enqueue_look(e, c, states, batch, d_mask, stream, wait, false, slot, n_more, n_cache_rows, host_lk);
}

static int enqueue_store_impl(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, void *hip_stream, bool wait, bool noalloc, uint32_t slot) {
    DeviceSide *d = e->dev;
    HostAutomaton &A = *e->host_aut;
    hipStream_t stream = (hipStream_t)hip_stream;
    static thread_local StoreCall c;
    std::unique_lock<std::mutex> host_lk(e->host_mu);     // the rows' states are read from the host automaton (a row it does not know is brought in)
    // ---- clear the store when it is new, half full, or has refused a request; only with no call in flight ----
    if (d->pending == 0 && (d->store_dirty || d->store_states > d->store.cap_states / 2 || d->store_items > d->store.cap_items / 2)) {
        HIP_TRY(launch_store_clear(d->store, (uint32_t)std::max(e->tab.n_cls, 1), d->d_root_items, d->n_root, stream));
        d->store_epoch++;
        d->store_states = 2; d->store_items = d->n_root;
        d->store_dirty = false;
    }
    if (d->hop_epoch != d->store_epoch) { if (d->hop_used) std::fill(d->hop_key.begin(), d->hop_key.end(), 0); d->hop_used = 0; d->hop_epoch = d->store_epoch; }
    // ---- group the rows by the state they stand in ----
    c.g.clear(); c.spare_ents.clear(); c.imports.clear(); c.unknown.clear();
    for (int32_t b = 0; b < batch; b++) {                 // rows the host automaton has to take in from their charts (all of them after it was emptied)
        zf_state *st = states[b];
        if (st->host_id != HostAutomaton::ROOT && st->host_id_epoch != e->host_epoch && !st->lag.empty()) c.unknown.push_back(st);
    }
    if (!c.unknown.empty()) catch_up_batch(c.unknown.data(), (int32_t)c.unknown.size());
    c.next_row.resize(batch);
    uint32_t places = 64;
    while (places < 2u * (uint32_t)batch) places <<= 1;
    c.table.assign(places, 0);
    for (int32_t b = 0; b < batch; b++) {
        zf_state *st = states[b];
        const uint32_t at = host_place(st);
        c.next_row[b] = -1;
        uint32_t k = 0;
        if (at) {
            k = (at * 0x9E3779B1u >> 7) & (places - 1);
            while (c.table[k] && c.g[c.table[k] - 1].at != at) k = (k + 1) & (places - 1);
        }
        if (at && c.table[k]) {                           // one more row of a group: whose knowledge is the better one to send?
            RowGroup &g = c.g[c.table[k] - 1];
            c.next_row[b] = g.last; g.last = b; g.n++;
            if (!g.dev) {
                const bool known = device_knows(d, st);
                if ((known && !g.known) || (known && st->pending.size() < g.lead->pending.size())) { g.lead = st; g.known = known; }
            }
            continue;
        }
        RowGroup g{};
        g.lead = st; g.at = at; g.last = b; g.n = 1;
        g.dev = at == HostAutomaton::ROOT ? STORE_ROOT_ID : at == HostAutomaton::SINK ? (uint32_t)HostAutomaton::SINK : device_name_of(e, st);
        g.known = device_knows(d, st);
        c.g.push_back(g);
        if (at) c.table[k] = (uint32_t)c.g.size();
    }
    const int ng = (int)c.g.size();
    // ---- state cache (Section 5.2): groups whose finished mask is in the pool, and slots for the others ----
    const bool sc = !noalloc && !d->cache.empty() && (size_t)batch * 2 <= d->cache.size();
    int n_miss = 0, n_hits = 0;
    if (sc) {
        if (d->pool_epoch != e->host_epoch) { forget_cached_masks(d); d->pool_epoch = e->host_epoch; }
        const uint32_t slots = (uint32_t)d->cache.size(), call = ++d->pool_call;
        d->host_of_slot.resize(slots, 0); d->slot_stamp.resize(slots, 0);
        for (RowGroup &g : c.g) {
            if (!g.at || g.at == HostAutomaton::SINK) { n_miss++; n_hits += g.n - 1; continue; }
            if (g.at >= d->slot_of_host.size()) d->slot_of_host.resize(std::max<size_t>(g.at + 1, d->slot_of_host.size() * 2), 0);
            const uint32_t have = d->slot_of_host[g.at];
            if (have) { g.pooled = 1; g.slot = have - 1; d->slot_stamp[g.slot] = call; n_hits += g.n; }
        }
        for (RowGroup &g : c.g) {                         // a slot for each of the others: round-robin victim, never one of this call's
            if (g.pooled || !g.at || g.at == HostAutomaton::SINK) continue;
            while (d->slot_stamp[d->pool_victim] == call) d->pool_victim = (d->pool_victim + 1) % slots;
            g.slot = d->pool_victim; g.keep = 1;
            d->pool_victim = (d->pool_victim + 1) % slots;
            if (d->host_of_slot[g.slot]) d->slot_of_host[d->host_of_slot[g.slot]] = 0;
            d->host_of_slot[g.slot] = g.at; d->slot_of_host[g.at] = g.slot + 1; d->slot_stamp[g.slot] = call;
            n_miss++; n_hits += g.n - 1;
        }
    }
    d->report.cache_hits = n_hits; d->report.cache_misses = n_miss;
    // ---- what each group sends ----
    DeviceSide::CallRecord &rec = d->rec[slot];
    rec.epoch = d->store_epoch; rec.host_epoch = e->host_epoch;
    rec.groups.clear(); rec.rows.clear(); rec.undecided = 0;
    const bool use_cache = !e->opt.disable_token_mask_cache;
    size_t widest = 0, biggest_set = 0, n_spill_ent = 0, n_spill_pend = 0, n_off = 0, n_items = 0;
    bool spill = false, short_rows = true;                // some record does not fit the short form; every cache row's number does
    size_t n_more = 0;                                    // cache rows that a look-up's record does not hold
    uint32_t n_cache_rows = 0;
    c.unknown.clear();
    for (RowGroup &g : c.g)
        if (!g.pooled && !g.dev && !g.known && !g.lead->lag.empty()) c.unknown.push_back(g.lead);
    if (!c.unknown.empty()) catch_up_batch(c.unknown.data(), (int32_t)c.unknown.size());
    for (int r = 0; r < ng; r++) {
        RowGroup &g = c.g[r];
        if (g.pooled) continue;
        const CurrentSet cs = current_set(g.lead);
        g.items = cs.items; g.n_items = cs.n;
        widest = std::max<size_t>(widest, cs.n); biggest_set = std::max<size_t>(biggest_set, cs.biggest);
        g.undecided = e->V;
        if (use_cache) {
            if (g.at && g.at != HostAutomaton::SINK) {    // worked out once per state
                HostAutomaton::State &hs = A.st(g.at);
                if (hs.undecided < 0) {
                    hs.ents.resize(cs.n);
                    hs.ents.resize(current_set_entries(e->tab, cs.items, cs.n, hs.ents.data()));
                    hs.undecided = hs.ents.size() <= 64 ? count_undecided(d, hs.ents.data(), (uint32_t)hs.ents.size()) : e->V;
                }
                g.ents = hs.ents.data(); g.n_ent = (uint32_t)hs.ents.size(); g.undecided = (double)hs.undecided;
            } else g.undecided = cs.n ? e->V : 0;         // gathered below, when the vector they go to no longer moves
        }
    }
    if (use_cache)
        for (RowGroup &g : c.g) {
            if (g.pooled || g.ents || !g.n_items) continue;
            const size_t at = c.spare_ents.size();
            c.spare_ents.resize(at + g.n_items);
            g.n_ent = current_set_entries(e->tab, g.items, g.n_items, c.spare_ents.data() + at);
            c.spare_ents.resize(at + g.n_ent);
        }
    {
        const uint32_t *at = c.spare_ents.data();
        for (RowGroup &g : c.g) if (!g.pooled && use_cache && !g.ents) { g.ents = at; at += g.n_ent; }
    }
    c.packed.resize(std::max<size_t>(c.packed.size(), ng));
    for (int r = 0; r < ng; r++) {
        RowGroup &g = c.g[r];
        if (g.pooled) continue;
        n_cache_rows += g.n_ent;
        rec.undecided += (int64_t)g.undecided;
        bool fits = g.n_ent <= (uint32_t)STORE_GROUP_ENT, low = g.n_ent <= LOOK_ENT_MAX;
        for (uint32_t k = 0; low && k < g.n_ent; k++) low = g.ents[k] < 65536u;
        if (!fits) n_more += g.n_ent - LOOK_ENT_OF_MORE;
        fits &= low; short_rows &= low;
        if (!g.dev) {
            if (g.known) { fits &= g.lead->pending.size() <= (size_t)STORE_GROUP_PEND; n_spill_pend += g.lead->pending.size(); }
            else {
                const Chart &ch = chart_of(g.lead);
                c.imports.push_back((uint32_t)r);
                pack_chart(e->tab, ch, c.packed[r]);
                n_off += ch.set_off.size(); n_items += ch.items.size();
            }
        }
        n_spill_ent += g.n_ent;
        spill |= !fits;
    }
    const int n_imp = (int)c.imports.size();
    // Look-ups only: the device's name of every group's state is known, and so is every transition its vocabulary walk can meet --
    // the mask there was computed before in this epoch of the store (a call enqueued earlier on the stream is earlier enough), or
    // the automaton was explored to its end.
    bool look = short_rows && n_imp == 0 && d->tab.W <= 65535 && (size_t)batch + n_more <= 65535;
    for (int r = 0; r < ng && look; r++) {
        const RowGroup &g = c.g[r];
        if (g.pooled || g.dev == HostAutomaton::SINK) continue;
        look = g.dev && g.at && (A.st(g.at).walked == d->store_epoch || (d->closed_epoch == d->store_epoch && g.at < d->closed_states && g.dev == g.at));
    }
    if (look) return enqueue_look(e, c, states, batch, d_mask, stream, wait, noalloc, slot, n_more, n_cache_rows, host_lk);
    const bool big = ng > STORE_INLINE_GROUPS;            // records and members travel in device memory instead of the argument block
    auto align16 = [](size_t x) { return (x + 15) & ~(size_t)15; };
    // staging: [group records][blocks][members] (uploaded when big), then what the kernels read in place
    const int max_blocks = std::max(ng, STORE_BLOCKS_PER_CU * std::max(1, d->cus)) + 8 * ng;
    const size_t off_block = align16(big ? sizeof(StoreGroup) * ng : 0), off_mem = align16(off_block + (big ? 8 * (size_t)max_blocks : 0));
    const size_t up_bytes = align16(off_mem + 2 * (size_t)batch);
    const size_t off_spill = up_bytes, off_ent = align16(off_spill + (spill ? sizeof(StoreRow) * ng : 0)), off_pend = align16(off_ent + (spill ? 4 * n_spill_ent : 0));
    const size_t off_rows = align16(off_pend + (spill ? n_spill_pend : 0)), off_so = align16(off_rows + sizeof(RowChart) * n_imp);
    const size_t off_items = align16(off_so + 4 * n_off), off_imp = align16(off_items + sizeof(Item) * n_items);
    const size_t total = off_imp + 4 * (size_t)n_imp + 16;
    if (noalloc && (total > d->stage_cap[slot] || (big && up_bytes > NOALLOC_SCRATCH_BYTES))) return STORE_NO_ROOM;
    if (total > d->stage_cap[slot]) {
        const int rc = grow_stage(d, slot, total * 2 + 4096);
        if (rc != ZF_OK) return rc;
    }
    if (big && !noalloc && up_bytes > d->chart_cap) {
        HIP_TRY(hipStreamSynchronize(stream));
        if (d->d_chart) (void)hipFree(d->d_chart);
        d->d_chart = nullptr; d->chart_cap = 0;
        const size_t cap = up_bytes * 2 + 4096;
        HIP_TRY(hipMalloc(&d->d_chart, cap));
        d->chart_cap = cap;
    }
    // ---- launch shape ----
    StoreArgs a{};
    int scratch = e->lane_cap_auto ? (int)std::min<size_t>(LANE_CAP_MAX, (4 * widest + 128 + 31) / 32 * 32) : e->opt.lane_item_cap;
    while (scratch > 32 && store_lds_bytes(d->tab, d->mode, scratch) > (uint32_t)STORE_LDS_MAX) scratch -= 32;
    const uint32_t lds = store_lds_bytes(d->tab, d->mode, scratch);
    if (lds > (uint32_t)STORE_LDS_MAX) return fail(ZF_ERR_INVALID_ARG, "the grammar tables leave no LDS for the mask kernel");
    int logit_bytes = 0;                                  // of a logit the mask kernel masks itself
    const size_t esz = g_apply.dtype == 0 ? 4 : 2;
    const bool whole = g_apply.out && (uintptr_t)g_apply.logits % esz == 0 && (uintptr_t)g_apply.out % esz == 0;
    if (g_apply.out) {
        // mask_store_kernel does both as long as the logits are few enough that masking them hides behind the walk of the vocabulary;
        // beyond, a launch of its own masks them at the memory's rate with the work spread evenly over the chip.
        if (whole && 2ull * (uint64_t)batch * (uint64_t)e->V * esz <= STORE_FUSE_BYTES) {
            a.logits = g_apply.logits; a.out = g_apply.out; a.stride = g_apply.stride; a.dtype = (uint8_t)(g_apply.dtype + 1);
            g_apply.fused = true;
            logit_bytes = (int)esz;
        }
    }
    const int budget = std::max(ng, std::min(STORE_BLOCKS_PER_CU, store_blocks_per_cu(d->tab, d->mode, scratch)) * std::max(1, d->cus));
    a.n_blocks = (uint32_t)store_launch_shape(c.g, d->tab.W, e->V, budget, logit_bytes, 0);
    // ---- the records ----
    {
        uint8_t *h = (uint8_t *)d->h_stage[slot];
        StoreGroup *gr = big ? (StoreGroup *)h : c.in.g;
        uint32_t *blk = (uint32_t *)(h + off_block);
        uint16_t *mem = big || batch > STORE_INLINE_ROWS ? (uint16_t *)(h + off_mem) : c.in.member;
        StoreRow *srow = (StoreRow *)(h + off_spill);
        uint32_t *ents = (uint32_t *)(h + off_ent);
        uint8_t *pend = h + off_pend;
        RowChart *rows = (RowChart *)(h + off_rows);
        uint32_t *so = (uint32_t *)(h + off_so);
        uint32_t *dev_items = (uint32_t *)(h + off_items);
        uint32_t *imp = (uint32_t *)(h + off_imp);
        uint32_t mem_at = 0, en_at = 0, pe_at = 0, so_at = 0, it_at = 0, k_imp = 0, blk_at = 0;
        for (int r = 0; r < ng; r++) {
            RowGroup &g = c.g[r];
            zf_state *st = g.lead;
            uint32_t flags = use_cache ? STORE_ROW_CACHE : 0u, start, n_pending = 0;
            const uint8_t *pending = nullptr;
            uint64_t hop = 0;
            if (g.pooled) { flags = STORE_ROW_POOLED; start = g.slot; }
            else if (g.dev) start = g.dev;
            else if (g.known) {
                start = st->dev_id; n_pending = (uint32_t)st->pending.size(); pending = st->pending.data();
                if (n_pending && st->pending_token >= 0 && st->dev_id != HostAutomaton::SINK) {
                    const uint64_t key = (uint64_t)st->dev_id << 32 | ((uint32_t)st->pending_token + 1u);
                    const uint32_t to = d->hop_find(key);
                    if (to) { start = to; n_pending = 0; }            // somebody has walked this token from this state before
                    else hop = key;
                }
            } else {
                const Chart &ch = chart_of(st);
                const std::vector<uint32_t> &k = c.packed[r];
                flags |= STORE_ROW_IMPORTED; start = 0;
                rows[k_imp] = RowChart{ch.n_sets(), so_at, it_at, 0, 0, (uint32_t)ch.items.size(), {0, 0}};
                memcpy(so + so_at, k.data() + 1, 4 * ch.set_off.size());
                memcpy(dev_items + 2 * (size_t)it_at, k.data() + 1 + ch.set_off.size(), 8 * ch.items.size());
                so_at += (uint32_t)ch.set_off.size(); it_at += (uint32_t)ch.items.size();
                imp[k_imp++] = (uint32_t)r;
            }
            if (g.keep) flags |= STORE_ROW_KEEP;
            if (!g.pooled && !g.dev) {                    // the kernel says where these rows stand: noted by zf_mask_wait
                flags |= STORE_ROW_REPORT;
                rec.groups.push_back({(uint32_t)r, g.at < HostAutomaton::SINK ? g.at : 0u, (uint32_t)rec.rows.size(), (uint32_t)g.n, hop});
            }
            const uint32_t first_mem = mem_at;
            for (int32_t b = g.last; b >= 0; b = c.next_row[b]) {
                mem[mem_at++] = (uint16_t)b;
                if (g.dev) note_device_state(d, states[b], g.dev);
                else if (!g.pooled) {
                    rec.rows.push_back({states[b]->link, states[b]->generation, states[b]->fed_total});
                    if (!g.known) { states[b]->pending.clear(); states[b]->pending_base = states[b]->fed_total; states[b]->pending_token = -1; }   // the chart holds everything fed so far
                }
            }
            StoreGroup &m = gr[r];
            m.start = start; m.slot = (uint16_t)g.slot; m.member_at = (uint16_t)first_mem; m.n_members = (uint16_t)g.n;
            bool fits = n_pending <= (uint32_t)STORE_GROUP_PEND && g.n_ent <= (uint32_t)STORE_GROUP_ENT;
            for (uint32_t k = 0; fits && k < g.n_ent; k++) fits = g.ents[k] < 65536u;
            if (fits) {
                m.meta = n_pending | g.n_ent << 8;
                if (n_pending) memcpy(m.pend, pending, n_pending);
                for (uint32_t k = 0; k < g.n_ent; k++) m.ent[k] = (uint16_t)g.ents[k];
            } else {
                m.meta = 0; flags |= STORE_ROW_SPILL;
                StoreRow &sr = srow[r];
                sr.start = start; sr.n_pending = n_pending; sr.pend_off = pe_at; sr.n_ent = g.n_ent; sr.ent_off = en_at; sr.flags = flags;
                if (g.n_ent <= (uint32_t)STORE_ROW_ENT) memcpy(sr.ent, g.ents, 4 * (size_t)g.n_ent);
                else { memcpy(ents + en_at, g.ents, 4 * (size_t)g.n_ent); en_at += g.n_ent; }
                if (n_pending <= (uint32_t)STORE_ROW_PEND) memcpy(sr.pend, pending, n_pending);
                else { memcpy(pend + pe_at, pending, n_pending); pe_at += n_pending; }
            }
            m.meta |= flags << 16 | (uint32_t)(g.seg_w - 1) << 24;
            if (big) for (int p = 0; p < g.parts; p++) { blk[2 * blk_at] = (uint32_t)r; blk[2 * blk_at + 1] = (uint32_t)p | (uint32_t)g.parts << 16; blk_at++; }
            else { c.in.first_block[r] = (uint16_t)blk_at; blk_at += (uint32_t)g.parts; }
        }
        if (!big) for (int r = ng; r < STORE_INLINE_GROUPS + 8; r++) c.in.first_block[r] = r == ng ? (uint16_t)blk_at : (uint16_t)0xFFFF;   // the kernel compares against all of them
    }
    const DeviceTables &T = d->tab;
    uint8_t *stage = (uint8_t *)d->h_stage[slot];
    a.cache = T.ci_tok; a.tok16 = T.tok16; a.trans = d->store.trans;
    a.out_mask = d_mask; a.pool = d->d_pool; a.konst = d->d_konst;
    a.spilled = (const StoreRow *)(stage + off_spill); a.entries = (const uint32_t *)(stage + off_ent); a.pending = stage + off_pend;
    a.import_root = d->d_import_root;
    uint8_t *const uploaded = noalloc ? d->scratch : (uint8_t *)d->d_chart;
    if (big) {
        a.groups = (const StoreGroup *)uploaded;
        a.block_of = (const uint32_t *)(uploaded + off_block);
        a.members = (const uint16_t *)(uploaded + off_mem);
    } else if (batch > STORE_INLINE_ROWS) a.members = (const uint16_t *)(stage + off_mem);
    a.tickets = d->d_tickets + d->ticket_set * STORE_TICKETS; a.tickets_next = d->d_tickets + (d->ticket_set ^ 1u) * STORE_TICKETS;
    a.status = (unsigned long long *)d->h_store_status + slot * STORE_STATUS_WORDS;
    HIP_TRY(next_call_number(d, stream));
    a.seq = rec.seq = d->call_seq;
    a.V = (uint32_t)e->V; a.W = (uint32_t)T.W; a.ncls = (uint32_t)T.n_cls; a.cap_states = d->store.cap_states; a.tab_mode = (uint32_t)d->mode;
    a.scratch = scratch;
    a.wide = biggest_set > (size_t)AUT_NARROW_SET_MAX ? 1 : 0;   // a hint: which variant of the byte step to try first on larger sets
    a.complete = wait ? 1 : 0;
    a.report_size = n_imp ? 1 : 0;
    const bool prof = d->profiling;
    d->report.chart_bytes = (int64_t)(total + (big ? 0 : sizeof(StoreGroup) * ng));
    d->report.cache_rows = (int32_t)n_cache_rows;
    d->report.main_ms = d->report.fallback_ms = d->report.permute_ms = 0.f;
    d->report.overflow_chunks = d->report.walk_chunks = d->report.parser_steps = 0;
    if (big) HIP_TRY(launch_upload(stage, uploaded, up_bytes, stream));
    if (n_imp) HIP_TRY(launch_store_import(d->store, (const RowChart *)(stage + off_rows), (const uint32_t *)(stage + off_so), (const Item *)(stage + off_items),
                                           (const uint32_t *)(stage + off_imp), (uint32_t)n_imp, d->d_import_root, stream));
    if (prof) HIP_TRY(hipEventRecord(d->ev[0], stream));
    d->closing_kernel = false;
    rec.debug_failed = 0;
    rec.done_groups = 0;
    HIP_TRY(launch_mask_store(a, c.in, lds, stream));
    for (const RowGroup &g : c.g) if (!g.pooled && g.at && g.at != HostAutomaton::SINK) A.st(g.at).walked = d->store_epoch;
    d->ticket_set ^= 1u;
    if (prof) { HIP_TRY(hipEventRecord(d->ev[1], stream)); HIP_TRY(hipEventRecord(d->ev[3], stream)); }
    d->next_slot = (slot + 1) % DeviceSide::N_SLOTS;
    d->pending++;
    d->last_seq = a.seq; d->last_slot = slot;
    rec.active = true;
    rec.sure = false;
    host_lk.unlock();
    // the waiting call returns with the mask complete: the kernel wrote it through to memory before it drew its tickets
    return wait ? wait_for_calls(e, hip_stream) : ZF_OK;
}

// A call that fails part-way may have registered cache slots whose masks were never written.
static int enqueue_mask(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, void *hip_stream, bool wait, bool noalloc = false) {
    DeviceSide *d = e ? e->dev : nullptr;
    bool per_block = false;                               // persistent automaton on hold after a call it had no room for
    if (d && e->store_on && d->store_backoff) { d->store_backoff--; per_block = true; }
    int rc = enqueue_mask_impl(e, states, batch, d_mask, hip_stream, wait, noalloc, per_block);
    if (rc != ZF_OK && d) forget_cached_masks(d);
    if (rc == ZF_ERR_OVERFLOW && d && e->store_on && !per_block && !(noalloc && !e->lane_cap_auto)) {
        // A set outgrew a wavefront's scratch, or the store filled up within one call.  The waiting call answers through the
        // per-block automaton, whose fallback pass has room in global memory; either way the next calls go that way too,
        // for longer each time it happens, and the store starts over when it is used again.
        d->store_dirty = true;
        d->store_backoff = d->store_backoff_next;
        d->store_backoff_next = std::min<uint32_t>(1024, d->store_backoff_next * 2);
        if (wait) {
            rc = enqueue_mask_impl(e, states, batch, d_mask, hip_stream, wait, noalloc, true);
            if (rc != ZF_OK) forget_cached_masks(d);
        }
    }
    if (rc == ZF_OK && wait) {                            // calls that were let go of are behind the stream's newest by now: what they have to report is there
        rc = settle_calls(d);
        if (rc == ZF_OK) rc = report_late(d);
    }
    return rc;
}

int zf_compute_mask(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, void *hip_stream) {
    return enqueue_mask(e, states, batch, d_mask, hip_stream, true);
}

// What the persistent automaton holds when a decode loop starts (zf_options.precompute_states).  The host's automaton is explored
// breadth first from the state of the empty prefix, one byte class at a time (every DFA treats the bytes of a class alike), and
// the device's is filled with it: the same states under the same names, and every transition the host knows.  The exploration
// ends when no new state turns up -- a grammar without recursion has a finite automaton, which is then built whole, as engines
// for regular constraints build theirs when they compile -- or at the budget of states or of time, or when it would fill a
// quarter of the store (the store starts over when it is half full, and what a decode loop adds needs room).
//   Built by the library's own calls before -- a zf_state cloned and advanced per state and class, a mask call per 64 states
// and 64 transitions -- the 20,962 states of a JSON schema took 417 ms: 55 clones and steps per state where four classes are
// live (State::trans: a class on which no item leaves anything is known to be dead), chart copies, an ordered map of item lists.
static bool wants_exploration(const zf_engine *e) { return e->store_on && e->host_aut && e->opt.precompute_states > 0; }

// The host's part: touches nothing but the host automaton.  True when the automaton is finite and whole.
// lk: the engine's lock, held, when others may be at work with the engine (null: nobody else knows it yet).  It is let go during
// every Earley byte step, as zf_advance lets it go: rows that are advanced meanwhile wait for one transition to be written
// down, not for the exploration.  It is held again when this returns, and nothing has been added since the answer was found.
static bool explore_host(zf_engine *e, size_t cap_states, size_t cap_items, std::unique_lock<std::mutex> *lk) {
    HostAutomaton &A = *e->host_aut;
    const auto t0 = std::chrono::steady_clock::now();
    const double budget_s = 1.0;
    const size_t most_states = std::min((size_t)e->opt.precompute_states, cap_states / 4), most_items = cap_items / 4;
    HostAutomaton::Work w;
    HostAutomaton::Completed known;
    std::vector<Item> scanned;
    for (uint32_t s = HostAutomaton::ROOT; s < A.n_states; s++) {
        if ((s & 63u) == 0 && std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() >= budget_s) return false;
        const HostAutomaton::Classes live = A.live_classes(A.st(s).items, A.st(s).n_items);
        for (int k = 0; k < 4; k++) for (uint64_t left = live.w[k]; left; left &= left - 1) {
            const int c = 64 * k + __builtin_ctzll(left);
            if (A.st(s).trans[c] != HostAutomaton::NONE) continue;
            if (A.n_states > most_states || (size_t)A.n_items >= most_items) return false;
            const HostAutomaton::Completed::Entry *to = nullptr;
            uint32_t sig = 0;
            bool completes = false;
            auto step = [&]() {
                A.scan(s, c, s, w);
                completes = A.completes(w);
                if (completes && (to = known.find(w.set, sig))) return;
                if (completes) scanned = w.set;
                A.close(w);
            };
            if (lk) {
                struct Walker {                           // keeps the automaton from being emptied meanwhile
                    int &n;
                    std::unique_lock<std::mutex> &lk;
                    Walker(int &n_, std::unique_lock<std::mutex> &lk_) : n(n_), lk(lk_) { n++; lk.unlock(); }
                    ~Walker() { lk.lock(); n--; }
                } walker(e->host_walkers, *lk);
                step();
            } else step();
            if (A.st(s).trans[c] != HostAutomaton::NONE) continue;   // somebody else has made it meanwhile
            if (to) { A.record(s, c, to->to, to->accepted); continue; }
            A.record(s, c, w);
            if (completes) known.add(scanned, sig, A.st(s).trans[c], w.accepted);
        }
    }
    return true;
}

// What a mask call works out when it meets a list of several cache rows for the first time -- the tokens they leave undecided, 10 us and more
// per list of a large vocabulary -- is worked out for the explored states when the engine is compiled: left to the calls, the first pass over
// 64 rows of the query language took 125 us per step, the following ones 83; with it the first takes 85, and compiling a schema 19.0 ms
// either way.
// The lists are gathered by the exploring thread, while the vocabulary is sorted elsewhere, nearest states first; they are
// few (56 to 1,397 distinct ones in 65,536 states of the grammars of workloads/, most of them of one row).
static std::vector<std::vector<uint32_t>> explored_entries(const zf_engine *e) {
    const HostAutomaton &A = *e->host_aut;
    std::vector<std::vector<uint32_t>> lists;
    std::unordered_map<uint64_t, bool> met;
    std::vector<uint32_t> ents;
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t s = HostAutomaton::ROOT; s < A.n_states && lists.size() < 4096; s++) {
        if ((s & 255u) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(20)) break;
        const HostAutomaton::State &st = A.st(s);
        ents.resize(std::max<size_t>(ents.size(), st.n_items));
        const uint32_t n = current_set_entries(e->tab, st.items, st.n_items, ents.data());
        if (n < 2 || n > 64 || !met.emplace(entries_signature(ents.data(), n), true).second) continue;
        lists.emplace_back(ents.begin(), ents.begin() + n);
    }
    return lists;
}
static void count_lists(zf_engine *e, const std::vector<std::vector<uint32_t>> &lists) {
    DeviceSide *d = e->dev;
    std::vector<uint32_t> count(lists.size());
    parallel_for(lists.size(), lists.size() >= 64 ? 4 : 1, [&](size_t k) { count[k] = undecided_tokens(d->h_ci_tok, (size_t)e->W, lists[k].data(), (uint32_t)lists[k].size()); });
    for (size_t k = 0; k < lists.size(); k++) d->undecided_of.emplace(entries_signature(lists[k].data(), (uint32_t)lists[k].size()), count[k]);
}

// The device's part: the store is cleared and takes over what the host automaton holds, names and all.  A failure is no error:
// the store then starts empty, as it does without an exploration.  lk as above; it is let go as soon as what goes to the device has been copied.
static void store_adopt(zf_engine *e, bool whole, std::unique_lock<std::mutex> *lk) {
    DeviceSide *d = e->dev;
    const HostAutomaton &A = *e->host_aut;
    const Tables &t = e->tab;
    const StoreView &G = d->store;
    const size_t n = A.n_states, ncls = (size_t)std::max(t.n_cls, 1);
    static_assert(HostAutomaton::ROOT == 1 && HostAutomaton::NONE == ~0u && HostAutomaton::DEAD == ~1u && HostAutomaton::SINK == ~2u, "the device's table uses the same words");
    if (n < 2 || n > G.cap_states / 2 || (size_t)A.n_items + d->n_root > G.cap_items / 2) return;
    std::vector<uint2> hdr(n), items;
    items.reserve((size_t)A.n_items + d->n_root);
    hdr[0] = make_uint2(0, 0xFFFFFFFFu);                  // no such state: as the clearing kernel leaves it
    for (uint32_t id = 1; id < n; id++) {
        const HostAutomaton::State &s = A.st(id);
        hdr[id] = make_uint2((uint32_t)items.size(), s.n_items);
        for (uint32_t i = 0; i < s.n_items; i++) {
            const uint32_t aw = t.advpq[s.items[i].p];
            items.push_back(make_uint2((aw & IW_TERM) ? ((aw & 0xFFFFu) | ((uint32_t)s.items[i].q << 16)) : aw, s.items[i].o));
        }
    }
    // the host's rows of the table, block by block: where they are, or copies that others' work on the automaton cannot change
    std::vector<uint32_t> rows_now;
    std::vector<const uint32_t *> block_rows;
    if (lk) rows_now.resize(n * ncls);
    for (size_t b = 0; b * HostAutomaton::BLOCK < n; b++) {
        const size_t first = b * HostAutomaton::BLOCK, rows = std::min<size_t>(HostAutomaton::BLOCK, n - first);
        if (lk) memcpy(rows_now.data() + first * ncls, A.blocks[b].trans.get(), rows * ncls * 4);
        block_rows.push_back(lk ? rows_now.data() + first * ncls : A.blocks[b].trans.get());
    }
    const uint32_t host_epoch = e->host_epoch;
    if (lk) lk->unlock();
    auto run = [&]() -> hipError_t {
        hipError_t rc = hipSetDevice(d->device);
        if (rc == hipSuccess) rc = launch_store_clear(G, (uint32_t)ncls, d->d_root_items, d->n_root, nullptr);
        if (rc == hipSuccess) rc = hipMemcpyAsync(G.hdr, hdr.data(), n * sizeof(uint2), hipMemcpyHostToDevice, nullptr);
        if (rc == hipSuccess) rc = hipMemcpyAsync(G.arena, items.data(), items.size() * sizeof(uint2), hipMemcpyHostToDevice, nullptr);
        for (size_t b = 0; rc == hipSuccess && b < block_rows.size(); b++) {
            const size_t rows = std::min<size_t>(HostAutomaton::BLOCK, n - b * HostAutomaton::BLOCK);
            rc = hipMemcpyAsync(G.trans + b * HostAutomaton::BLOCK * ncls, block_rows[b], rows * ncls * 4, hipMemcpyHostToDevice, nullptr);
        }
        if (rc == hipSuccess) rc = launch_store_adopt(G, (uint32_t)n, (uint32_t)items.size(), nullptr);
        if (rc == hipSuccess) rc = hipStreamSynchronize(nullptr);
        return rc;
    };
    d->store_dirty = true;
    if (run() != hipSuccess) { (void)hipGetLastError(); return; }
    d->store_dirty = false;
    d->store_epoch++;
    d->store_states = (uint32_t)n; d->store_items = (uint32_t)items.size();
    d->name_host_epoch = host_epoch; d->name_store_epoch = d->store_epoch;
    d->name_of_host.resize(n);
    for (uint32_t id = 0; id < n; id++) d->name_of_host[id] = id;
    if (whole) { d->closed_states = (uint32_t)n; d->closed_epoch = d->store_epoch; }
}

int zf_compute_mask_noalloc(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, void *hip_stream) {
    if (e && e->dev && e->dev->pending) return fail(ZF_ERR_INVALID_ARG, "zf_compute_mask_noalloc: asynchronous mask calls are in flight: call zf_mask_wait first");
    return enqueue_mask(e, states, batch, d_mask, hip_stream, true, true);
}

int zf_compute_mask_async(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, void *hip_stream) {
    return enqueue_mask(e, states, batch, d_mask, hip_stream, false);
}

int zf_compute_mask_apply_async(zf_engine *e, zf_state *const *states, int32_t batch, uint32_t *d_mask, const void *d_logits, void *d_out,
                                int32_t dtype, int64_t row_stride, void *hip_stream) {
    if (!e || !d_logits || !d_out || (dtype != 0 && dtype != 1) || row_stride < (e ? e->V : 0)) return fail(ZF_ERR_INVALID_ARG, "bad argument");
    g_apply = ApplyRequest{d_logits, d_out, row_stride, dtype, false};
    const int rc = enqueue_mask(e, states, batch, d_mask, hip_stream, false);
    const bool fused = g_apply.fused;
    g_apply = ApplyRequest{};
    if (rc != ZF_OK || fused) return rc;
    return zf_apply_mask(e, d_logits, d_out, dtype, batch, row_stride, d_mask, hip_stream);   // the trie walk, the state cache, first visits over many logits, odd addresses: two launches
}

static int wait_for_calls(zf_engine *e, void *hip_stream) {
    DeviceSide *d = e->dev;
    HIP_TRY(hipSetDevice(d->device));
    volatile uint32_t *st = d->h_status;
    auto await = [&](auto arrived) -> int { return await_status(arrived, [&] { return hipStreamSynchronize((hipStream_t)hip_stream); }); };
    uint32_t unresolved = 0;
    if (d->pending) {
        int rc = ZF_OK;
        // calls of one engine run in stream order: once the newest has reported, the older ones in flight have finished too
        if (!d->rec[d->last_slot].active) {
            volatile uint32_t *flag = st + 8 * d->last_slot + 4;
            rc = await([&]() { return *flag == d->last_seq; });
        }
        // the calls through the persistent automaton, oldest first: their status, and where their rows stand
        for (int i = 0; i < DeviceSide::N_SLOTS; i++) {
            const uint32_t k = (d->next_slot + i) % DeviceSide::N_SLOTS;
            DeviceSide::CallRecord &rec = d->rec[k];
            if (!rec.active) continue;
            rec.active = false;
            struct Release { DeviceSide::CallRecord &r; ~Release() { r.rows.clear(); r.groups.clear(); } } release{rec};
            if (rc != ZF_OK) continue;
            if (rec.sure) {                               // its status was final when it was enqueued
                rec.lazy = true; d->n_lazy++;
                d->report.walk_chunks = rec.undecided;
                d->report.parser_steps = 0;
                continue;
            }
            const volatile uint64_t *out = d->h_store_status + k * STORE_STATUS_WORDS;
            auto got = [&](size_t w) { return (uint32_t)(out[w] >> 32) == rec.seq; };
            if ((rc = await([&]() { return rec.done_groups ? look_done(out, rec) : got(STORE_ST_DONE); })) != ZF_OK) continue;
            const uint32_t done = rec.done_groups ? look_failed(out, rec) : (uint32_t)out[STORE_ST_DONE], failed = done & 0xFFFFFFu;
            unresolved += failed;
            d->report.walk_chunks = rec.undecided;
            d->report.parser_steps = 0;
            if (failed) d->store_dirty = true;            // a walk failed: start over
            if (done & STORE_ST_MORE) {                   // every word says by itself whether it is in
                if ((rc = await([&]() { return got(STORE_ST_STEPS) && got(STORE_ST_STATES) && got(STORE_ST_ITEMS) && got(STORE_ST_REFUSED); })) != ZF_OK) continue;
                d->report.parser_steps = (int32_t)(uint32_t)out[STORE_ST_STEPS];
                d->store_states = (uint32_t)out[STORE_ST_STATES]; d->store_items = (uint32_t)out[STORE_ST_ITEMS];
                if ((uint32_t)out[STORE_ST_REFUSED]) d->store_dirty = true;   // the store refused a request: start over
            }
            if (failed || rec.epoch != d->store_epoch) continue;
            for (const DeviceSide::CallRecord::Group &g : rec.groups) {
                if ((rc = await([&]() { return got(STORE_ST_ROW + g.group); })) != ZF_OK) break;
                const uint32_t at = (uint32_t)out[STORE_ST_ROW + g.group];
                if (at == 0 || (at >= d->store.cap_states && at != HostAutomaton::SINK)) continue;
                if (g.hop) d->hop_note(g.hop, at);                                // a fact about the automaton, whatever has become of the rows
                if (g.host_id && at != HostAutomaton::SINK) d->name_note(g.host_id, rec.host_epoch, rec.epoch, at);   // and so is this
                for (uint32_t r = g.first; r < g.first + g.n; r++) {
                    const DeviceSide::CallRecord::Row &row = rec.rows[r];
                    zf_state *s = row.st ? row.st->s : nullptr;
                    if (!s || s->generation != row.gen) continue;
                    if (row.upto < s->pending_base) continue;                     // a later call's result is already in
                    const size_t drop = std::min<size_t>((size_t)(row.upto - s->pending_base), s->pending.size());
                    s->pending_token = -1;
                    s->pending.erase(s->pending.begin(), s->pending.begin() + drop);
                    s->pending_base = row.upto;
                    s->dev_id = at; s->dev_epoch = rec.epoch;
                }
            }
        }
        if (rc != ZF_OK) { d->pending = 0; return rc; }
        if (d->profiling) HIP_TRY(hipEventSynchronize(d->ev[3]));
    } else {
        HIP_TRY(hipStreamSynchronize((hipStream_t)hip_stream));   // nothing of this engine in flight: plain stream synchronisation ...
        const int rc = settle_calls(d);                   // ... but for calls that were let go of
        if (rc != ZF_OK) return rc;
    }
    for (int k = 0; k < DeviceSide::N_SLOTS; k++) {
        unresolved += st[8 * k + 2];
        if (st[8 * k + 0] && d->lanes_call[k]) d->lanes_outgrown = true;
        if (st[8 * k + 0] || st[8 * k + 1]) { d->report.overflow_chunks = st[8 * k + 0]; d->report.walk_chunks = st[8 * k + 1]; d->report.parser_steps = st[8 * k + 3]; }
        st[8 * k + 0] = st[8 * k + 1] = st[8 * k + 2] = st[8 * k + 3] = 0;
    }
    if (d->pending && d->profiling) {
        (void)hipEventElapsedTime(&d->report.main_ms, d->ev[0], d->ev[1]);
        d->report.fallback_ms = 0.f;                      // the fallback pass is part of the closing kernel
        if (d->closing_kernel) (void)hipEventElapsedTime(&d->report.permute_ms, d->ev[1], d->ev[3]);
        else d->report.permute_ms = 0.f;                  // the mask kernel was the call's only kernel
    }
    d->pending = 0;
    if (unresolved) forget_cached_masks(d);               // masks written by the failed call must not be served from the cache
    if (unresolved) return fail(ZF_ERR_OVERFLOW, std::to_string(unresolved) + " trie chunks exceeded the fallback arena");
    return ZF_OK;
}

int zf_mask_wait(zf_engine *e, void *hip_stream) {
    if (!e || !e->dev) return fail(ZF_ERR_INVALID_ARG, "bad argument");
    const int rc = wait_for_calls(e, hip_stream);
    return rc != ZF_OK ? rc : report_late(e->dev);
}

int zf_engine_clear_state_cache(zf_engine *e) {
    if (!e) return fail(ZF_ERR_INVALID_ARG, "null argument");
    if (e->dev && e->dev->n_lazy) {
        HIP_TRY(hipSetDevice(e->dev->device));
        const int rc = settle_calls(e->dev);
        if (rc != ZF_OK) return rc;
    }
    if (e->dev) { forget_cached_masks(e->dev); e->dev->store_dirty = true; }   // the persistent automaton starts over as well
    if (e->host_aut) {                                    // and so does the host's: the states find their way back through their charts
        std::unique_lock<std::mutex> lk(e->host_mu);
        while (e->host_walkers != 0) { lk.unlock(); std::this_thread::yield(); lk.lock(); }   // somebody is at work on a transition (and waits for nobody)
        e->host_aut->clear();
        e->host_epoch++;
        if (wants_exploration(e) && e->dev && e->dev->pending == 0) {   // back to what the engine knew when it was compiled (with calls in flight the store is cleared later, and starts empty)
            try {
                const bool whole = explore_host(e, e->dev->store.cap_states, e->dev->store.cap_items, &lk);
                store_adopt(e, whole, &lk);
            } catch (const std::bad_alloc &) {}           // the store starts empty, then
        }
    }
    return ZF_OK;
}

int zf_last_mask_report(const zf_engine *e, zf_mask_report *out) {
    if (!e || !out || !e->dev) return fail(ZF_ERR_INVALID_ARG, "bad argument");
    *out = e->dev->report;
    return ZF_OK;
}

int zf_engine_set_profiling(zf_engine *e, int32_t on) {
    if (!e || !e->dev) return fail(ZF_ERR_INVALID_ARG, "bad argument");
    HIP_TRY(hipSetDevice(e->dev->device));
    if (on) for (auto &ev : e->dev->ev) if (!ev) HIP_TRY(hipEventCreate(&ev));
    e->dev->profiling = on != 0;
    return ZF_OK;
}

int zf_apply_mask(zf_engine *e, const void *d_logits, void *d_out, int32_t dtype, int32_t batch,
                  int64_t row_stride, const uint32_t *d_mask, void *hip_stream) {
    if (!e || !d_logits || !d_out || !d_mask || batch <= 0 || (dtype != 0 && dtype != 1) || row_stride < e->V)
        return fail(ZF_ERR_INVALID_ARG, "bad argument");
    if (!e->dev) return fail(ZF_ERR_DEVICE, "engine was compiled without a device (device = -1)");
    HIP_TRY(hipSetDevice(e->dev->device));
    if (e->V == 0) return ZF_OK;
    HIP_TRY(launch_apply_mask(d_logits, d_out, dtype, batch, row_stride, e->V, e->W, d_mask, (hipStream_t)hip_stream));
    return ZF_OK;
}

}  // extern "C"
