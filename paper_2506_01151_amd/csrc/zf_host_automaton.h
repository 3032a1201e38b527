// The persistent automaton on the host: every Earley set named by its content, items carrying the name of the
// set their rule started in, so the sets of all rows and decode steps are the states of one deterministic
// automaton over byte classes (Sections 4.4, 5.2).  zf_advance walks a token's bytes through it (a look-up per
// byte once a transition is known, one Earley byte step -- Scan, Complete, tabulated Predict: Section 3.2 --
// the first time); the diagnostics of include/zapformat_debug.h use a second instance as the twin of the
// device's store.  A state refers only to the sets its items started in, transitively, which is what
// ZapFormat's reachability closure keeps of a chart (Section 4.2.3); completed items are dropped when a set is
// closed (Figure 3, first rule), so no separate Compact pass is needed here.
//
// Sharing.  A state's items never change once the state has a name, and states live in blocks whose addresses
// never change, so a thread that has learnt a name under the owner's lock may read that state's items without
// it (lay_out); everything that writes (record, import, clear) and every look-up of a transition runs under the
// lock.  clear() frees the blocks: the owner calls it only while no thread is between lay_out and record.
#pragma once
#include <algorithm>
#include <cstring>
#include <memory>
#include "zf_internal.h"

namespace zf {

struct HostAutomaton {
    const Tables &t;
    static constexpr uint32_t ROOT = 1, SINK = 0xFFFFFFFDu, DEAD = 0xFFFFFFFEu, NONE = 0xFFFFFFFFu;
    static constexpr uint32_t BLOCK = 1024, MAX_BLOCKS = 1024;     // at most BLOCK x MAX_BLOCKS states
    static constexpr uint32_t ITEM_CHUNK = 1u << 15;               // items are kept in chunks of this many (a larger set has a chunk of its own)
    struct State {
        const Item *items = nullptr;      // an item's origin is a state id
        uint32_t n_items = 0;
        uint32_t widest = 0;              // items of the largest set among the state and the sets it refers to
        uint32_t sig = 0;                 // signature of the content
        uint32_t *trans = nullptr;        // [n_cls] next state, NONE, DEAD or SINK
        uint8_t *acc = nullptr;           // [n_cls] the prefix is a sentence after that byte
        std::vector<uint32_t> ents;       // what the mask calls work out about the state once: the rows of the token-mask cache its items select ...
        int64_t undecided = -1;           // ... and how many tokens these leave to the parser (-1: not yet)
        uint32_t walked = 0;              // epoch of the device's store in which the mask at this state was computed: its transitions are all there
    };
    // States, and their rows of the transition table (one run of memory per block: the device's table is filled from it).
    struct Block { std::unique_ptr<State[]> states; std::unique_ptr<uint32_t[]> trans; std::unique_ptr<uint8_t[]> acc; };
    std::vector<Block> blocks;            // room for MAX_BLOCKS from the start: the array never moves
    std::vector<std::unique_ptr<Item[]>> chunks;
    uint32_t chunk_used = ITEM_CHUNK;
    uint32_t n_states = 0;                // ids 0 .. n_states - 1 are taken (0 is not used)
    std::vector<uint64_t> interned;       // open addressing by State::sig, at most half full: sig << 32 | id (a look at a state of another signature is spared); 0 = free
    int64_t n_steps = 0, n_items = 0;
    struct Classes { uint64_t w[4] = {0, 0, 0, 0}; void add(int c) { w[c >> 6] |= 1ull << (c & 63); } void add(const Classes &o) { for (int k = 0; k < 4; k++) w[k] |= o.w[k]; } bool has(int c) const { return (w[c >> 6] >> (c & 63)) & 1u; } };
    std::vector<Classes> q_live, nt_live; // [Q] [N] byte classes on which an item in that DFA state, or waiting for that nonterminal, leaves something

    explicit HostAutomaton(const Tables &t_) : t(t_) {
        blocks.reserve(MAX_BLOCKS);
        q_live.resize(t.Q); nt_live.resize(t.N);
        for (int q = 0; q < t.Q; q++) for (int c = 0; c < t.n_cls; c++) if (t.delta[(size_t)q * t.n_cls + c] != DFA_DEAD) q_live[q].add(c);
        for (int y = 0; y < t.N; y++) for (int c = 0; c < t.n_cls; c++) if (t.scan_off[(size_t)y * t.n_cls + c + 1] > t.scan_off[(size_t)y * t.n_cls + c]) nt_live[y].add(c);
        clear();
    }

    State &st(uint32_t id) { return blocks[id / BLOCK].states[id % BLOCK]; }
    const State &st(uint32_t id) const { return blocks[id / BLOCK].states[id % BLOCK]; }
    // The classes on which some item leaves something: the only ones that can lead anywhere (add).
    Classes live_classes(const Item *items, uint32_t n) const {
        Classes live;
        for (uint32_t i = 0; i < n; i++) {
            const uint16_t code = t.sym[items[i].p];
            if ((code >> SYM_KIND_SHIFT) == SYM_TERM) live.add(q_live[items[i].q]);
            else if ((code >> SYM_KIND_SHIFT) == SYM_NT) live.add(nt_live[code & SYM_ID_MASK_NT]);
        }
        return live;
    }
    // Eight words of a state's transitions for eight bits of its live classes.
    struct Unknown {
        uint32_t words[256][8];
        Unknown() { for (int b = 0; b < 256; b++) for (int k = 0; k < 8; k++) words[b][k] = (b >> k) & 1 ? NONE : DEAD; }
    };
    static const Unknown &unknown() { static const Unknown u; return u; }
    static constexpr uint32_t IMPORT_SETS_MAX = 1u << 16;          // the largest chart import takes
    bool full() const { return n_states + IMPORT_SETS_MAX + 2 >= BLOCK * MAX_BLOCKS; }   // no room for another import

    uint32_t add(const Item *items, uint32_t n, uint32_t widest, uint32_t sig) {
        const uint32_t id = n_states;
        if (id / BLOCK >= blocks.size())
            blocks.push_back(Block{std::unique_ptr<State[]>(new State[BLOCK]), std::unique_ptr<uint32_t[]>(new uint32_t[(size_t)BLOCK * t.n_cls]), std::unique_ptr<uint8_t[]>(new uint8_t[(size_t)BLOCK * t.n_cls])});
        if (n > ITEM_CHUNK - chunk_used || chunks.empty()) { chunks.emplace_back(new Item[std::max(n, ITEM_CHUNK)]); chunk_used = 0; }
        Item *to = chunks.back().get() + chunk_used;
        std::copy(items, items + n, to);
        chunk_used = n > ITEM_CHUNK - chunk_used ? ITEM_CHUNK : chunk_used + n;
        Block &b = blocks[id / BLOCK];
        State &s = st(id);
        s.items = to; s.n_items = n;
        s.widest = widest; s.sig = sig;
        s.trans = b.trans.get() + (size_t)(id % BLOCK) * t.n_cls;
        s.acc = b.acc.get() + (size_t)(id % BLOCK) * t.n_cls;
        // a class on which no item leaves anything needs no step to be known as a dead end
        const Classes live = live_classes(to, n);
        const Unknown &u = unknown();
        int c = 0;
        for (; c + 8 <= t.n_cls; c += 8) memcpy(s.trans + c, u.words[(live.w[c >> 6] >> (c & 63)) & 0xFF], 32);
        for (; c < t.n_cls; c++) s.trans[c] = live.has(c) ? NONE : DEAD;
        memset(s.acc, 0, (size_t)t.n_cls);
        n_states++;
        return id;
    }

    void clear() {
        blocks.clear();
        chunks.clear(); chunk_used = ITEM_CHUNK;
        interned.assign(1u << 12, 0);
        n_states = 0; n_items = 0;
        add(nullptr, 0, 0, 0);                                 // id 0 is not used
        Chart c;
        chart_init(t, c);
        std::vector<Item> root;
        for (Item it : c.items) {                              // the closure of the start item; its items started in this very set
            if ((t.sym[it.p] >> SYM_KIND_SHIFT) == SYM_END) continue;
            it.o = ROOT;
            root.push_back(it);
        }
        add(root.data(), (uint32_t)root.size(), (uint32_t)root.size(), 0);
    }

    // A transition in two parts, so that callers that share the automaton can run the Earley byte step (Scan and Complete
    // with tabulated Predict, as earley_step does over a chart) without holding the lock: look_ahead reads the state and the
    // sets it refers to, by their names, and leaves the new set in w; record writes it down.
    struct Work {
        std::vector<Item> set;
        bool alive = false, accepted = false;
        std::vector<uint32_t> seen;       // sets of more than a few items find duplicates by hashing: item number + 1, 0 = free
        static constexpr size_t FEW = 16;
        static uint32_t hash(const Item &it) { uint32_t h = ((uint32_t)it.p | (uint32_t)it.q << 16) * 0x9E3779B1u ^ it.o * 0x85EBCA77u; h ^= h >> 15; h *= 0x2C1B3C6Du; return h ^ h >> 13; }
        static bool same(const Item &a, const Item &b) { return a.p == b.p && a.q == b.q && a.o == b.o; }
        void insert(const Item &it) {     // a set holds each item once (Section 3.2)
            if (set.size() <= FEW) {
                for (const Item &x : set) if (same(x, it)) return;
                set.push_back(it);
                if (set.size() > FEW) rehash(64);
                return;
            }
            uint32_t k = hash(it) & (uint32_t)(seen.size() - 1);
            for (; seen[k]; k = (k + 1) & (uint32_t)(seen.size() - 1)) if (same(set[seen[k] - 1], it)) return;
            set.push_back(it);
            seen[k] = (uint32_t)set.size();
            if (2 * set.size() > seen.size()) rehash(2 * seen.size());
        }
        void rehash(size_t room) {
            seen.assign(room, 0);
            for (size_t i = 0; i < set.size(); i++) {
                uint32_t k = hash(set[i]) & (uint32_t)(room - 1);
                while (seen[k]) k = (k + 1) & (uint32_t)(room - 1);
                seen[k] = (uint32_t)i + 1;
            }
        }
    };
    // The dot arrives at position p (origin o): a nullable postdot nonterminal is also skipped, the end of the rule is the
    // canonical "lhs complete since o" item.
    void advanced(Work &w, uint32_t p, uint32_t o) const {
        for (;; p++) {
            const uint16_t code = t.sym[p];
            const int kind = code >> SYM_KIND_SHIFT;
            if (kind == SYM_END) { w.insert(Item{t.end_pos[code & SYM_ID_MASK], 0, o}); return; }
            if (kind == SYM_TERM) { w.insert(Item{(uint16_t)p, t.term_start[code & SYM_ID_MASK], o}); return; }
            w.insert(Item{(uint16_t)p, 0, o});
            if (!(code & SYM_NULLABLE_BIT)) return;
        }
    }
    void look_ahead(uint32_t s, int cl, Work &w) const {
        scan(s, cl, s, w);
        close(w);
    }
    void scan(uint32_t s, int cl, uint32_t begun, Work &w) const { scan(s, cl, [&](uint32_t) { return begun; }, w); }
    template <class Begun>
    void scan(uint32_t s, int cl, Begun begun_for, Work &w) const {   // begun_for(Y): the set that rules begun by this byte, for an item that waits for Y, are said to start in
        w.set.clear();
        const State &src = st(s);
        for (uint32_t i = 0; i < src.n_items; i++) {           // Scan
            const Item it = src.items[i];
            const uint16_t code = t.sym[it.p];
            if ((code >> SYM_KIND_SHIFT) == SYM_TERM) {
                const uint16_t q2 = t.delta[(size_t)it.q * t.n_cls + cl];
                if (q2 == DFA_DEAD) continue;
                const uint8_t f = t.qflags[q2];
                if (f & QF_CONT) w.insert(Item{it.p, q2, it.o});
                if (f & QF_ACCEPT) advanced(w, it.p + 1u, it.o);
            } else if ((code >> SYM_KIND_SHIFT) == SYM_NT) {
                const size_t at = (size_t)(code & SYM_ID_MASK_NT) * t.n_cls + cl;
                const uint32_t begun = begun_for((uint32_t)(code & SYM_ID_MASK_NT));
                for (uint32_t k = t.scan_off[at]; k < t.scan_off[at + 1]; k++) {
                    const uint16_t p0 = t.scan_list[k] & 0xFFFF, q2 = t.scan_list[k] >> 16;
                    const uint8_t f = t.qflags[q2];
                    if (f & QF_CONT) w.insert(Item{p0, q2, begun});
                    if (f & QF_ACCEPT) advanced(w, p0 + 1u, begun);
                }
            }
        }
    }
    void close(Work &w) const {
        w.accepted = false;
        for (size_t i = 0; i < w.set.size(); i++) {            // Complete (the set grows on the way)
            const Item it = w.set[i];
            const uint16_t code = t.sym[it.p];
            if ((code >> SYM_KIND_SHIFT) != SYM_END) continue;
            const int X = code & SYM_ID_MASK;
            if (X == t.N - 1) { w.accepted = true; continue; }
            completed(w, it, (uint32_t)X);
        }
        drop_completed(w);
    }
    void completed(Work &w, const Item it, uint32_t X) const {   // it: "X is complete"
        const State &org = st(it.o);
        for (uint32_t j = 0; j < org.n_items; j++) {
            const Item y = org.items[j];
            const uint16_t yc = t.sym[y.p];
            if ((yc >> SYM_KIND_SHIFT) != SYM_NT) continue;
            const size_t at = (size_t)(yc & SYM_ID_MASK_NT) * t.N + X;
            for (uint32_t k = t.comp_off[at]; k < t.comp_off[at + 1]; k++) {
                const uint16_t p = t.comp_list[k];
                if (p == COMP_ADVANCE_WAITING) advanced(w, y.p + 1u, y.o);
                else w.insert(Item{p, (t.sym[p] >> SYM_KIND_SHIFT) == SYM_TERM ? t.term_start[t.sym[p] & SYM_ID_MASK] : (uint16_t)0, it.o});
            }
        }
    }
    void drop_completed(Work &w) const {
        w.alive = !w.set.empty();
        size_t n = 0;                                          // completed items only matter while their own set is worked on (Figure 3, first rule)
        for (const Item &it : w.set) if ((t.sym[it.p] >> SYM_KIND_SHIFT) != SYM_END) w.set[n++] = it;
        w.set.resize(n);
    }
    void record(uint32_t s, int cl, const Work &w) {
        record(s, cl, !w.alive ? DEAD : w.set.empty() ? SINK : intern(w.set.data(), (uint32_t)w.set.size()), w.accepted);
    }
    void record(uint32_t s, int cl, uint32_t to, bool accepted) {
        n_steps++;
        st(s).acc[cl] = accepted;
        st(s).trans[cl] = to;
    }

    // What Complete makes of a set is a function of what Scan has left in it, and an exploration meets the same again and again: a number goes on, a string
    // goes on, a word may end here or there.  So it keeps, by what Scan has left, where Complete led (while the automaton is not emptied): 70,000 of the 84,000 steps of
    // a JSON schema complete something, 16,500 of them something new (18.0 -> 13.2 ms on a slow host).  Sets that nothing is complete in are looked up as they are (intern).
    struct Completed {
        struct Entry { uint32_t at, n, to; bool accepted; };
        std::vector<Entry> entries;
        std::vector<Item> items;
        std::vector<uint64_t> places = std::vector<uint64_t>(1u << 12, 0);   // open addressing, at most half full: signature << 32 | entry + 1; 0 = free
        const Entry *find(const std::vector<Item> &set, uint32_t &sig) const {
            sig = signature(set.data(), (uint32_t)set.size());
            for (uint32_t k = sig & (uint32_t)(places.size() - 1); places[k]; k = (k + 1) & (uint32_t)(places.size() - 1)) {
                if ((uint32_t)(places[k] >> 32) != sig) continue;
                const Entry &e = entries[(uint32_t)places[k] - 1u];
                if (e.n == set.size() && std::equal(set.begin(), set.end(), items.begin() + e.at, Work::same)) return &e;
            }
            return nullptr;
        }
        void add(const std::vector<Item> &set, uint32_t sig, uint32_t to, bool accepted) {
            entries.push_back(Entry{(uint32_t)items.size(), (uint32_t)set.size(), to, accepted});
            items.insert(items.end(), set.begin(), set.end());
            put(places, (uint64_t)sig << 32 | entries.size());
            if (2 * entries.size() <= places.size()) return;
            std::vector<uint64_t> old(2 * places.size(), 0);
            old.swap(places);
            for (uint64_t e : old) if (e) put(places, e);
        }
    };
    bool completes(const Work &w) const {
        for (const Item &it : w.set) if ((t.sym[it.p] >> SYM_KIND_SHIFT) == SYM_END) return true;
        return false;
    }
    static uint32_t signature(const Item *items, uint32_t n) {
        uint32_t h = n;
        for (uint32_t i = 0; i < n; i++) h = (h ^ Work::hash(items[i])) * 0x01000193u + (h >> 13);
        return h;
    }
    static void put(std::vector<uint64_t> &places, uint64_t e) {   // into a table that has room
        uint32_t k = (uint32_t)(e >> 32) & (uint32_t)(places.size() - 1);
        while (places[k]) k = (k + 1) & (uint32_t)(places.size() - 1);
        places[k] = e;
    }

    // The state that holds exactly `items` (origins are state ids), made if it is new.
    uint32_t intern(const Item *items, uint32_t n) {
        const uint32_t h = signature(items, n);
        uint32_t k = h & (uint32_t)(interned.size() - 1);
        for (; interned[k]; k = (k + 1) & (uint32_t)(interned.size() - 1)) {
            if ((uint32_t)(interned[k] >> 32) != h) continue;
            const State &x = st((uint32_t)interned[k]);
            if (x.n_items == n && std::equal(items, items + n, x.items, Work::same)) return (uint32_t)interned[k];
        }
        n_items += n;
        uint32_t w = n;
        for (uint32_t i = 0; i < n; i++) w = std::max(w, st(items[i].o).widest);
        const uint32_t id = add(items, n, w, h);
        interned[k] = (uint64_t)h << 32 | id;
        if (2 * (size_t)n_states > interned.size()) {
            std::vector<uint64_t> old(2 * interned.size(), 0);
            old.swap(interned);
            for (uint64_t e : old) if (e) put(interned, e);
        }
        return id;
    }

    void compute(uint32_t s, int cl, Work &w) {
        look_ahead(s, cl, w);
        record(s, cl, w);
    }

    // One byte from state s; returns the next state, SINK or DEAD.
    uint32_t step(uint32_t s, uint8_t byte, bool *accepted) {
        if (s == SINK) { if (accepted) *accepted = false; return DEAD; }
        const int cl = t.cls[byte];
        static thread_local Work w;
        if (st(s).trans[cl] == NONE) compute(s, cl, w);
        if (accepted) *accepted = st(s).acc[cl] != 0;
        return st(s).trans[cl];
    }

    // The state of a chart's current set: every set of the chart becomes a state (found by content when it is
    // there already), origins renamed from set indices to state names.  The chart's first set is the set of the
    // empty prefix (everything refers back to it).  A chart whose current set is empty of items stands at SINK.
    uint32_t import(const Chart &c) {
        if (full() || c.n_sets() > IMPORT_SETS_MAX) return 0;       // no room: the caller empties the automaton, or fails
        std::vector<uint32_t> name(c.n_sets(), ROOT);
        for (uint32_t k = 1; k < c.n_sets(); k++) {
            std::vector<Item> items(c.items.begin() + c.set_off[k], c.items.begin() + c.set_off[k + 1]);
            if (items.empty()) { name[k] = SINK; continue; }
            for (Item &it : items) it.o = it.o < k ? name[it.o] : ROOT;
            name[k] = intern(items.data(), (uint32_t)items.size());
        }
        return name[c.n_sets() - 1];
    }
};

}  // namespace zf
