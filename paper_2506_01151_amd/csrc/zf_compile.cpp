// Grammar compiler: grammar clean-up (paper Section 4.5: useless rules, nullable symbols),
// per-terminal DFAs merged into one state numbering with byte equivalence classes (Section
// 4.1), the look-up tables that replace explicit Predict items, and the flattened
// vocabulary trie.
//
// Table-driven Earley used throughout the library.  Only items that have consumed at least
// one byte ("kernel" items) are stored in a set.  Everything Predict would add to a set is a
// function of the postdot nonterminals of its kernel items, so it is tabulated once:
//   PRED(Y)  = nonterminals that can start a derivation of Y (left corners, skipping nullable
//              prefixes), Y included;
//   I(Y)     = dotted positions (Z -> alpha . beta) with Z in PRED(Y) and alpha nullable;
//   SCAN(Y,c)= for positions of I(Y) that stand before a terminal t: (position, delta_t(start, c))
//              for every byte class c the terminal can start with;
//   COMP(Y,X)= what the completion of X does to the predicted items of I(Y): the positions that
//              stand behind X in I(Y), with nullable symbols skipped -- and, where such a
//              position is the end of its rule, its left-hand side counts as completed too (same
//              origin, the set that predicted it) and is followed up here, at compile time.  The
//              list holds the resulting items and, if Y itself is among the completed
//              nonterminals, a marker that tells the recognizer to advance the waiting item.
// Nullable nonterminals are handled when an item is added: the item is also added with the dot
// moved over the nullable symbol (Aycock-Horspool), so no epsilon rule survives at run time.
#include <algorithm>
#include <cstring>
#include <map>
#include <set>
#include "zf_internal.h"
#include "zf_host_automaton.h"

namespace zf {

bool build_tables(const zf_grammar_desc *g, Tables &t) {
    if (!g || g->n_nonterminals <= 0 || g->n_rules < 0 || g->n_terminals < 0 || g->start < 0 ||
        g->start >= g->n_nonterminals || (g->n_rules && (!g->rule_lhs || !g->rhs_off)) ||
        (g->n_terminals && (!g->term_kind || !g->term_off))) {
        set_error("grammar: bad sizes or null arrays");
        return false;
    }
    const int NT0 = g->n_nonterminals, R0 = g->n_rules, T = g->n_terminals;
    for (int r = 0; r < R0; r++) {
        if (g->rule_lhs[r] < 0 || g->rule_lhs[r] >= NT0 || g->rhs_off[r + 1] < g->rhs_off[r]) { set_error("grammar: bad rule " + std::to_string(r)); return false; }
        for (int k = g->rhs_off[r]; k < g->rhs_off[r + 1]; k++) {
            int s = g->rhs_sym[k];
            if ((s >= 0 && s >= NT0) || (s < 0 && ~s >= T)) { set_error("grammar: bad symbol in rule " + std::to_string(r)); return false; }
        }
    }
    // ---- terminals -> DFAs ----
    std::vector<Dfa> dfas(T);
    for (int k = 0; k < T; k++) {
        const uint8_t *src = g->term_data + g->term_off[k];
        size_t n = (size_t)(g->term_off[k + 1] - g->term_off[k]);
        if (g->term_kind[k] == 0) literal_to_dfa(src, n, dfas[k]);
        else if (g->term_kind[k] == 1) { if (!regex_to_dfa(src, n, dfas[k])) return false; }
        else { set_error("grammar: bad terminal kind"); return false; }
        if (dfas[k].accept[0]) { set_error("grammar: terminal " + std::to_string(k) + " matches the empty string; make it optional in a rule instead"); return false; }
        bool any = false;
        for (int b = 0; b < 256; b++) any |= dfas[k].trans[b] >= 0;
        if (!any) { set_error("grammar: terminal " + std::to_string(k) + " has an empty language"); return false; }
    }
    // ---- useless-rule removal: productive, then reachable ----
    std::vector<uint8_t> productive(NT0, 0), reachable(NT0, 0);
    for (bool ch = true; ch;) {
        ch = false;
        for (int r = 0; r < R0; r++) {
            if (productive[g->rule_lhs[r]]) continue;
            bool all = true;
            for (int k = g->rhs_off[r]; k < g->rhs_off[r + 1] && all; k++) { int s = g->rhs_sym[k]; if (s >= 0 && !productive[s]) all = false; }
            if (all) { productive[g->rule_lhs[r]] = 1; ch = true; }
        }
    }
    if (!productive[g->start]) { set_error("grammar: the start symbol derives no string"); return false; }
    auto rule_ok = [&](int r) {
        if (!productive[g->rule_lhs[r]]) return false;
        for (int k = g->rhs_off[r]; k < g->rhs_off[r + 1]; k++) { int s = g->rhs_sym[k]; if (s >= 0 && !productive[s]) return false; }
        return true;
    };
    reachable[g->start] = 1;
    for (bool ch = true; ch;) {
        ch = false;
        for (int r = 0; r < R0; r++) if (rule_ok(r) && reachable[g->rule_lhs[r]])
            for (int k = g->rhs_off[r]; k < g->rhs_off[r + 1]; k++) { int s = g->rhs_sym[k]; if (s >= 0 && !reachable[s]) { reachable[s] = 1; ch = true; } }
    }
    std::vector<int> nt_new(NT0, -1);
    int N = 0;
    for (int a = 0; a < NT0; a++) if (productive[a] && reachable[a]) nt_new[a] = N++;
    const int SP = N++;   // the added start symbol S'
    if (N > (int)SYM_ID_MASK_NT) { set_error("grammar: too many nonterminals"); return false; }
    if (T > (int)SYM_ID_MASK) { set_error("grammar: too many terminals"); return false; }
    struct Rule { int lhs, orig; std::vector<int> rhs; };   // rhs: >=0 new nonterminal id, <0 terminal
    std::vector<Rule> rules;
    for (int r = 0; r < R0; r++) if (rule_ok(r) && reachable[g->rule_lhs[r]]) {
        Rule x{nt_new[g->rule_lhs[r]], r, {}};
        for (int k = g->rhs_off[r]; k < g->rhs_off[r + 1]; k++) { int s = g->rhs_sym[k]; x.rhs.push_back(s >= 0 ? nt_new[s] : s); }
        rules.push_back(x);
    }
    rules.push_back(Rule{SP, -1, {nt_new[g->start]}});
    t.n_rules_kept = (int)rules.size() - 1;
    t.operators = std::any_of(rules.begin(), rules.end(), [](const Rule &r) { return r.rhs.size() > 1 && r.rhs.front() == r.lhs && r.rhs.back() == r.lhs; });
    // ---- nullable ----
    std::vector<uint8_t> nullable(N, 0);
    for (bool ch = true; ch;) {
        ch = false;
        for (auto &r : rules) if (!nullable[r.lhs]) {
            bool all = true;
            for (int s : r.rhs) if (s < 0 || !nullable[s]) { all = false; break; }
            if (all) { nullable[r.lhs] = 1; ch = true; }
        }
    }
    // ---- terminals actually used; merge DFAs into one numbering; byte classes ----
    t.T = T;
    t.term_start.assign(T, 0);
    std::vector<int> base(T, 0);
    int Q = 0;
    for (int k = 0; k < T; k++) { base[k] = Q; Q += dfas[k].n_states(); }
    if (Q >= (int)DFA_DEAD) { set_error("grammar: too many DFA states"); return false; }
    t.Q = Q;
    {   // two bytes are equivalent when every state of every DFA treats them alike
        std::map<std::vector<int32_t>, int> col_ix;
        for (int b = 0; b < 256; b++) {
            std::vector<int32_t> col;
            col.reserve(Q);
            for (int k = 0; k < T; k++) for (int s = 0; s < dfas[k].n_states(); s++) col.push_back(dfas[k].trans[s * 256 + b]);
            auto it = col_ix.find(col);
            if (it == col_ix.end()) it = col_ix.emplace(col, (int)col_ix.size()).first;
            t.cls[b] = (uint8_t)it->second;
        }
        t.n_cls = (int)col_ix.size();
    }
    t.delta.assign((size_t)Q * t.n_cls, DFA_DEAD);
    t.qflags.assign(Q, 0);
    for (int k = 0; k < T; k++) {
        t.term_start[k] = (uint16_t)base[k];
        for (int s = 0; s < dfas[k].n_states(); s++) {
            bool cont = false;
            for (int b = 0; b < 256; b++) {
                int to = dfas[k].trans[s * 256 + b];
                if (to >= 0) { t.delta[(size_t)(base[k] + s) * t.n_cls + t.cls[b]] = (uint16_t)(base[k] + to); cont = true; }
            }
            t.qflags[base[k] + s] = (dfas[k].accept[s] ? QF_ACCEPT : 0) | (cont ? QF_CONT : 0);
        }
    }
    // ---- dotted positions ----
    t.N = N;
    t.sym.clear(); t.lhs_of.clear(); t.pos_rule.clear(); t.pos_dot.clear(); t.pos_lhs_orig.clear();
    std::vector<int> rule_base(rules.size());
    std::vector<int> orig_of_new(N, -1);
    for (int a = 0; a < NT0; a++) if (nt_new[a] >= 0) orig_of_new[nt_new[a]] = a;
    for (size_t r = 0; r < rules.size(); r++) {
        rule_base[r] = (int)t.sym.size();
        for (size_t d = 0; d <= rules[r].rhs.size(); d++) {
            uint16_t code;
            if (d == rules[r].rhs.size()) code = (uint16_t)((SYM_END << SYM_KIND_SHIFT) | rules[r].lhs);
            else if (rules[r].rhs[d] < 0) code = (uint16_t)((SYM_TERM << SYM_KIND_SHIFT) | (~rules[r].rhs[d]));
            else code = (uint16_t)((SYM_NT << SYM_KIND_SHIFT) | rules[r].rhs[d] | (nullable[rules[r].rhs[d]] ? SYM_NULLABLE_BIT : 0));
            t.sym.push_back(code);
            t.lhs_of.push_back((uint16_t)rules[r].lhs);
            t.pos_rule.push_back(rules[r].orig); t.pos_dot.push_back((int)d); t.pos_lhs_orig.push_back(orig_of_new[rules[r].lhs]);
        }
    }
    t.start_pos = rule_base.back();
    t.end_pos.assign(N, 0);
    for (int a = 0; a < N; a++) {   // one canonical "X is complete" position per nonterminal
        t.end_pos[a] = (uint16_t)t.sym.size();
        t.sym.push_back((uint16_t)((SYM_END << SYM_KIND_SHIFT) | a));
        t.lhs_of.push_back((uint16_t)a);
        t.pos_rule.push_back(-1); t.pos_dot.push_back(-1); t.pos_lhs_orig.push_back(orig_of_new[a]);
    }
    t.P = (int)t.sym.size();
    if (t.P > (int)MAX_POSITIONS) { set_error("grammar: too many dotted positions"); return false; }
    t.end_base = t.end_pos[0];
    t.advpq.assign(t.P, 0);
    for (int p = 0; p < t.P; p++) {
        uint16_t code = t.sym[p];
        int k = code >> SYM_KIND_SHIFT;
        if (k == SYM_END) t.advpq[p] = (uint32_t)t.end_pos[code & SYM_ID_MASK] | IW_END;
        else if (k == SYM_TERM) t.advpq[p] = (uint32_t)p | IW_TERM | ((uint32_t)t.term_start[code & SYM_ID_MASK] << 16);
        else t.advpq[p] = (uint32_t)p | ((code & SYM_NULLABLE_BIT) ? (uint32_t)IW_NT_NULLABLE : 0u) | ((uint32_t)(code & SYM_ID_MASK_NT) << IW_NT_SHIFT);
    }
    // hybrid DFA encoding for the device: literal chains carry their byte, other states a dense row
    t.qinfo.assign(Q, 0);
    t.delta_dense.clear();
    for (int k = 0; k < T; k++) {
        const bool lit = g->term_kind[k] == 0;
        for (int s = 0; s < dfas[k].n_states(); s++) {
            int q = base[k] + s;
            uint32_t info = t.qflags[q];
            if (lit) {
                int b = 0;
                for (int x = 0; x < 256; x++) if (dfas[k].trans[s * 256 + x] >= 0) b = x;
                info |= QF_LITERAL | ((uint32_t)b << 8);
                if (s + 1 < dfas[k].n_states()) info |= (uint32_t)t.qflags[q + 1] << 16;
            } else {
                uint32_t row = (uint32_t)(t.delta_dense.size() / t.n_cls);
                for (int c = 0; c < t.n_cls; c++) {
                    uint16_t to = t.delta[(size_t)q * t.n_cls + c];
                    t.delta_dense.push_back(to == DFA_DEAD ? (uint32_t)DFA_DEAD : ((uint32_t)to | ((uint32_t)t.qflags[to] << 16)));
                }
                info |= row << 16;
            }
            t.qinfo[q] = info;
        }
    }
    // ---- PRED / I / SCAN / COMP ----
    // lead[Z] = positions of Z's rules reachable from the rule start over nullable symbols
    std::vector<std::vector<int>> lead(N);
    for (size_t r = 0; r < rules.size(); r++)
        for (size_t d = 0; d < rules[r].rhs.size(); d++) {
            lead[rules[r].lhs].push_back(rule_base[r] + (int)d);
            int s = rules[r].rhs[d];
            if (s < 0 || !nullable[s]) break;
        }
    t.reach.assign((size_t)N * N, 0);
    t.first_terms.assign(N, {});
    t.scan_off.assign((size_t)N * t.n_cls + 1, 0);
    t.comp_off.assign((size_t)N * N + 1, 0);
    t.scan_list.clear(); t.comp_list.clear();
    std::vector<std::vector<std::vector<uint32_t>>> scan_tmp(N, std::vector<std::vector<uint32_t>>(t.n_cls));
    std::vector<std::vector<std::vector<uint16_t>>> comp_tmp(N, std::vector<std::vector<uint16_t>>(N));
    for (int Y = 0; Y < N; Y++) {
        std::vector<int> stack{Y};
        t.reach[(size_t)Y * N + Y] = 1;
        std::vector<int> I;
        while (!stack.empty()) {
            int Z = stack.back(); stack.pop_back();
            for (int p : lead[Z]) {
                I.push_back(p);
                uint16_t code = t.sym[p];
                if ((code >> SYM_KIND_SHIFT) == SYM_NT) {
                    int X = code & SYM_ID_MASK_NT;
                    if (!t.reach[(size_t)Y * N + X]) { t.reach[(size_t)Y * N + X] = 1; stack.push_back(X); }
                }
            }
        }
        std::sort(I.begin(), I.end());
        for (int p : I) {
            uint16_t code = t.sym[p];
            if ((code >> SYM_KIND_SHIFT) == SYM_TERM) {
                int term = code & SYM_ID_MASK;
                if (std::find(t.first_terms[Y].begin(), t.first_terms[Y].end(), (uint16_t)term) == t.first_terms[Y].end())
                    t.first_terms[Y].push_back((uint16_t)term);
                for (int c = 0; c < t.n_cls; c++) {
                    uint16_t to = t.delta[(size_t)t.term_start[term] * t.n_cls + c];
                    if (to != DFA_DEAD) scan_tmp[Y][c].push_back((uint32_t)p | ((uint32_t)to << 16));
                }
            } else if ((code >> SYM_KIND_SHIFT) == SYM_NT) {
                comp_tmp[Y][code & SYM_ID_MASK_NT].push_back((uint16_t)(p + 1));
            }
        }
    }
    for (int Y = 0; Y < N; Y++) for (int c = 0; c < t.n_cls; c++) {
        t.scan_off[(size_t)Y * t.n_cls + c] = (uint32_t)t.scan_list.size();
        t.scan_list.insert(t.scan_list.end(), scan_tmp[Y][c].begin(), scan_tmp[Y][c].end());
    }
    t.scan_off[(size_t)N * t.n_cls] = (uint32_t)t.scan_list.size();
    for (int Y = 0; Y < N; Y++) for (int X = 0; X < N; X++) {
        t.comp_off[(size_t)Y * N + X] = (uint32_t)t.comp_list.size();
        if (!t.reach[(size_t)Y * N + X]) continue;       // no item predicted by Y waits for X or for anything X leads to
        std::vector<uint8_t> completed(N, 0);
        std::vector<int> work{X};
        std::vector<uint16_t> out;
        completed[X] = 1;
        bool y_completes = false;
        while (!work.empty()) {
            const int C = work.back(); work.pop_back();
            if (C == Y) y_completes = true;
            for (uint16_t p1 : comp_tmp[Y][C]) {
                for (int p = p1;; p++) {                   // the dot arrives at p: same walk as the recognizer's add step
                    const uint16_t code = t.sym[p];
                    const int k = code >> SYM_KIND_SHIFT;
                    if (k == SYM_END) { const int L = code & SYM_ID_MASK; if (!completed[L]) { completed[L] = 1; work.push_back(L); } break; }
                    if (std::find(out.begin(), out.end(), (uint16_t)p) == out.end()) out.push_back((uint16_t)p);
                    if (k == SYM_TERM || !(code & SYM_NULLABLE_BIT)) break;
                }
            }
        }
        std::sort(out.begin(), out.end());
        t.comp_list.insert(t.comp_list.end(), out.begin(), out.end());
        if (y_completes) t.comp_list.push_back(COMP_ADVANCE_WAITING);
    }
    t.comp_off[(size_t)N * N] = (uint32_t)t.comp_list.size();
    t.dev_comp_list.resize(t.comp_list.size());
    for (size_t k = 0; k < t.comp_list.size(); k++)
        t.dev_comp_list[k] = t.comp_list[k] == COMP_ADVANCE_WAITING ? 0xFFFFFFFFu : t.advpq[t.comp_list[k]];
    t.dev_scan_list.resize(2 * t.scan_list.size());
    for (size_t k = 0; k < t.scan_list.size(); k++) {
        t.dev_scan_list[2 * k] = t.scan_list[k] | IW_TERM;
        t.dev_scan_list[2 * k + 1] = t.qflags[t.scan_list[k] >> 16];
    }
    return true;
}

// ---- vocabulary -> flattened prefix trie ---------------------------------------------------
void build_trie(const zf_vocab_desc *v, int CHUNK_RANKS, const uint8_t *cls, Trie &t) {
    t.chunk_ranks = CHUNK_RANKS;
    const int V = v->V;
    // Sorted by their bytes, then by their numbers: dealt to 256 buckets by the first byte, each sorted by the next eight bytes as
    // one number; only strings that agree in these are compared byte by byte.  The buckets are independent.
    auto tok = [&](int i, const uint8_t *&p, size_t &n) { p = v->bytes + v->off[i]; n = (size_t)(v->off[i + 1] - v->off[i]); };
    // So are the subtrees that they make: how many nodes, strings and bytes a bucket has is counted where it is sorted, and the buckets are then written side by
    // side (a schema with 128,256 tokens, 67,435 of them distinct strings: 6.7 ms with the nodes made one after the other, 2.5 so; the whole compile, with the exploration
    // by what Scan has left, 14.2 -> 10.5 ms).
    struct Key { uint64_t next; int id; uint32_t common; };   // common: leading bytes that the distinct string before has as well; SAME: it is that string
    static const uint32_t SAME = 0xFFFFFFFFu;
    std::vector<uint32_t> bucket(257, 0);
    for (int i = 0; i < V; i++) if (v->off[i + 1] > v->off[i]) bucket[v->bytes[v->off[i]] + 1u]++;
    for (int b = 0; b < 256; b++) bucket[b + 1] += bucket[b];
    std::vector<Key> order(bucket[256]);
    {
        std::vector<uint32_t> at(bucket.begin(), bucket.end() - 1);
        for (int i = 0; i < V; i++) {
            const uint8_t *p; size_t n;
            tok(i, p, n);
            if (n == 0) continue;
            uint64_t next = 0;
            for (size_t k = 1; k <= 8; k++) next = next << 8 | (k < n ? p[k] : 0u);
            order[at[p[0]]++] = Key{next, i, 0};
        }
    }
    const unsigned threads = order.size() >= 8192 ? 8 : 1;
    struct Sizes { uint32_t nodes, strings, bytes; };
    std::vector<Sizes> from(257, Sizes{0, 0, 0});             // what the buckets before have
    parallel_for(256, threads, [&](size_t b) {
        std::sort(order.begin() + bucket[b], order.begin() + bucket[b + 1], [&](const Key &a, const Key &c) {
            if (a.next != c.next) return a.next < c.next;
            const uint8_t *pa, *pb; size_t na, nb;
            tok(a.id, pa, na); tok(c.id, pb, nb);
            const int r = memcmp(pa, pb, std::min(na, nb));
            if (r) return r < 0;
            if (na != nb) return na < nb;
            return a.id < c.id;
        });
        Sizes has{0, 0, 0};
        const uint8_t *prev = nullptr; size_t prev_n = 0;
        for (uint32_t i = bucket[b]; i < bucket[b + 1]; i++) {
            const uint8_t *p; size_t n, common = 0;
            tok(order[i].id, p, n);
            while (common < prev_n && common < n && prev[common] == p[common]) common++;
            order[i].common = prev && common == n && common == prev_n ? SAME : (uint32_t)common;
            if (order[i].common == SAME) continue;
            has.nodes += (uint32_t)(n - common); has.strings++; has.bytes += (uint32_t)n;
            prev = p; prev_n = n;
        }
        from[b + 1] = has;
    });
    for (int b = 0; b < 256; b++) { from[b + 1].nodes += from[b].nodes; from[b + 1].strings += from[b].strings; from[b + 1].bytes += from[b].bytes; }
    const Sizes all = from[256];
    const uint32_t n_chunks = (all.strings + (uint32_t)CHUNK_RANKS - 1u) / (uint32_t)CHUNK_RANKS;
    t.n_strings = (int)all.strings;
    t.nodes.resize(all.nodes); t.parent.resize(all.nodes); t.rank_of.assign(V, 0xFFFFFFFFu);
    t.str_off.resize((size_t)all.strings + 1); t.str_bytes.resize(all.bytes);
    t.str_off[all.strings] = all.bytes;
    t.chunk_begin.assign(n_chunks, 0); t.chunk_end.assign(n_chunks, 0);
    t.chunk_anc.assign((size_t)n_chunks * CHUNK_ANC, TrieNode{});
    t.Wr = ((int)n_chunks * CHUNK_RANKS + 31) / 32;
    parallel_for(256, threads, [&](size_t b) {
        uint32_t node = from[b].nodes, rank = from[b].strings, byte = from[b].bytes, depth = 0;
        uint32_t path[MAX_TOKEN_LEN_ON_DEVICE];               // path[d]: the node at depth d + 1 of the current path
        // the subtrees that are left end before the next node: that is where they are skipped to, and its rank tells their strings
        auto leave = [&](uint32_t down_to) { for (; depth > down_to; depth--) { TrieNode &nd = t.nodes[path[depth - 1]]; nd.skip = node; nd.n_sub = rank - nd.rank; } };
        for (uint32_t i = bucket[b]; i < bucket[b + 1]; i++) {
            const int id = order[i].id;
            if (order[i].common == SAME) { t.rank_of[id] = rank - 1; continue; }
            const uint8_t *p; size_t n;
            tok(id, p, n);
            leave(order[i].common);
            for (; depth < n; depth++) {
                TrieNode &nd = t.nodes[node];
                nd.byte = p[depth]; nd.cls = cls[p[depth]]; nd.depth = (uint8_t)(depth + 1); nd.has_string = depth + 1 == n; nd.rank = rank;
                t.parent[node] = depth == 0 ? 0xFFFFFFFFu : path[depth - 1];
                path[depth] = node++;
            }
            // chunks of CHUNK_RANKS strings: [node that carries rank CHUNK_RANKS c, node that carries the chunk's last rank + 1)
            if (rank % (uint32_t)CHUNK_RANKS == 0) t.chunk_begin[rank / (uint32_t)CHUNK_RANKS] = node - 1;
            if ((rank + 1) % (uint32_t)CHUNK_RANKS == 0 || rank + 1 == all.strings) t.chunk_end[rank / (uint32_t)CHUNK_RANKS] = node;
            memcpy(&t.str_bytes[byte], p, n);
            t.str_off[rank] = byte; byte += (uint32_t)n;
            t.rank_of[id] = rank++;
        }
        leave(0);
        // ancestors of each chunk's first node (top down), for the lanes that start in mid-trie
        for (uint32_t c = (from[b].strings + (uint32_t)CHUNK_RANKS - 1u) / (uint32_t)CHUNK_RANKS; c * (uint32_t)CHUNK_RANKS < rank; c++) {
            uint32_t d = t.nodes[t.chunk_begin[c]].depth;
            for (uint32_t a = t.parent[t.chunk_begin[c]]; a != 0xFFFFFFFFu; a = t.parent[a]) {
                d--;
                if (d <= (uint32_t)CHUNK_ANC) t.chunk_anc[(size_t)c * CHUNK_ANC + d - 1] = t.nodes[a];
            }
        }
    });
}

}  // namespace zf

namespace zf {

// Earley sets behind a terminal whose context is not known: a rule that a string begins itself starts in a set that is known, and completing it leads where it
// leads there; what started before starts in one of a few sets that stand for the unknown ones (`unknown`: begun by an item that waits for nonterminal Y, in the set
// unknown[Y]; complete: what completing X in such a set leads to).  Sets that are known to a depth of DEEPEST, or beyond EXACT_STATES of them, count as unknown,
// so that grammars with recursion have finitely many.  What that leaves undecided in the rows of a cache, of 67,435 strings: JSON 24,767, a schema 16,017, the expression grammar 3,817 with what may follow alone and
// nothing known exactly; with what surely follows 24,106, 15,117 and none; with sets known to a depth of 1 17,208 and 6,287, of 2 16,247 and 5,638, of 3 15,929 and
// 5,606 (and twice the states).
//   What all of it may cost is bounded by what it does: every candidate of Scan and Complete, and every item of an origin set that Complete looks at, is paid for
// before it is looked at (`left`); a step that cannot be paid for is not made, and what is not known then stays open.  A candidate takes 2 to 12 ns.  JSON spends
// 126,000 on what may follow and 82,000 on what surely does, a schema 582,000 and 90,000, the query language 219,000 and 286,000, the expression grammar 9,000 each;
// their cache rows are the same from 200,000 on (with 100,000 the query language leaves 92 of 32,000 tokens open in place of 8).  The budget is 0.5 to 3 ms for either, beside an exploration of 8 ms and more.
// (Bounded by steps, whatever they cost, a value of 500 object types took 1.3 s, a hundred mutually recursive nonterminals 0.15 and four hundred 10.)
struct BehindTerminal {
    static constexpr uint8_t DEEPEST = 2;
    static constexpr uint32_t EXACT_STATES = 256;
    static constexpr size_t BUDGET = 1u << 18, STEP = 32;      // STEP: what a step costs besides: its set is looked up, its transitions are laid out
    const Tables &t;
    HostAutomaton A;
    HostAutomaton::Work w;
    HostAutomaton::Completed done;                             // where Complete led from what Scan has left
    std::vector<Item> scanned;
    std::vector<uint32_t> unknown;
    uint32_t first = 0;                                        // ids below it are unknown sets
    std::vector<uint8_t> depth;                                // [id - first]
    std::vector<uint32_t> arriving;                            // [position] items that the dot's arrival there makes (HostAutomaton::advanced)
    size_t left = BUDGET;
    explicit BehindTerminal(const Tables &t_) : t(t_), A(t_), unknown(t_.N, 0), arriving(t_.P, 1) {
        for (int p = t.P - 2; p >= 0; p--) if ((t.sym[p] >> SYM_KIND_SHIFT) == SYM_NT && (t.sym[p] & SYM_NULLABLE_BIT)) arriving[p] += arriving[p + 1];
    }
    bool spend(size_t n) { if (n > left) { left = 0; return false; } left -= n; return true; }
    uint32_t depth_of(uint32_t id) {                           // how many known sets stand between the set and the unknown ones, itself included
        for (uint32_t s = first + (uint32_t)depth.size(); s < A.n_states; s++) {   // (a set refers to earlier ones only)
            uint8_t d = 0;
            for (uint32_t i = 0; i < A.st(s).n_items; i++) { const uint32_t o = A.st(s).items[i].o; if (o >= first) d = std::max(d, depth[o - first]); }
            depth.push_back((uint8_t)(d + 1));
        }
        return depth[id - first];
    }
    bool spend_scan(uint32_t s, int c) {
        const HostAutomaton::State &src = A.st(s);
        size_t n = STEP;
        for (uint32_t i = 0; i < src.n_items && n <= left; i++) {
            const uint16_t p = src.items[i].p, code = t.sym[p];
            if ((code >> SYM_KIND_SHIFT) == SYM_TERM) n += 1 + arriving[p + 1];
            else if ((code >> SYM_KIND_SHIFT) == SYM_NT) {
                const size_t at = (size_t)(code & SYM_ID_MASK_NT) * t.n_cls + c;
                for (uint32_t k = t.scan_off[at]; k < t.scan_off[at + 1]; k++) n += 1 + arriving[(t.scan_list[k] & 0xFFFF) + 1];
            }
        }
        return spend(n);
    }
    bool spend_completed(const Item &it, uint32_t X) {
        const HostAutomaton::State &org = A.st(it.o);
        size_t n = org.n_items;
        for (uint32_t j = 0; j < org.n_items && n <= left; j++) {
            const uint16_t p = org.items[j].p, code = t.sym[p];
            if ((code >> SYM_KIND_SHIFT) != SYM_NT) continue;
            const size_t at = (size_t)(code & SYM_ID_MASK_NT) * t.N + X;
            n += t.comp_off[at + 1] - t.comp_off[at];
            if (t.comp_off[at + 1] > t.comp_off[at] && t.comp_list[t.comp_off[at + 1] - 1] == COMP_ADVANCE_WAITING) n += arriving[p + 1];
        }
        return spend(n);
    }
    // complete(item, X): what it leads to is in the set, or false: nothing is left to spend
    template <class Complete> bool close(Complete complete) {
        for (size_t i = 0; i < w.set.size(); i++) {
            const Item it = w.set[i];
            const uint16_t code = t.sym[it.p];
            if ((code >> SYM_KIND_SHIFT) != SYM_END || (code & SYM_ID_MASK) == t.N - 1) continue;
            const uint32_t X = code & SYM_ID_MASK;
            if (it.o < first) { if (!complete(it, X)) return false; continue; }
            if (!spend_completed(it, X)) return false;
            A.completed(w, it, X);
        }
        A.drop_completed(w);
        return true;
    }
    uint32_t set() { return !w.alive ? HostAutomaton::DEAD : w.set.empty() ? HostAutomaton::SINK : A.intern(w.set.data(), (uint32_t)w.set.size()); }
    // Behind the terminal at the positions p, in rules that started in the unknown sets begun_for(p); NONE: nothing is left to spend.
    template <class Positions, class Begun, class Complete> uint32_t behind(const Positions &p, Begun begun_for, Complete complete) {
        size_t n = STEP;
        for (uint16_t x : p) n += arriving[x + 1];
        if (!spend(n)) return HostAutomaton::NONE;
        w.set.clear();
        for (uint16_t x : p) A.advanced(w, x + 1u, begun_for(x));
        return close(complete) ? set() : HostAutomaton::NONE;
    }
    template <class Complete> uint32_t step(uint32_t s, int c, Complete complete) {
        if (A.st(s).trans[c] == HostAutomaton::NONE && spend_scan(s, c)) {
            const bool known = A.n_states < first + EXACT_STATES && depth_of(s) <= DEEPEST;
            A.scan(s, c, [&](uint32_t Y) { return known ? s : unknown[Y]; }, w);
            uint32_t sig = 0;
            const bool completes = A.completes(w);
            const HostAutomaton::Completed::Entry *met = completes ? done.find(w.set, sig) : nullptr;
            if (met) A.record(s, c, met->to, false);
            else {
                if (completes) scanned = w.set;
                if (close(complete)) {
                    A.record(s, c, set(), false);
                    if (completes) done.add(scanned, sig, A.st(s).trans[c], false);
                }
            }
        }
        return A.st(s).trans[c];
    }
};
static std::vector<std::vector<uint16_t>> positions_of_terminals(const Tables &t) {
    std::vector<std::vector<uint16_t>> at(t.T);
    for (int p = 0; p < t.P; p++) if ((t.sym[p] >> SYM_KIND_SHIFT) == SYM_TERM) at[t.sym[p] & SYM_ID_MASK].push_back((uint16_t)p);
    return at;
}

// What may follow a terminal, whatever its context: the unknown set waits for everything that the grammar waits for anywhere.  A real set
// is always contained in the set that the same bytes lead to here (by induction over Scan, Complete and Predict), so a string that dies here dies in
// every context.  What the budget does not reach takes everything.
void build_follow(const Tables &t, Follow &f) {
    static const size_t MOST_STATES = 4096;
    BehindTerminal B(t);
    HostAutomaton &A = B.A;
    const uint32_t all = A.n_states;
    std::vector<Item> waiting;
    const std::vector<std::vector<uint16_t>> at = positions_of_terminals(t);
    struct Waits { std::vector<uint16_t> at; size_t arriving = 0; };
    std::vector<Waits> waits(t.N);                             // the positions that wait for a nonterminal: behind them is all that completing it leads to, since what is predicted waits here as well
    for (int p = 0; p < t.P; p++) {
        if ((t.sym[p] >> SYM_KIND_SHIFT) != SYM_NT) continue;
        waiting.push_back(Item{(uint16_t)p, 0, all});
        Waits &x = waits[t.sym[p] & SYM_ID_MASK_NT];
        x.at.push_back((uint16_t)p); x.arriving += B.arriving[p + 1];
    }
    A.add(waiting.data(), (uint32_t)waiting.size(), 0, 0);
    B.unknown.assign(t.N, all);
    const uint32_t first = B.first = A.n_states;
    auto complete = [&](const Item &it, uint32_t X) {
        if (!B.spend(waits[X].arriving)) return false;
        for (uint16_t p : waits[X].at) A.advanced(B.w, p + 1u, it.o);
        return true;
    };
    std::vector<uint32_t> behind(t.T);
    for (int k = 0; k < t.T; k++) behind[k] = B.behind(at[k], [&](uint16_t) { return all; }, complete);
    for (uint32_t s = first; s < A.n_states && B.left; s++)
        for (int c = 0; c < t.n_cls && B.left; c++)
            if (A.st(s).trans[c] == HostAutomaton::NONE && A.n_states <= first + MOST_STATES) B.step(s, c, complete);
    const uint32_t sink = A.n_states - first + 1;              // a finished sentence: nothing follows
    auto name = [&](uint32_t s) -> uint16_t { return s == HostAutomaton::DEAD ? FOLLOW_DEAD : s == HostAutomaton::SINK ? (uint16_t)sink : s == HostAutomaton::NONE ? FOLLOW_ANY : (uint16_t)(s - first + 1); };
    f.behind.assign(t.Q, FOLLOW_DEAD);
    for (int k = 0; k < t.T; k++)
        for (int q = t.term_start[k]; q < (k + 1 < t.T ? (int)t.term_start[k + 1] : t.Q); q++) f.behind[q] = name(behind[k]);
    f.next.assign((size_t)(sink + 1) * t.n_cls, FOLLOW_DEAD);
    for (int c = 0; c < t.n_cls; c++) f.next[c] = FOLLOW_ANY;
    for (uint32_t s = first; s < A.n_states; s++)
        for (int c = 0; c < t.n_cls; c++) f.next[(size_t)(s - first + 1) * t.n_cls + c] = name(A.st(s).trans[c]);
}

// What every context takes behind a terminal: of an unknown set nothing is supposed but that it waits for one nonterminal Z, a set for each, and completing X
// there leads to COMP(Z, X) without the item that waits (its continuation is not known).  A rule that started before a string started in a set
// that waits for something that its left-hand side L begins, Y, and COMP(L, X) is contained in COMP(Y, X).  So every real set contains what stands here (by the same
// induction), and a string that lives here lives in every context.  A terminal may stand in several positions: a state is the list of the sets behind
// each, all of which must live.  Of what the budget does not reach nothing is sure.
void build_sure(const Tables &t, Follow &f) {
    static const size_t MOST_STATES = 2048;
    BehindTerminal B(t);
    HostAutomaton &A = B.A;
    for (int p = 0; p < t.P; p++) {
        const uint16_t code = t.sym[p];
        if ((code >> SYM_KIND_SHIFT) != SYM_NT || B.unknown[code & SYM_ID_MASK_NT]) continue;
        const Item it{(uint16_t)p, 0, A.n_states};
        B.unknown[code & SYM_ID_MASK_NT] = A.add(&it, 1, 0, 0);
    }
    B.first = A.n_states;
    auto complete = [&](const Item &it, uint32_t X) {          // (every nonterminal with rules but the added start symbol is waited for: rules that nothing reaches are gone, and the start symbol's has no terminal)
        const size_t at = (size_t)(t.sym[A.st(it.o).items[0].p] & SYM_ID_MASK_NT) * t.N + X;
        if (!B.spend(t.comp_off[at + 1] - t.comp_off[at])) return false;
        for (uint32_t k = t.comp_off[at]; k < t.comp_off[at + 1]; k++) {
            const uint16_t p = t.comp_list[k];
            if (p != COMP_ADVANCE_WAITING) B.w.insert(Item{p, (t.sym[p] >> SYM_KIND_SHIFT) == SYM_TERM ? t.term_start[t.sym[p] & SYM_ID_MASK] : (uint16_t)0, it.o});
        }
        return true;
    };
    std::map<std::vector<uint32_t>, uint32_t> names;
    std::vector<const std::vector<uint32_t> *> states{nullptr};   // 0: SURE_NOT
    std::vector<uint32_t> key;
    auto name = [&]() -> uint16_t {
        std::sort(key.begin(), key.end());
        key.erase(std::unique(key.begin(), key.end()), key.end());
        const auto found = names.find(key);
        if (found != names.end()) return (uint16_t)found->second;
        if (states.size() > MOST_STATES) return SURE_NOT;
        const auto at = names.emplace(key, (uint32_t)states.size()).first;
        states.push_back(&at->first);
        return (uint16_t)at->second;
    };
    const std::vector<std::vector<uint16_t>> at = positions_of_terminals(t);
    f.sure_behind.assign(t.Q, SURE_NOT);
    std::vector<uint16_t> one(1);
    for (int k = 0; k < t.T; k++) {
        bool all = !at[k].empty();
        key.clear();
        for (size_t i = 0; all && i < at[k].size(); i++) {
            one[0] = at[k][i];
            key.push_back(B.behind(one, [&](uint16_t p) { return B.unknown[t.lhs_of[p]]; }, complete));
            all = key.back() != HostAutomaton::NONE;
        }
        if (!all) continue;
        const uint16_t behind = name();
        for (int q = t.term_start[k]; q < (k + 1 < t.T ? (int)t.term_start[k + 1] : t.Q); q++) f.sure_behind[q] = behind;
    }
    f.sure_next.assign(t.n_cls, SURE_NOT);
    for (size_t s = 1; s < states.size(); s++)
        for (int c = 0; c < t.n_cls; c++) {
            bool all = true;
            key.clear();
            for (size_t i = 0; all && i < states[s]->size(); i++) {
                const uint32_t from = (*states[s])[i];
                const uint32_t to = from == HostAutomaton::SINK || !B.spend(1) ? HostAutomaton::DEAD : B.step(from, c, complete);
                all = to != HostAutomaton::DEAD && to != HostAutomaton::NONE;
                key.push_back(to);
            }
            f.sure_next.push_back(all ? name() : (uint16_t)SURE_NOT);
        }
}

// Whether the terminal, entered in DFA state q, ends inside the string with the rest of it behind: in no context, in some perhaps, in every one.
enum class EndsInside { NO, PERHAPS, SURELY };
static EndsInside ends_inside(const Tables &t, const Follow &f, uint32_t q, const uint8_t *bytes, size_t n) {
    EndsInside answer = EndsInside::NO;
    size_t walked = 0;
    for (size_t k = 0; k + 1 < n; k++) {
        q = t.delta[(size_t)q * t.n_cls + t.cls[bytes[k]]];
        if (q == DFA_DEAD) break;
        if (!(t.qflags[q] & QF_ACCEPT)) continue;
        uint32_t s = f.behind[q], sure = f.sure_behind[q];
        for (size_t j = k + 1; j < n && s != FOLLOW_DEAD; j++, walked++) {
            if (walked == FOLLOW_BYTES_MAX) return EndsInside::PERHAPS;
            s = f.next[(size_t)s * t.n_cls + t.cls[bytes[j]]];
            sure = f.sure_next[(size_t)sure * t.n_cls + t.cls[bytes[j]]];
        }
        if (s == FOLLOW_DEAD) continue;
        if (sure != SURE_NOT) return EndsInside::SURELY;
        answer = EndsInside::PERHAPS;
    }
    return answer;
}

// For every DFA state q: run the DFA alone from q down the trie.  A string the DFA survives is
// valid whatever the context (the in-progress terminal item survives or has just completed).  A
// string on which the DFA dies is hopeless for this item unless the DFA passed an accepting state
// first -- then the terminal may end there: it is valid if every context takes the rest, hopeless if none does, and else depends on the parser.  Rows of
// nonterminals are the union over the terminals that can begin them.
void build_token_mask_cache(const Tables &t, const Follow &f, Trie &tr) {
    const int Wr = tr.Wr, rows = t.Q + t.N;
    tr.ci_valid.assign((size_t)rows * Wr, 0);
    tr.ci_cd.assign((size_t)rows * Wr, 0);
    tr.ci_ends.assign((size_t)rows * Wr, 0);
    tr.ci_alone.assign((size_t)rows * Wr, 0);
    const uint32_t n = (uint32_t)tr.nodes.size();
    std::vector<uint16_t> st(MAX_TOKEN_LEN_ON_DEVICE + 2);
    std::vector<uint8_t> acc(MAX_TOKEN_LEN_ON_DEVICE + 2);
    for (int q = 0; q < t.Q; q++) {
        if (!(t.qflags[q] & QF_CONT)) continue;   // no item ever waits in a state without outgoing edges
        uint32_t *V = &tr.ci_valid[(size_t)q * Wr], *C = &tr.ci_cd[(size_t)q * Wr], *E = &tr.ci_ends[(size_t)q * Wr], *S = &tr.ci_alone[(size_t)q * Wr];
        st[0] = (uint16_t)q; acc[0] = 0;
        for (uint32_t i = 0; i < n;) {
            const TrieNode &nd = tr.nodes[i];
            const int d = nd.depth;
            uint16_t s2 = t.delta[(size_t)st[d - 1] * t.n_cls + t.cls[nd.byte]];
            if (s2 == DFA_DEAD) {
                if (acc[d - 1])
                    for (uint32_t r = nd.rank; r < nd.rank + nd.n_sub; r++) {
                        E[r >> 5] |= 1u << (r & 31);
                        const EndsInside ends = ends_inside(t, f, (uint32_t)q, &tr.str_bytes[tr.str_off[r]], tr.str_off[r + 1] - tr.str_off[r]);
                        if (ends == EndsInside::PERHAPS) C[r >> 5] |= 1u << (r & 31);
                        if (ends == EndsInside::SURELY) V[r >> 5] |= 1u << (r & 31);
                    }
                i = nd.skip;
            } else {
                st[d] = s2; acc[d] = acc[d - 1] | (t.qflags[s2] & QF_ACCEPT);
                if (nd.has_string) { V[nd.rank >> 5] |= 1u << (nd.rank & 31); S[nd.rank >> 5] |= 1u << (nd.rank & 31); }
                i++;
            }
        }
    }
    for (int Y = 0; Y < t.N; Y++) {
        uint32_t *V = &tr.ci_valid[(size_t)(t.Q + Y) * Wr], *C = &tr.ci_cd[(size_t)(t.Q + Y) * Wr], *E = &tr.ci_ends[(size_t)(t.Q + Y) * Wr], *S = &tr.ci_alone[(size_t)(t.Q + Y) * Wr];
        for (uint16_t term : t.first_terms[Y]) {
            const size_t from = (size_t)t.term_start[term] * Wr;
            for (int w = 0; w < Wr; w++) { V[w] |= tr.ci_valid[from + w]; C[w] |= tr.ci_cd[from + w]; E[w] |= tr.ci_ends[from + w]; S[w] |= tr.ci_alone[from + w]; }
        }
    }
}

}  // namespace zf
