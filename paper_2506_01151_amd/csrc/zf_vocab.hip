// What zf_compile derives from the vocabulary's bytes and the terminals' DFAs, worked out on the device: the strings as byte
// classes, and the token-mask cache (Section 4.3): for every DFA state and every nonterminal, the strings that a terminal
// entered in that state swallows whole or on which it dies behind an accepting state with a rest that every context takes, and those with a rest that some context
// takes.  (Against leaving what every context takes to the mask kernels: 8 steps of 64 x 152,064 of the expression grammar without pruning 574 -> 274 us, 16
// with it 314 -> 294, 32 of one row x 32,000 JSON 211 -> 196, 16 of 16 x 128,256 of the schema 138 -> 132.)
//   Every row is independent of every other and every string of every other string, so a lane takes a string and walks it through the DFAs of 32 rows
// one after the other; most walks end at the first byte.  A schema of 229 rows and a vocabulary of 128,256 tokens are 29 million walks, which the
// host did down the trie and then turned into token order: 2.2 + 0.9 ms of a compile, and 1.5 + 0.7 for the strings as byte classes;
// here they run while the host sorts the vocabulary.
#include "zf_kernel_common.h"

namespace zf {
namespace {

static const uint32_t VOCAB_BLOCK = 256, VOCAB_ROWS = 32;   // strings, and rows, that a block takes

template <class Off>
__device__ __forceinline__ void string_at(const Off *off, uint32_t n, uint32_t i, uint64_t &from, uint32_t &len) {
    from = 0; len = 0;
    if (i < n) { from = (uint64_t)off[i]; len = (uint32_t)((uint64_t)off[i + 1] - from); }
}

// Rows of the DFA states.  Off: the offsets' type.  Grid: (blocks of strings, blocks of rows).
template <class Off>
__global__ __launch_bounds__(VOCAB_BLOCK) void vocab_rows_kernel(VocabRows a, const Off *off) {
    __shared__ uint8_t cls[256];
    __shared__ uint32_t left[VOCAB_ROWS];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, i = blockIdx.x * VOCAB_BLOCK + tid, q0 = blockIdx.y * VOCAB_ROWS;
    cls[tid] = a.cls[tid];
    if (tid < VOCAB_ROWS) left[tid] = 0;
    __syncthreads();
    uint64_t from;
    uint32_t len, at_hand[2] = {0, 0};                       // the first eight classes
    string_at(off, a.n, i, from, len);
#pragma unroll
    for (uint32_t k = 0; k < 8u; k++) if (k < len) at_hand[k >> 2] |= (uint32_t)cls[a.bytes[from + k]] << (8u * (k & 3u));
    auto class_at = [&](uint32_t k) __attribute__((always_inline)) -> uint32_t { return k < 8u ? (at_hand[k >> 2] >> (8u * (k & 3u))) & 0xFFu : (uint32_t)cls[a.bytes[from + k]]; };
    for (uint32_t q = q0; q < q0 + VOCAB_ROWS && q < a.Q; q++) {
        bool valid = false, undecided = false;
        if (a.qflags[q] & QF_CONT) {                         // no item ever waits in a state without outgoing edges
            uint32_t s = q, k = 0;
            bool accepted = false;
            while (k < len) {
                s = a.delta[(size_t)s * a.n_cls + class_at(k)];
                if (s == DFA_DEAD) break;
                accepted |= (a.qflags[s] & QF_ACCEPT) != 0;
                k++;
            }
            valid = len > 0 && k == len;
            if (k < len && accepted) {                       // it dies behind an accepting state: where it may end, does every context take the rest, or does any?
                uint32_t left = FOLLOW_BYTES_MAX;
                s = q;
                for (k = 0; !valid && left && k + 1u < len; k++) {
                    s = a.delta[(size_t)s * a.n_cls + class_at(k)];
                    if (s == DFA_DEAD) break;
                    if (!(a.qflags[s] & QF_ACCEPT)) continue;
                    uint32_t f = a.behind[s], g = a.sure_behind[s];
                    uint32_t j = k + 1u;
                    for (; left && f != FOLLOW_DEAD && j < len; j++, left--) {
                        f = a.follow[(size_t)f * a.n_cls + class_at(j)];
                        g = a.sure_next[(size_t)g * a.n_cls + class_at(j)];
                    }
                    undecided |= f != FOLLOW_DEAD || !left;   // (the bytes that are walked for may end with a walk: the next end is then not known to lead nowhere)
                    valid = f != FOLLOW_DEAD && j == len && g != SURE_NOT;
                }
                undecided = undecided && !valid;
            }
        }
        const unsigned long long v = __ballot(valid), u = __ballot(undecided);
        const uint32_t w = i >> 5;
        if ((lane & 31u) == 0 && w < a.words) {
            const uint32_t vw = (uint32_t)(v >> lane), uw = (uint32_t)(u >> lane);
            if (a.both) a.both[(size_t)q * a.words + w] = make_uint2(vw, uw);
            else { a.valid[(size_t)q * a.words + w] = vw; a.undecided[(size_t)q * a.words + w] = uw; }
        }
        if (lane == 0 && u) atomicAdd(&left[q - q0], (uint32_t)__popcll(u));
    }
    __syncthreads();
    if (a.counts && tid < VOCAB_ROWS && left[tid]) atomicAdd(&a.counts[q0 + tid], left[tid]);
}

// Row of nonterminal Y: the union over the terminals that can begin it.
__global__ __launch_bounds__(VOCAB_BLOCK) void vocab_nonterminal_rows_kernel(VocabRows a) {
    const uint32_t w = blockIdx.x * VOCAB_BLOCK + threadIdx.x, Y = blockIdx.y;
    uint32_t v = 0, u = 0;
    if (w < a.words) {
        for (uint32_t k = a.first_off[Y]; k < a.first_off[Y + 1u]; k++) {
            const size_t at = (size_t)a.first_state[k] * a.words + w;
            if (a.both) { const uint2 x = a.both[at]; v |= x.x; u |= x.y; }
            else { v |= a.valid[at]; u |= a.undecided[at]; }
        }
        const size_t to = (size_t)(a.Q + Y) * a.words + w;
        if (a.both) a.both[to] = make_uint2(v, u);
        else { a.valid[to] = v; a.undecided[to] = u; }
    }
    if (!a.counts) return;
    uint32_t n = (uint32_t)__popc(u & ~v);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) n += __shfl_xor(n, d);
    if ((threadIdx.x & 63u) == 0 && n) atomicAdd(&a.counts[a.Q + Y], n);
}

// The tokens' records (DeviceTables::tok16).
__global__ __launch_bounds__(VOCAB_BLOCK) void vocab_tokens_kernel(const int64_t *off, const uint8_t *bytes, const uint8_t *cls_g, uint32_t n, Str16 *out) {
    __shared__ uint8_t cls[256];
    cls[threadIdx.x] = cls_g[threadIdx.x];
    __syncthreads();
    const uint32_t i = blockIdx.x * VOCAB_BLOCK + threadIdx.x;
    if (i >= n) return;
    uint64_t from;
    uint32_t len;
    string_at(off, n, i, from, len);
    Str16 r{{0, 0, 0, 0}};
#pragma unroll
    for (uint32_t k = 0; k <= TOK_AT_HAND; k++) {
        uint32_t b = 0;
        if (k < TOK_AT_HAND && k < len) b = cls[bytes[from + k]];
        else if (k == (len < TOK_AT_HAND ? len : TOK_AT_HAND)) b = len > TOK_AT_HAND ? TOK_MORE : TOK_END;
        r.w[k >> 2] |= b << (8u * (k & 3u));
    }
    out[i] = r;
}

// The distinct strings in rank order (DeviceTables::str_cls, str16).
__global__ __launch_bounds__(VOCAB_BLOCK) void vocab_strings_kernel(const uint32_t *off, const uint8_t *bytes, const uint8_t *cls_g, uint32_t n, uint8_t *str_cls, Str16 *out) {
    __shared__ uint8_t cls[256];
    cls[threadIdx.x] = cls_g[threadIdx.x];
    __syncthreads();
    const uint32_t i = blockIdx.x * VOCAB_BLOCK + threadIdx.x;
    if (i >= n) return;
    uint64_t from;
    uint32_t len;
    string_at(off, n, i, from, len);
    Str16 r{{0, 0, 0, 0}};
#pragma unroll
    for (uint32_t k = 0; k < 16u; k++) if (k < len) r.w[k >> 2] |= (uint32_t)cls[bytes[from + k]] << (8u * (k & 3u));
    for (uint32_t k = 0; k < len; k++) str_cls[from + k] = cls[bytes[from + k]];
    out[i] = r;
}

}  // namespace

static hipError_t launch_rows(const VocabRows &a, const int64_t *off64, const uint32_t *off32, hipStream_t s) {
    if (a.words == 0) return hipSuccess;
    const uint32_t blocks = (a.words * 32u + VOCAB_BLOCK - 1u) / VOCAB_BLOCK;
    if (a.Q) {
        const dim3 grid(blocks, (a.Q + VOCAB_ROWS - 1u) / VOCAB_ROWS);
        if (off64) hipLaunchKernelGGL((vocab_rows_kernel<int64_t>), grid, dim3(VOCAB_BLOCK), 0, s, a, off64);
        else hipLaunchKernelGGL((vocab_rows_kernel<uint32_t>), grid, dim3(VOCAB_BLOCK), 0, s, a, off32);
    }
    if (a.N) hipLaunchKernelGGL(vocab_nonterminal_rows_kernel, dim3((a.words + VOCAB_BLOCK - 1u) / VOCAB_BLOCK, a.N), dim3(VOCAB_BLOCK), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_vocab_rows(const VocabRows &a, const int64_t *off, hipStream_t s) { return launch_rows(a, off, nullptr, s); }
hipError_t launch_vocab_rows(const VocabRows &a, const uint32_t *off, hipStream_t s) { return launch_rows(a, nullptr, off, s); }
hipError_t launch_vocab_tokens(const int64_t *off, const uint8_t *bytes, const uint8_t *cls, uint32_t n, Str16 *out, hipStream_t s) {
    if (n) hipLaunchKernelGGL(vocab_tokens_kernel, dim3((n + VOCAB_BLOCK - 1u) / VOCAB_BLOCK), dim3(VOCAB_BLOCK), 0, s, off, bytes, cls, n, out);
    return hipGetLastError();
}
hipError_t launch_vocab_strings(const uint32_t *off, const uint8_t *bytes, const uint8_t *cls, uint32_t n, uint8_t *str_cls, Str16 *out, hipStream_t s) {
    if (n) hipLaunchKernelGGL(vocab_strings_kernel, dim3((n + VOCAB_BLOCK - 1u) / VOCAB_BLOCK), dim3(VOCAB_BLOCK), 0, s, off, bytes, cls, n, str_cls, out);
    return hipGetLastError();
}

}  // namespace zf
