// Searched programs over equal spans of bytes (device code of the table form).
//
// A searched program accepts a string when a match begins at one of its
// positions.  The byte step maps a union of thread sets to the union of their
// images (Def. 5.1 / 5.2), so the threads that begin in one part of a string
// can be followed on their own: every lane takes B consecutive bytes of the
// text (the strings' bytes, one after another, whatever the strings' lengths),
// starts every position's threads there, and after its last byte follows the
// threads that are left, without starting new ones, until none is left, the
// string ends, or the lanes after it hold them all.  A string's result is the
// OR (earliest accept: the minimum) over the lanes that saw its bytes.  So the
// work of a lane does not depend on where strings begin and end, and one long
// string runs on as many lanes as it has spans.
//
// What bounds it: vector instructions (the counters of 10^6 lines, 120 MB, 67
// leaves in three words: 52 of them per wavefront and byte, four fifths of
// the chip's issue; 5 LDS reads).  236 us there, 510 GB/s; a lane per string
// took 1,890 us, each wavefront waiting for the longest of its 64 lines, and
// the longest line of all (4,096 bytes) 600 us however few lines there were.
// 20,000 lines: 20 us, of which the spans' serial chains are most (16 bytes a
// lane and about as many after them).
#pragma once

#include <cstdint>

namespace rx {

struct SpanText {             // string i: bytes[offsets[i], offsets[i + 1]), or with offsets NULL
    const uint8_t* bytes;     // bytes[i * stride, (i + 1) * stride)
    const int64_t* offsets;
    int64_t stride, n;
};

struct SpanProg {             // a searched, non-nullable program's tables (Def. 5.1)
    const uint32_t* first;
    const uint32_t* follow;
    const uint32_t* bytemask;
    int32_t L, prefix;        // prefix: rank of the search prefix's any-byte leaf
};

struct SpanOut {
    uint8_t* out;             // results (0 before the launch), or
    int64_t* first_pos;       // earliest accepts (-1 before the launch)
    int64_t* undone;          // not NULL: a lane gives up after `limit` bytes past its span and sets it
    int64_t limit;
};

constexpr int kSpanMax = 64;    // bytes per lane and turn: 16, 32 or 64
constexpr int kSpanTail = 32;   // bytes past its span that a lane reads from the staged text
// (512 together: more, and sets of three words have room for four workgroups in
// a compute unit instead of five, whose LDS goes by 1,280 bytes; 100,000 lines 41 -> 55 us)
constexpr int kSpanList = 416;  // string starts of a region kept in LDS
constexpr int kSpanPend = 96;   // words for the threads that outlive the staged text (see span_regions)

// LDS words per table row: rows of more than two words in whole 16-byte reads
constexpr int span_row_words(int W) { return W <= 2 ? W : (W + 3) / 4 * 4; }
// threads per workgroup: the larger tables are shared by more wavefronts
constexpr int span_threads(int W) { return W <= 4 ? 256 : W <= 8 ? 512 : 1024; }
// Dynamic LDS words of a workgroup of T threads: masks, the images of First,
// Follow rows, text (an odd row stride of B / 4 + 1 words: no bank conflicts),
// start bits, starts, listed threads.
constexpr int span_tile_words(int T) { return (T + 2) * (kSpanMax / 4 + 1); }
constexpr int span_bit_words(int T) { return (T * kSpanMax + kSpanTail + 31) / 32 + 1; }
constexpr int span_lds_words(int W, int L, int T) {
    return span_row_words(W) * (256 + 257 + L) + span_tile_words(T) + span_bit_words(T) + kSpanList + kSpanPend;
}

template <int W>
__device__ __forceinline__ void span_row(const uint32_t* __restrict__ p, uint32_t (&r)[W]) {
    if constexpr (W <= 2) {
#pragma unroll
        for (int w = 0; w < W; ++w) r[w] = p[w];
    } else {
#pragma unroll
        for (int q = 0; q < (W + 3) / 4; ++q) {
            const uint4 v = reinterpret_cast<const uint4*>(p)[q];
            r[4 * q] = v.x;
            if (4 * q + 1 < W) r[4 * q + 1 < W ? 4 * q + 1 : 0] = v.y;
            if (4 * q + 2 < W) r[4 * q + 2 < W ? 4 * q + 2 : 0] = v.z;
            if (4 * q + 3 < W) r[4 * q + 3 < W ? 4 * q + 3 : 0] = v.w;
        }
    }
}

// R |= Follow rows of the leaves in X
template <int W>
__device__ __forceinline__ void span_follow(const uint32_t (&X)[W], const uint32_t* __restrict__ F, uint32_t (&R)[W]) {
    constexpr int WP = span_row_words(W);
#pragma unroll
    for (int w = 0; w < W; ++w) {
        uint32_t x = X[w];
        while (x) {
            const int b = __builtin_ctz(x);
            x &= x - 1;
            uint32_t r[W];
            span_row<W>(F + (w * 32 + b) * WP, r);
#pragma unroll
            for (int v = 0; v < W; ++v) R[v] |= r[v];
        }
    }
}

template <int W>
__device__ __forceinline__ bool span_any(const uint32_t (&R)[W]) {
    uint32_t a = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) a |= R[w];
    return a != 0;
}

// Stages a program's tables: M (256 rows), N (257 rows: the image of First
// under each byte, which the threads begun at one position become; row 256 is
// empty), F (L rows).  The prefix leaf is in none of them: where it is live,
// its image is First, and N already holds what First becomes.
template <int W, int T>
__device__ __forceinline__ void span_tables(const SpanProg& P, uint32_t* M, uint32_t* N, uint32_t* F) {
    constexpr int WP = span_row_words(W);
    const int tid = threadIdx.x;
    for (int i = tid; i < 256 * WP; i += T) {
        const int c = i / WP, w = i % WP;
        M[i] = w < W ? P.bytemask[c * W + w] & ~((P.prefix >> 5) == w ? 1u << (P.prefix & 31) : 0u) : 0u;
    }
    for (int i = tid; i < P.L * WP; i += T) F[i] = i % WP < W ? P.follow[i / WP * W + i % WP] : 0u;
    __syncthreads();
    for (int c = tid; c < 257; c += T) {
        uint32_t X[W], R[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            X[w] = c < 256 ? P.first[w] & M[c * WP + w] : 0u;
            R[w] = 0u;
        }
        span_follow<W>(X, F, R);
#pragma unroll
        for (int w = 0; w < WP; ++w) N[c * WP + w] = w < W ? R[w < W ? w : 0] : 0u;
    }
    __syncthreads();
}

// The first i in [lo, hi] with i == hi or offsets[i] >= v, searched by the
// whole workgroup (every thread returns it).
template <int T>
__device__ __forceinline__ int64_t span_lower_bound(const int64_t* __restrict__ offsets, int64_t lo, int64_t hi,
                                                    int64_t v) {
    while (hi - lo > T) {
        const int64_t step = (hi - lo + T - 1) / T;
        const int64_t i = lo + (int64_t)threadIdx.x * step;
        const int k = __syncthreads_count(i < hi && offsets[i] < v);
        if (k == 0) return lo;
        // probes 0 .. k - 1 are below v, probe k (if there is one) is not
        const int64_t top = lo + (int64_t)k * step;
        lo += (int64_t)(k - 1) * step + 1;
        if (top < hi) hi = top;
    }
    const int64_t i = lo + threadIdx.x;
    return lo + __syncthreads_count(i < hi && offsets[i] < v);
}

// Where the strings of a region begin: strings sid .. next - 1 at `list` (the
// first kSpanList of them) bytes after `start`; string sid - 1 holds what lies
// before.
struct SpanStarts {
    int64_t start, sid, next;
    const uint32_t* list;
};

// The string that holds the byte p (>= 0) after the region's start: the last
// one that begins at or before it.
__device__ __forceinline__ int64_t span_string(const SpanText& X, const SpanStarts& S, int64_t p) {
    if (!X.offsets) return (S.start + p) / X.stride;
    int64_t lo = 0, hi = S.next - S.sid;   // starts before lo are <= p, starts from hi on are not
    if (hi <= kSpanList) {
        while (lo < hi) {
            const int mid = (int)(lo + hi) >> 1;
            if ((int64_t)S.list[mid] <= p) lo = mid + 1;
            else hi = mid;
        }
    } else {
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (X.offsets[S.sid + mid] - S.start <= p) lo = mid + 1;
            else hi = mid;
        }
    }
    return S.sid - 1 + lo;
}

// (crowded: many lanes to a string.  Atomics on one word take their turn, 23 ns
// each, so one that cannot lower the minimum is not made there.)
template <bool FIRST>
__device__ __forceinline__ void span_accept(const SpanText& X, const SpanOut& O, int64_t string, int64_t at, bool crowded) {
    if constexpr (FIRST) {
        const int64_t lo = X.offsets ? X.offsets[string] : string * X.stride;
        unsigned long long* p = reinterpret_cast<unsigned long long*>(O.first_pos + string);
        const unsigned long long v = (unsigned long long)(at + 1 - lo);
        if (!crowded || __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > v) atomicMin(p, v);
    } else {
        O.out[string] = 1;
    }
}

// The program over regions [r0, r1) of the text (T * B bytes each, counted
// from the 16-byte block that holds the first byte).  M, N, F: the staged
// tables; tile: the LDS after them.
template <int W, int T, bool FIRST>
__device__ __forceinline__ void span_regions(const SpanProg& P, const SpanText& X, const SpanOut& O, int64_t o0,
                                             int64_t oN, int B, int64_t r0, int64_t r1, const uint32_t* M,
                                             const uint32_t* N, const uint32_t* F, uint32_t* tile) {
    constexpr int WP = span_row_words(W);
    uint32_t* bits = tile + span_tile_words(T);
    uint32_t* list = bits + span_bit_words(T);
    const int tid = threadIdx.x;
    const int Q = B / 4, RS = Q + 1;   // words per span and per tile row
    const int RB = T * B;
    const uint32_t abit = 1u << (P.L & 31);   // in the last word: W = L / 32 + 1
    const int64_t skew = (int64_t)(reinterpret_cast<uintptr_t>(X.bytes + o0) & 15);
    uint32_t fst[W];   // the threads that the next lane starts, and accept never among them (not nullable)
#pragma unroll
    for (int w = 0; w < W; ++w) fst[w] = P.first[w];
    // kStill: where a thread goes on past the staged text, in sets of one or
    // two words: a byte that leaves the threads as they were is the rule there
    // (x.*y between its ends), and a step is a chain of LDS reads.  What it does
    // depends on the leaves of A and V that survive the byte and on the row of
    // N: where the survivors are those of a step that changed nothing, and N's
    // row adds nothing to V, neither does this one.  (Wider sets seldom stand
    // still: three words, random text, 38 us without, 41 with.)
    constexpr bool kStill = W <= 2;
    uint32_t* pend = list + kSpanList;   // how many, then {at, string, threads} each
    constexpr int kPendWords = W + 4, kPendMax = (kSpanPend - 1) / kPendWords;
    if (tid == 0) pend[0] = 0u;
    const bool crowded = oN - o0 >= 4096 * X.n;   // (from 192 on, lines of 320 bytes lost 8%)
    SpanStarts S;
    S.sid = -1;
    S.list = list;
    // One turn per region, then, with several regions, one for the listed threads.
    const bool lists = r1 - r0 > 1;
    for (int64_t r = r0; r < r1 + lists; ++r) {
        uint32_t A[W];   // threads that have read a byte
#pragma unroll
        for (int w = 0; w < W; ++w) A[w] = 0u;
        int64_t from = 0, string = -1;   // where A goes on past the staged text, in which string (-1: it does not)
        __syncthreads();                 // the last region's text and starts have been read
        if (r == r1) {
            // (over all wavefronts where lanes that stand still wait for those of theirs that do not, else in few)
            const int k = kStill ? (tid & 63) * (T / 64) + (tid >> 6) : tid;
            if (k < (int)pend[0]) {
                const uint32_t* e = pend + 1 + k * kPendWords;
                from = (int64_t)((uint64_t)e[1] << 32 | e[0]);
                string = (int64_t)((uint64_t)e[3] << 32 | e[2]);
#pragma unroll
                for (int w = 0; w < W; ++w) A[w] = e[4 + w];
            }
        } else {
            S.start = o0 - skew + r * RB;   // in the text's own offsets
            for (int i = tid; i < span_bit_words(T); i += T) bits[i] = 0u;
            for (int q = tid; q < (RB + kSpanTail) / 16; q += T) {
                const int64_t at = S.start + 16 * q;
                uint4 v = make_uint4(0u, 0u, 0u, 0u);
                if (at < oN) v = *reinterpret_cast<const uint4*>(X.bytes + at);
                uint32_t* t = tile + (4 * q / Q) * RS + 4 * q % Q;   // Q is 4, 8 or 16: the four words share a row
                t[0] = v.x;
                t[1] = v.y;
                t[2] = v.z;
                t[3] = v.w;
            }
            // one bit per byte where a string begins, and where the last one ends
            if (X.offsets) {
                S.sid = S.sid < 0 ? span_lower_bound<T>(X.offsets, 0, X.n + 1, S.start) : S.next;
                __syncthreads();
                S.next = S.sid;
                for (int64_t base = S.sid;; base += T) {
                    const int64_t i = base + tid;
                    const int64_t rel = i <= X.n ? X.offsets[i] - S.start : INT64_MAX;
                    const bool seen = rel < RB + kSpanTail;
                    if (seen) atomicOr(&bits[rel >> 5], 1u << (rel & 31));
                    if (rel < RB && i - S.sid < kSpanList) list[i - S.sid] = (uint32_t)rel;
                    S.next += __syncthreads_count(rel < RB);
                    if (__syncthreads_count(seen) < T) break;
                }
            } else {
                __syncthreads();
                const int64_t i0 = S.start > 0 ? (S.start + X.stride - 1) / X.stride : 0;
                for (int64_t i = i0 + tid; i <= X.n && i * X.stride - S.start < RB + kSpanTail; i += T) {
                    const int64_t rel = i * X.stride - S.start;
                    atomicOr(&bits[rel >> 5], 1u << (rel & 31));
                }
                __syncthreads();
            }
            const int64_t left = oN - S.start;   // bytes of the text from the region's start on
            const int p0 = tid * B;              // this lane's span
            if (p0 < left) {
                // no threads start before the first string (the block's head) nor after an accept, up to the next string
                bool off = S.start + p0 < o0;
                uint64_t ev = 0;   // accepts, by byte of the span
                const uint32_t* row = tile + tid * RS;
                for (int g = 0; g < Q; ++g) {
                    const uint32_t word = row[g];
                    const uint32_t sb = (bits[(p0 + 4 * g) >> 5] >> ((p0 + 4 * g) & 31)) & 15u;
                    bool slow = true;
                    if (__ballot(sb != 0u) == 0ull) {
                        // No string begins in any lane's four bytes: an accept
                        // stays (its leaf is in M and F), so one look after the
                        // four tells whether there was one.
                        if (__ballot(!off) == 0ull) continue;
                        uint32_t A0[W];
#pragma unroll
                        for (int w = 0; w < W; ++w) A0[w] = A[w];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t c = (word >> (8 * i)) & 255u;
                            uint32_t m[W], Y[W];
                            span_row<W>(M + c * WP, m);
#pragma unroll
                            for (int w = 0; w < W; ++w) Y[w] = A[w] & m[w];
                            span_row<W>(N + (off ? 256u : c) * WP, A);
                            span_follow<W>(Y, F, A);
                        }
                        slow = false;
                        if (A[W - 1] & abit) {
                            if constexpr (FIRST) {
                                slow = true;   // again, byte by byte
#pragma unroll
                                for (int w = 0; w < W; ++w) A[w] = A0[w];
                            } else {
                                ev |= 1ull << (4 * g);
                                off = true;
#pragma unroll
                                for (int w = 0; w < W; ++w) A[w] = 0u;
                            }
                        }
                    }
                    if (slow) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            if ((sb >> i) & 1u) {   // a string begins: nothing of the last one is left
#pragma unroll
                                for (int w = 0; w < W; ++w) A[w] = 0u;
                                off = false;
                            }
                            const uint32_t c = (word >> (8 * i)) & 255u;
                            uint32_t m[W], Y[W];
                            span_row<W>(M + c * WP, m);
#pragma unroll
                            for (int w = 0; w < W; ++w) Y[w] = A[w] & m[w];
                            span_row<W>(N + (off ? 256u : c) * WP, A);
                            span_follow<W>(Y, F, A);
                            if (A[W - 1] & abit) {
                                ev |= 1ull << (4 * g + i);
                                off = true;
#pragma unroll
                                for (int w = 0; w < W; ++w) A[w] = 0u;
                            }
                        }
                    }
                }
                if (p0 + B > left) {   // the text ends in this span: nothing counts past it
                    ev &= (1ull << (left - p0)) - 1;
#pragma unroll
                    for (int w = 0; w < W; ++w) A[w] = 0u;
                }
                if (FIRST && crowded) {
                    // a lane's first accept counts for nothing where a lane before it has one in the same string
                    const uint64_t with = __ballot(ev != 0u);
                    int64_t s1 = -1, s2 = -1;   // the strings of its first and its last
                    if (ev) {
                        s1 = span_string(X, S, p0 + __builtin_ctzll(ev));
                        s2 = ev & (ev - 1) ? span_string(X, S, p0 + 63 - __builtin_clzll(ev)) : s1;
                    }
                    const int lane = tid & 63;
                    const uint64_t lower = with & ((1ull << lane) - 1);
                    const int64_t before = __shfl(s2, lower ? 63 - __builtin_clzll(lower) : lane, 64);
                    if (lower && before == s1) ev &= ev - 1;
                }
                while (ev) {
                    const int k = __builtin_ctzll(ev);
                    ev &= ev - 1;
                    span_accept<FIRST>(X, O, span_string(X, S, p0 + k), S.start + p0 + k, crowded);
                }
                // What is left of the threads begun here, less those that the
                // next lane starts too, within the staged text.
                int64_t over = -1;   // the accept past the span
                int p = p0 + B;
                for (int g = 0; g < kSpanTail / 4; ++g, p += 4) {
                    if (!span_any<W>(A)) break;
                    const int d = (tid + 1) * Q + g;
                    const uint32_t word = tile[d / Q * RS + d % Q];
                    const uint32_t sb = bits[p >> 5] >> (p & 31);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t c = (word >> (8 * i)) & 255u;
                        uint32_t m[W], Y[W];
                        span_row<W>(M + c * WP, m);
                        const bool ends = (sb >> i) & 1u;
#pragma unroll
                        for (int w = 0; w < W; ++w) {
                            Y[w] = ends ? 0u : A[w] & ~fst[w] & m[w];
                            A[w] = 0u;
                        }
                        span_follow<W>(Y, F, A);
                        if (A[W - 1] & abit) {
                            over = S.start + p + i;
#pragma unroll
                            for (int w = 0; w < W; ++w) A[w] = 0u;
                        }
                    }
                }
                if (over >= 0) {
                    span_accept<FIRST>(X, O, span_string(X, S, p0 + B - 1), over, crowded);
                } else if (span_any<W>(A)) {
                    from = S.start + p;   // still going (no string began since)
                    string = span_string(X, S, p0 + B - 1);
                }
            }
            // One such thread holds up the whole workgroup at the next region,
            // so where there are few they are listed and followed together
            // after the last: 200,000 strings of 256 bytes, err.*timeout with
            // err in 5% of them, 270 us without, 140 with.
            if (lists) {
                const int held = (int)pend[0], more = __syncthreads_count(string >= 0);
                if (held + more <= kPendMax && string >= 0) {
                    uint32_t* e = pend + 1 + (int)atomicAdd(pend, 1u) * kPendWords;
                    e[0] = (uint32_t)from;
                    e[1] = (uint32_t)((uint64_t)from >> 32);
                    e[2] = (uint32_t)string;
                    e[3] = (uint32_t)((uint64_t)string >> 32);
#pragma unroll
                    for (int w = 0; w < W; ++w) e[4 + w] = A[w];
                    string = -1;
                }
            }
        }
        if (string >= 0) {
            // Up to the string's end, beside the threads that the next lanes
            // start from here on, less those that are among them.
            const int64_t end = X.offsets ? X.offsets[string + 1] : (string + 1) * X.stride;
            const bool limited = O.undone && end - from > O.limit;
            const int64_t stop = limited ? from + O.limit : end;
            uint32_t V[W];   // threads begun from here on
#pragma unroll
            for (int w = 0; w < W; ++w) V[w] = 0u;
            bool done = false;
            // (16-byte aligned; the next 16 bytes are on their way)
            uint4 nx = make_uint4(0u, 0u, 0u, 0u);
            if (from < stop) nx = *reinterpret_cast<const uint4*>(X.bytes + from);
            constexpr int kAhead = W == 1 && !FIRST ? 4 : 1;   // bytes looked at together
            bool still = false;
            uint32_t fy[W] = {}, fz[W] = {};
            for (int64_t at = from; at < stop && !done; at += 16) {
                const uint4 v = nx;
                if (at + 16 < stop) nx = *reinterpret_cast<const uint4*>(X.bytes + at + 16);
                const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
                for (int b = 0; b < 16 && at + b < stop && !done; ++b) {
                    if constexpr (kAhead > 1) {
                        if (still && b % kAhead == 0 && at + b + kAhead <= stop) {
                            const uint32_t word = (b & 8 ? (b & 4 ? wv[3] : wv[2]) : (b & 4 ? wv[1] : wv[0])) >> (8 * (b & 3));
                            uint32_t diff = 0u;
#pragma unroll
                            for (int k = 0; k < kAhead; ++k) {
                                const uint32_t c = (word >> (8 * k)) & 255u;
                                uint32_t m[W], U[W];
                                span_row<W>(M + c * WP, m);
                                span_row<W>(N + c * WP, U);
#pragma unroll
                                for (int w = 0; w < W; ++w)
                                    diff |= ((A[w] & ~(V[w] | fst[w]) & m[w]) ^ fy[w]) | ((V[w] & m[w]) ^ fz[w]) | (U[w] & ~V[w]);
                            }
                            if (diff == 0u) {
                                b += kAhead - 1;
                                continue;
                            }
                        }
                    }
                    const uint32_t lo2 = b & 4 ? wv[1] : wv[0], hi2 = b & 4 ? wv[3] : wv[2];
                    const uint32_t c = ((b & 8 ? hi2 : lo2) >> (8 * (b & 3))) & 255u;
                    uint32_t m[W], Y[W], Z[W];
                    span_row<W>(M + c * WP, m);
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        Y[w] = A[w] & ~(V[w] | fst[w]) & m[w];
                        Z[w] = V[w] & m[w];
                    }
                    if constexpr (kStill) {
                        uint32_t U[W], R[W], diff = 0u, adds = 0u;
                        span_row<W>(N + c * WP, U);
#pragma unroll
                        for (int w = 0; w < W; ++w) {
                            diff |= (Y[w] ^ fy[w]) | (Z[w] ^ fz[w]);
                            adds |= U[w] & ~V[w];
                            R[w] = 0u;
                        }
                        if (still && (diff | adds) == 0u) continue;
                        uint32_t moved = adds;
                        span_follow<W>(Z, F, R);
#pragma unroll
                        for (int w = 0; w < W; ++w) {
                            moved |= R[w] ^ V[w];
                            V[w] = R[w] | U[w];
                            fz[w] = Z[w];
                            R[w] = 0u;
                        }
                        span_follow<W>(Y, F, R);
#pragma unroll
                        for (int w = 0; w < W; ++w) {
                            moved |= R[w] ^ A[w];
                            A[w] = R[w];
                            fy[w] = Y[w];
                        }
                        still = moved == 0u;
                    } else {
#pragma unroll
                        for (int w = 0; w < W; ++w) A[w] = 0u;
                        span_follow<W>(Y, F, A);
                        span_row<W>(N + c * WP, V);
                        span_follow<W>(Z, F, V);
                    }
                    if (V[W - 1] & abit) {
                        done = true;   // a later lane has the string's accept, here or before
                    } else if (A[W - 1] & abit) {
                        span_accept<FIRST>(X, O, string, at + b, crowded);
                        done = true;
                    } else {
                        uint32_t rest = 0u;
#pragma unroll
                        for (int w = 0; w < W; ++w) rest |= A[w] & ~(V[w] | fst[w]);
                        done = rest == 0u;
                    }
                }
            }
            if (!done && limited) *O.undone = 1;
        }
    }
}

// The bytes per lane and turn for `total` bytes on `lanes` lanes: 64, or
// fewer where that leaves lanes without any (a span's bytes are one serial
// chain of table lookups).
__device__ __forceinline__ int span_bytes(int64_t total, int64_t lanes) {
    return total > 32 * lanes ? 64 : total > 16 * lanes ? 32 : 16;
}

}  // namespace rx
