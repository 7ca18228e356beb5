// Stage A8: a device-resident LSH index answering batches of similarity
// queries with per-query thresholds.
//
// Build: the index strings go through A0-A3 once (alphabet, truncation,
// randomness, embedding, per-table sort by (top key bits, length,
// position)); the sorted tables, the full keys and the lengths stay in HBM.
// Query batch: the queries are embedded with the same random streams,
// truncation and alphabet (A1-A2); for every (table, query) a binary search
// finds the group of entries with the query key's top bits and, inside it,
// the length window [|q| - K_q, |q| + K_q]; entries with the same full key
// are candidates.  Candidates are de-duplicated per query, verified with the
// banded kernel at the query's own threshold (A5) and returned per query
// sorted by index position.
#include <string.h>

#include <algorithm>

#include "ej_internal.h"

using namespace ej;

struct ej_index {
    ej_ctx *ctx = nullptr;
    std::shared_ptr<bool> alive;   // whether ctx still exists
    int device = 0;
    ej_params p{};
    uint32_t n = 0, sigma = 0, L = 0, maxlen = 0, minlen = 0, T = 0;
    uint64_t total = 0;            // characters of the indexed strings
    uint8_t lut[256];
    uint64_t hbm_limit = 0;
    // owned device memory
    uint8_t *d_codes = nullptr;
    uint64_t *d_offsets = nullptr;
    uint32_t *d_dk = nullptr;      // [T][n] top 32 key bits, sorted per table
    uint64_t *d_key_s = nullptr;   // [T][n] full keys in sorted order
    uint32_t *d_len_s = nullptr;   // [T][n] lengths in sorted order
    uint32_t *d_ids = nullptr;     // [T][n] positions in sorted order
    RowMasks masks;                // match masks of the index strings (verification)
    uint32_t *d_planes = nullptr;  // bit planes of their codes (verification)
    Rand rd;                       // random streams (owned copies)
    std::vector<void *> owned;
    // the arrays that grow with the strings (codes, offsets, tables, planes)
    void *slab = nullptr;
    size_t slab_bytes = 0;
};

namespace {

inline uint32_t grid_for(ej_ctx *ctx, uint64_t work, uint32_t block) {
    uint64_t g = (work + block - 1) / block;
    uint64_t cap = (uint64_t)ctx->num_cu * 16;
    if (g > cap) g = cap;
    if (g == 0) g = 1;
    return (uint32_t)g;
}

// The arrays of an index of n strings with `total` characters and tot table
// entries, in one slab.
struct SlabParts {
    uint8_t *codes;
    uint64_t *offsets, *key_s;
    uint32_t *dk, *len_s, *ids, *planes;
};

SlabParts slab_parts(ej_ctx *ctx, uint64_t n, uint64_t total, uint64_t tot, uint32_t sigma,
                     void **slab, size_t *bytes) {
    size_t at = 0;
    auto part = [&](uint64_t b) {
        const size_t o = at;
        at += (b + 255) & ~(uint64_t)255;
        return o;
    };
    const size_t codes = part(total + 64), offsets = part(8 * (n + 1)), key_s = part(8 * tot),
                 dk = part(4 * tot), len_s = part(4 * tot), ids = part(4 * tot),
                 planes = part(4 * plane_words(total) * plane_count(sigma));
    char *p = (char *)slab_take(ctx, at, bytes);
    *slab = p;
    return SlabParts{(uint8_t *)(p + codes),    (uint64_t *)(p + offsets),
                     (uint64_t *)(p + key_s),   (uint32_t *)(p + dk),
                     (uint32_t *)(p + len_s),   (uint32_t *)(p + ids),
                     (uint32_t *)(p + planes)};
}

template <typename T>
void copy_on(ej_ctx *ctx, T *dst, const T *src, uint64_t count) {
    if (count)
        EJ_HIP(hipMemcpyAsync(dst, src, count * sizeof(T), hipMemcpyDeviceToDevice, ctx->stream));
}

template <typename T>
T *own_copy(ej_index *ix, const T *src, size_t count) {
    T *dst = nullptr;
    size_t bytes = std::max<size_t>(count * sizeof(T), 16);
    hipError_t e = hipMalloc((void **)&dst, bytes);
    if (e == hipErrorOutOfMemory && spare_release(ix->ctx)) e = hipMalloc((void **)&dst, bytes);
    if (e != hipSuccess) fail(EJ_ENOMEM, "index allocation failed");
    ix->owned.push_back(dst);
    if (src && count)
        EJ_HIP(hipMemcpyAsync(dst, src, count * sizeof(T), hipMemcpyDeviceToDevice,
                              ix->ctx->stream));
    return dst;
}

// Attributes of a table's sorted entries; the entries come as length ranks
// (place[e], keys and lengths by rank) and leave as string positions.
__global__ void k_sorted_attrs_full(const uint64_t *__restrict__ keys,
                                    const uint32_t *place, const uint32_t *__restrict__ perm,
                                    const uint32_t *__restrict__ perm_len, uint32_t n,
                                    uint64_t tot, uint32_t *ids, uint32_t *__restrict__ dk,
                                    uint64_t *__restrict__ key_s, uint32_t *__restrict__ len_s) {
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < tot;
         e += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t t = e / n;
        const uint32_t rank = place[e];
        const uint64_t k = keys[t * n + rank];
        key_s[e] = k;
        dk[e] = (uint32_t)(k >> 29);
        len_s[e] = perm_len[rank];
        ids[e] = perm[rank];
    }
}

// The first of the n sorted values that is not below `top`.  The values are
// the top bits of hashes, so a value's place is close to its share of the
// range: three interpolations come within a few entries of it, and a search
// in doubling steps from there finds it in any case (values that are not
// spread evenly, long runs of one value, cost more steps of that search).
__device__ inline uint32_t probe_lower(const uint32_t *__restrict__ d, uint32_t n, uint32_t top) {
    uint32_t lo = 0, hi = n;  // below `top` before lo, not below it from hi on
    uint32_t x = __umulhi(top, n);
    bool less = false;
    for (int it = 0; it < 3 && lo < hi; it++) {
        const uint32_t v = d[x];
        less = v < top;
        if (less) lo = x + 1; else hi = x;
        if (lo >= hi) break;
        const int64_t y = (int64_t)x + (((int64_t)top - (int64_t)v) * (int64_t)n >> 32);
        x = (uint32_t)min(max(y, (int64_t)lo), (int64_t)hi - 1);
    }
    uint32_t step = 2;
    if (less) {
        while (hi - lo > step) {
            if (d[lo + step] >= top) {
                hi = lo + step;
                break;
            }
            lo += step + 1;
            step *= 4;
        }
    } else {
        while (hi - lo > step) {
            if (d[hi - 1 - step] < top) {
                lo = hi - step;
                break;
            }
            hi -= step + 1;
            step *= 4;
        }
    }
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (d[mid] < top) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// One thread per (table, query): candidates are the entries of the table
// with the query's full key whose length is within K_q of the query's.
// Counts them and notes where the first entry of fitting length is.
// Bound by random 64-byte reads (about 100 G/s on the chip): 4,096 queries in
// 256 tables of 100,000 entries took 340 us with two binary searches over the
// whole table, and as much again to emit, which now starts at `first`.
__global__ void k_query_count(const uint64_t *__restrict__ qkeys, const uint32_t *__restrict__ qlen,
                              const uint32_t *__restrict__ Kq, uint32_t nq,
                              const uint32_t *__restrict__ dk, const uint64_t *__restrict__ key_s,
                              const uint32_t *__restrict__ len_s, uint32_t n, uint32_t T,
                              uint64_t *__restrict__ counts, uint32_t *__restrict__ first) {
    const uint64_t tot = (uint64_t)T * nq;
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < tot;
         e += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t t = (uint32_t)(e / nq), q = (uint32_t)(e % nq);
        const uint64_t key = qkeys[(uint64_t)t * nq + q];
        const uint32_t top = (uint32_t)(key >> 29);
        const uint32_t *d = dk + (uint64_t)t * n;
        const uint64_t *ks = key_s + (uint64_t)t * n;
        const uint32_t *ls = len_s + (uint64_t)t * n;
        uint64_t c = 0;
        uint32_t lo = probe_lower(d, n, top);
        if (lo < n && d[lo] == top) {
            // the end of the entries with the query's top bits
            uint32_t g1 = lo + 1, hi = n, step = 2;
            while (hi - g1 > step) {
                if (d[g1 + step] > top) {
                    hi = g1 + step;
                    break;
                }
                g1 += step + 1;
                step *= 4;
            }
            while (g1 < hi) {
                const uint32_t mid = g1 + (hi - g1) / 2;
                if (d[mid] <= top) g1 = mid + 1; else hi = mid;
            }
            const uint32_t lq = qlen[q], kq = Kq[q];
            const uint32_t lmin = lq > kq ? lq - kq : 0u;
            const uint64_t lmax = (uint64_t)lq + kq;
            hi = g1;
            while (lo < hi) {  // first entry of the group with length >= lmin
                const uint32_t mid = (lo + hi) >> 1;
                if (ls[mid] < lmin) lo = mid + 1; else hi = mid;
            }
            for (uint32_t x = lo; x < g1 && (uint64_t)ls[x] <= lmax; x++)
                c += ks[x] == key ? 1u : 0u;
        }
        counts[e] = c;
        first[e] = lo;
    }
}

// The counted candidates' codes (q << B | id), from offs[e] on.
template <typename C>
__global__ void k_query_emit(const uint64_t *__restrict__ qkeys, uint32_t nq,
                             const uint64_t *__restrict__ key_s, const uint32_t *__restrict__ ids,
                             uint32_t n, uint32_t T, uint32_t B, const uint64_t *__restrict__ offs,
                             const uint32_t *__restrict__ first, uint64_t raw,
                             C *__restrict__ out) {
    const uint64_t tot = (uint64_t)T * nq;
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < tot;
         e += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t o = offs[e];
        const uint64_t end = e + 1 < tot ? offs[e + 1] : raw;
        if (o == end) continue;
        const uint32_t t = (uint32_t)(e / nq), q = (uint32_t)(e % nq);
        const uint64_t key = qkeys[(uint64_t)t * nq + q];
        for (uint64_t x = (uint64_t)t * n + first[e]; o < end; x++)
            if (key_s[x] == key) out[o++] = ((C)q << B) | (C)ids[x];
    }
}

// Incremental insert (Algorithm 3 inserts strings one by one in length
// order; here a batch at once).  Per table, the index's entries and the new
// ones are each sorted by (top key bits, length, position), and every new
// position is above every old one, so the merged order puts an old entry
// before a new one with equal (top bits, length).  Each entry's merged
// position is its own rank plus the number of the other list's entries that
// go before it (binary search); old and new entries are scattered there.
__device__ inline bool before_or_tie(uint32_t d0, uint32_t l0, uint32_t d1, uint32_t l1) {
    return d0 < d1 || (d0 == d1 && l0 <= l1);
}

__global__ void k_merge_tables(const uint32_t *__restrict__ dkA, const uint64_t *__restrict__ keyA,
                               const uint32_t *__restrict__ lenA, const uint32_t *__restrict__ idA,
                               uint32_t nA, const uint32_t *__restrict__ dkB,
                               const uint64_t *__restrict__ keyB, const uint32_t *__restrict__ lenB,
                               const uint32_t *__restrict__ idB, uint32_t nB, uint32_t T,
                               uint32_t *__restrict__ dk, uint64_t *__restrict__ key,
                               uint32_t *__restrict__ len, uint32_t *__restrict__ id) {
    const uint64_t nN = (uint64_t)nA + nB;
    const uint64_t tot = (uint64_t)T * nN;
    for (uint64_t g = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; g < tot;
         g += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t t = (uint32_t)(g / nN);
        const uint32_t x = (uint32_t)(g - (uint64_t)t * nN);
        const uint64_t a0 = (uint64_t)t * nA, b0 = (uint64_t)t * nB;
        uint32_t rank, d, l;
        uint64_t k;
        uint32_t i;
        if (x < nA) {  // old entry: new entries strictly before it
            d = dkA[a0 + x];
            l = lenA[a0 + x];
            uint32_t lo = 0, hi = nB;
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                const uint32_t dm = dkB[b0 + mid], lm = lenB[b0 + mid];
                if (dm < d || (dm == d && lm < l)) lo = mid + 1; else hi = mid;
            }
            rank = x + lo;
            k = keyA[a0 + x];
            i = idA[a0 + x];
        } else {  // new entry: old entries before it or tied with it
            const uint32_t y = x - nA;
            d = dkB[b0 + y];
            l = lenB[b0 + y];
            uint32_t lo = 0, hi = nA;
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (before_or_tie(dkA[a0 + mid], lenA[a0 + mid], d, l)) lo = mid + 1; else hi = mid;
            }
            rank = y + lo;
            k = keyB[b0 + y];
            i = idB[b0 + y];
        }
        const uint64_t o = (uint64_t)t * nN + rank;
        dk[o] = d;
        key[o] = k;
        len[o] = l;
        id[o] = i;
    }
}

// New entries' positions after the index's n0 strings.
__global__ void k_add_u32(uint32_t *__restrict__ a, uint64_t cnt, uint32_t add) {
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < cnt;
         e += (uint64_t)gridDim.x * blockDim.x)
        a[e] += add;
}

// Offsets of the inserted strings, relative to the new strings' first
// character, placed after the index's characters.
__global__ void k_append_offsets(const uint64_t *__restrict__ off, uint32_t n, uint64_t base,
                                 uint64_t shift, uint64_t *__restrict__ out) {
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e <= n;
         e += (uint64_t)gridDim.x * blockDim.x)
        out[e] = off[e] - base + shift;
}

template <typename C>
__global__ void k_uniq_flags(const C *__restrict__ codes, uint64_t cnt,
                             uint32_t *__restrict__ flags) {
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < cnt;
         e += (uint64_t)gridDim.x * blockDim.x)
        flags[e] = (e == 0 || codes[e] != codes[e - 1]) ? 1u : 0u;
}

// Unique (q << B | id) codes -> verification pairs (id << 32 | q) and the
// threshold of each pair.
template <typename C>
__global__ void k_to_pairs(const C *__restrict__ codes, uint64_t cnt, uint32_t B,
                           const uint32_t *__restrict__ flags, const uint32_t *__restrict__ pos,
                           const uint32_t *__restrict__ Kq, uint64_t *__restrict__ pairs,
                           uint32_t *__restrict__ pk) {
    const uint64_t mask = (1ULL << B) - 1ULL;
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < cnt;
         e += (uint64_t)gridDim.x * blockDim.x) {
        if (flags[e]) {
            uint64_t c = codes[e];
            uint32_t q = (uint32_t)(c >> B), id = (uint32_t)(c & mask);
            pairs[pos[e]] = ((uint64_t)id << 32) | q;
            pk[pos[e]] = Kq[q];
        }
    }
}

__global__ void k_q_out_flags(const int32_t *__restrict__ dist, const uint32_t *__restrict__ pk,
                              uint64_t cnt, uint32_t *__restrict__ flags) {
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < cnt;
         e += (uint64_t)gridDim.x * blockDim.x)
        flags[e] = (dist[e] >= 0 && (uint32_t)dist[e] <= pk[e]) ? 1u : 0u;
}

__global__ void k_q_out_compact(const uint64_t *__restrict__ pairs, const int32_t *__restrict__ dist,
                                uint64_t cnt, const uint32_t *__restrict__ flags,
                                const uint32_t *__restrict__ pos, uint32_t *__restrict__ ids,
                                int32_t *__restrict__ od, uint32_t *__restrict__ per_q) {
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < cnt;
         e += (uint64_t)gridDim.x * blockDim.x) {
        if (flags[e]) {
            uint64_t c = pairs[e];
            ids[pos[e]] = (uint32_t)(c >> 32);
            od[pos[e]] = dist[e];
            atomicAdd(&per_q[(uint32_t)c], 1u);
        }
    }
}

// Device bytes of a batch before its candidates are known (the admission
// estimate of ej_query_workspace_estimate).
uint64_t estimate(const ej_index *ix, uint64_t qbytes, uint32_t nq) {
    const uint64_t T = ix->T;
    uint64_t b = 0;
    b += 2 * qbytes + 64 * 1024;                 // chars, codes, packed
    b += (uint64_t)nq * (8 + 4 * 6);             // offsets, lengths, order, thresholds
    b += T * nq * (8 + 8 + 8);                   // keys, counts, scan
    b += T * nq * 4 * 8;                         // expected candidates (a few per table)
    return b;
}

// Bytes of the candidate stage once the raw (pre-de-duplication) count is
// known: raw codes, their sorted copy and the radix sort's scratch, unique
// flags and positions, then the pairs and thresholds.
uint64_t probe_bytes(uint64_t raw) { return raw * (8 + 8 + 8 + 4 + 4 + 8 + 4); }

// Bytes of verification and output once the de-duplicated count is known:
// distances, the queries' match masks (their bit planes are at most half of
// that), the state kept per pair (the larger of the two forms that keep any:
// the two-pass form's Pv and Mv of NL band words, rounded up to whole lanes of
// up to 4 words, with its ordering buffers, and the strips'), output flags and
// positions, result ids and distances.
uint64_t verify_bytes(const ej_ctx *ctx, uint64_t cnt, uint64_t qbytes, uint32_t nq,
                      uint32_t sigma, uint32_t Kmax) {
    const uint64_t NL = verify_lanes_for(Kmax);
    uint64_t b = cnt * 4;                                           // distances
    b += mask_words_bound(qbytes, nq, sigma) * 4 + 24ull * (nq + 1);  // query masks
    if (ctx->tune.verify_mode == 0)
        b += std::max(cnt * (8 * (NL + 3) + 4 * 8 + 8), strip_bytes(cnt, Kmax));
    b += cnt * (4 + 4 + 4 + 4);                                     // output
    return b;
}

// The match masks of n indexed strings, in one piece: the words, then the
// offsets.  Only the verification forms other than the strips read them, so
// they are built when a batch first runs such a form, after its admission has
// counted them.
uint64_t mask_offsets_at(uint64_t total, uint64_t n, uint32_t sigma) {
    return (4 * mask_words_bound(total, (uint32_t)n, sigma) + 255) & ~255ull;
}
uint64_t mask_bytes(uint64_t total, uint64_t n, uint32_t sigma) {
    return mask_offsets_at(total, n, sigma) + 8 * (n + 1);
}

void index_masks(ej_index *ix) {
    ej_ctx *ctx = ix->ctx;
    char *p = own_copy<char>(ix, nullptr, mask_bytes(ix->total, ix->n, ix->sigma));
    RowMasks rm;
    try {
        build_masks(ctx, ix->d_codes, ix->d_offsets, 0, ix->n, ix->total, ix->sigma, rm, "ixm",
                    (uint32_t *)p, (uint64_t *)(p + mask_offsets_at(ix->total, ix->n, ix->sigma)));
    } catch (...) {
        // nothing of a failed build stays with the index
        (void)hipStreamSynchronize(ctx->stream);
        ix->owned.pop_back();
        (void)hipFree(p);
        throw;
    }
    ix->masks = rm;
}

}  // namespace

extern "C" {

ej_status ej_index_build(ej_ctx *ctx, const uint8_t *strings, const uint64_t *offsets, uint32_t n,
                         const ej_params *p, int on_device, ej_index **out) {
    if (!ctx || !p || !out || !offsets) return EJ_EINVAL;
    *out = nullptr;
    ej_index *ix = new (std::nothrow) ej_index();
    if (!ix) return EJ_ENOMEM;
    ix->ctx = ctx;
    ix->alive = ctx->alive;
    ix->device = ctx->device;
    ej_status st = run_guarded(ctx, [&] {
        if (p->r == 0 || p->z == 0 || p->m == 0 || p->m > 64 || (uint64_t)p->r * p->z > 4096)
            fail(EJ_EINVAL, "invalid r, z, m");
        if (n >= 0x80000000u) fail(EJ_EINVAL, "n must be below 2^31");
        ix->p = *p;
        ix->n = n;
        ix->T = p->r * p->z;
        const uint8_t *d_chars = strings;
        const uint64_t *d_off = offsets;
        if (!on_device) {
            std::vector<uint64_t> reb(offsets, offsets + n + 1);
            for (uint32_t i = 0; i < n; i++)
                if (offsets[i + 1] < offsets[i]) fail(EJ_EINVAL, "offsets are not non-decreasing");
            uint64_t base = offsets[0], total = offsets[n] - base;
            for (auto &o : reb) o -= base;
            uint8_t *dc = ws<uint8_t>(ctx, "ix_hchars", total + 16);
            uint64_t *dofs = ws<uint64_t>(ctx, "ix_hoff", (uint64_t)n + 1);
            if (total) EJ_HIP(hipMemcpyAsync(dc, strings + base, total, hipMemcpyHostToDevice, ctx->stream));
            EJ_HIP(hipMemcpyAsync(dofs, reb.data(), 8ull * (n + 1), hipMemcpyHostToDevice, ctx->stream));
            sync(ctx);
            d_chars = dc;
            d_off = dofs;
        }
        Prep pp;
        prepare(ctx, d_chars, d_off, n, p->L, pp, "ix");
        ix->sigma = pp.sigma;
        ix->L = pp.L;
        ix->maxlen = pp.maxlen;
        ix->minlen = pp.minlen;
        ix->total = pp.total;
        memcpy(ix->lut, pp.lut, 256);
        Rand rd;
        draw_randomness(ctx, *p, pp.L, pp.sigma, rd, "ix");
        const uint64_t tot = (uint64_t)ix->T * n;
        uint64_t *keys = ws<uint64_t>(ctx, "ix_keys", tot);
        uint32_t *bdk = bucket_input(ctx, tot, "ix");
        embed_keys(ctx, pp, rd, keys, nullptr, bdk, 61u - 32u);
        Buckets bk;
        bucket(ctx, keys, pp.d_len, pp.d_perm, n, ix->T, 32, bk, "ix", false, true, false);
        // owned copies
        const SlabParts parts = slab_parts(ctx, n, pp.total, tot, pp.sigma, &ix->slab,
                                           &ix->slab_bytes);
        ix->d_codes = parts.codes;
        copy_on(ctx, ix->d_codes, (const uint8_t *)pp.d_codes, pp.total + 64);
        // offsets rebased onto the owned code array
        ix->d_offsets = parts.offsets;
        copy_on(ctx, ix->d_offsets, d_off, (uint64_t)n + 1);
        ix->rd = rd;
        ix->rd.d_Rwords = own_copy(ix, rd.d_Rwords, (size_t)rd.r * rd.nw);
        ix->rd.d_Rstep = own_copy(ix, rd.d_Rstep, (size_t)rd.r * rd.Lpad);
        ix->rd.d_pos = own_copy(ix, rd.d_pos, (size_t)ix->T * rd.m);
        ix->rd.d_v = own_copy(ix, rd.d_v, (size_t)ix->T * rd.m);
        ix->rd.d_spos = own_copy(ix, rd.d_spos, (size_t)ix->T * rd.m);
        ix->rd.d_sslot = own_copy(ix, rd.d_sslot, (size_t)ix->T * rd.m);
        ix->rd.d_J = own_copy(ix, rd.d_J, (size_t)rd.r);
        ix->d_ids = parts.ids;
        ix->d_dk = parts.dk;
        ix->d_key_s = parts.key_s;
        ix->d_len_s = parts.len_s;
        if (tot)
            hipLaunchKernelGGL(k_sorted_attrs_full, dim3(grid_for(ctx, tot, 256)), dim3(256), 0,
                               ctx->stream, (const uint64_t *)keys, (const uint32_t *)bk.d_ids,
                               (const uint32_t *)pp.d_perm, (const uint32_t *)pp.d_perm_len, n,
                               tot, ix->d_ids, ix->d_dk, ix->d_key_s, ix->d_len_s);
        EJ_CHECK_LAUNCH();
        // what verification needs of the index strings, kept for every query
        // batch: the bit planes (the match masks of the other forms, twice
        // their size for 4 letters and five times for 25, follow when a batch
        // first asks for such a form)
        ix->d_planes = parts.planes;
        build_planes(ctx, pp.d_codes, pp.total, pp.sigma, ix->d_planes);
        // the owned offsets must be relative to the owned codes: base 0
        if (pp.base) {
            std::vector<uint64_t> h(n + 1);
            EJ_HIP(hipMemcpyAsync(h.data(), ix->d_offsets, 8ull * (n + 1), hipMemcpyDeviceToHost,
                                  ctx->stream));
            sync(ctx);
            for (auto &o : h) o -= pp.base;
            EJ_HIP(hipMemcpyAsync(ix->d_offsets, h.data(), 8ull * (n + 1), hipMemcpyHostToDevice,
                                  ctx->stream));
        }
        sync(ctx);
    });
    if (st != EJ_OK) {
        ej_index_free(ix);
        return st;
    }
    *out = ix;
    return EJ_OK;
}

ej_status ej_index_insert(ej_index *ix, const uint8_t *strings, const uint64_t *offsets,
                          uint32_t n_new, int on_device) {
    if (!ix || !offsets) return EJ_EINVAL;
    ej_ctx *ctx = ix->ctx;
    std::vector<void *> fresh;  // allocations of this call, released on failure
    void *slab = nullptr;
    size_t slab_bytes = 0;
    ej_status st = run_guarded(ctx, [&] {
        if (n_new == 0) return;
        if ((uint64_t)ix->n + n_new >= 0x80000000ull) fail(EJ_EINVAL, "n must stay below 2^31");
        const uint64_t nN = (uint64_t)ix->n + n_new;
        if (nN * ix->T >= 0xFFFFFFFFull) fail(EJ_EUNSUPPORTED, "r*z*n must stay below 2^32");
        const uint8_t *d_chars = strings;
        const uint64_t *d_off = offsets;
        if (!on_device) {
            std::vector<uint64_t> reb(offsets, offsets + n_new + 1);
            for (uint32_t i = 0; i < n_new; i++)
                if (offsets[i + 1] < offsets[i]) fail(EJ_EINVAL, "offsets are not non-decreasing");
            const uint64_t base = offsets[0], total = offsets[n_new] - base;
            if (total && !strings) fail(EJ_EINVAL, "null strings");
            for (auto &o : reb) o -= base;
            uint8_t *dc = ws<uint8_t>(ctx, "ii_hchars", total + 16);
            uint64_t *dofs = ws<uint64_t>(ctx, "ii_hoff", (uint64_t)n_new + 1);
            if (total)
                EJ_HIP(hipMemcpyAsync(dc, strings + base, total, hipMemcpyHostToDevice,
                                      ctx->stream));
            EJ_HIP(hipMemcpyAsync(dofs, reb.data(), 8ull * (n_new + 1), hipMemcpyHostToDevice,
                                  ctx->stream));
            sync(ctx);
            d_chars = dc;
            d_off = dofs;
        }
        // the new strings under the index's alphabet, truncation and streams
        Prep pq;
        prepare(ctx, d_chars, d_off, n_new, 0, pq, "ii", ix->lut, ix->sigma, ix->L);
        const uint32_t T = ix->T;
        const uint64_t totB = (uint64_t)T * n_new;
        uint64_t *keys = ws<uint64_t>(ctx, "ii_keys", totB);
        uint32_t *bdk = bucket_input(ctx, totB, "ii");
        embed_keys(ctx, pq, ix->rd, keys, nullptr, bdk, 61u - 32u);
        Buckets bk;
        bucket(ctx, keys, pq.d_len, pq.d_perm, n_new, T, 32, bk, "ii", false, true, false);
        uint32_t *dkB = ws<uint32_t>(ctx, "ii_dkB", totB);
        uint64_t *keyB = ws<uint64_t>(ctx, "ii_keyB", totB);
        uint32_t *lenB = ws<uint32_t>(ctx, "ii_lenB", totB);
        hipLaunchKernelGGL(k_sorted_attrs_full, dim3(grid_for(ctx, totB, 256)), dim3(256), 0,
                           ctx->stream, (const uint64_t *)keys, (const uint32_t *)bk.d_ids,
                           (const uint32_t *)pq.d_perm, (const uint32_t *)pq.d_perm_len, n_new,
                           totB, bk.d_ids, dkB, keyB, lenB);
        EJ_CHECK_LAUNCH();
        hipLaunchKernelGGL(k_add_u32, dim3(grid_for(ctx, totB, 256)), dim3(256), 0, ctx->stream,
                           bk.d_ids, totB, ix->n);
        EJ_CHECK_LAUNCH();
        // the grown index, built beside the current one (which stays whole
        // until every allocation has succeeded)
        auto alloc = [&](size_t bytes) -> void * {
            void *p = nullptr;
            hipError_t e = hipMalloc(&p, std::max<size_t>(bytes, 16));
            if (e == hipErrorOutOfMemory && spare_release(ctx))
                e = hipMalloc(&p, std::max<size_t>(bytes, 16));
            if (e != hipSuccess) {
                (void)hipGetLastError();
                fail(EJ_ENOMEM, "index insert: device allocation failed");
            }
            fresh.push_back(p);
            return p;
        };
        const uint64_t totN = (uint64_t)T * nN;
        const uint64_t charsN = ix->total + pq.total;
        const SlabParts parts = slab_parts(ctx, nN, charsN, totN, ix->sigma, &slab, &slab_bytes);
        uint32_t *dk = parts.dk, *len = parts.len_s, *id = parts.ids, *planes = parts.planes;
        uint64_t *key = parts.key_s, *offs = parts.offsets;
        uint8_t *codes = parts.codes;
        const bool masked = ix->masks.words != nullptr;  // a batch has asked for them
        char *mp = masked ? (char *)alloc(mask_bytes(charsN, nN, ix->sigma)) : nullptr;
        hipLaunchKernelGGL(k_merge_tables, dim3(grid_for(ctx, totN, 256)), dim3(256), 0,
                           ctx->stream, (const uint32_t *)ix->d_dk, (const uint64_t *)ix->d_key_s,
                           (const uint32_t *)ix->d_len_s, (const uint32_t *)ix->d_ids, ix->n,
                           (const uint32_t *)dkB, (const uint64_t *)keyB, (const uint32_t *)lenB,
                           (const uint32_t *)bk.d_ids, n_new, T, dk, key, len, id);
        EJ_CHECK_LAUNCH();
        // codes and offsets: the new strings after the indexed ones (the new
        // codes carry their zero padding along)
        if (ix->total)
            EJ_HIP(hipMemcpyAsync(codes, ix->d_codes, ix->total, hipMemcpyDeviceToDevice,
                                  ctx->stream));
        EJ_HIP(hipMemcpyAsync(codes + ix->total, pq.d_codes, pq.total + 64,
                              hipMemcpyDeviceToDevice, ctx->stream));
        EJ_HIP(hipMemcpyAsync(offs, ix->d_offsets, 8ull * ix->n, hipMemcpyDeviceToDevice,
                              ctx->stream));
        hipLaunchKernelGGL(k_append_offsets, dim3(grid_for(ctx, (uint64_t)n_new + 1, 256)),
                           dim3(256), 0, ctx->stream, d_off, n_new, pq.base, ix->total,
                           offs + ix->n);
        EJ_CHECK_LAUNCH();
        RowMasks masks;
        if (masked)
            build_masks(ctx, codes, offs, 0, (uint32_t)nN, charsN, ix->sigma, masks, "ixm",
                        (uint32_t *)mp, (uint64_t *)(mp + mask_offsets_at(charsN, nN, ix->sigma)));
        build_planes(ctx, codes, charsN, ix->sigma, planes);
        sync(ctx);
        // swap in the grown arrays; release the replaced ones
        if (masked) {
            void *old = (void *)ix->masks.words;
            ix->owned.erase(std::find(ix->owned.begin(), ix->owned.end(), old));
            (void)hipFree(old);
        }
        ix->owned.insert(ix->owned.end(), fresh.begin(), fresh.end());
        fresh.clear();
        std::swap(ix->slab, slab);
        std::swap(ix->slab_bytes, slab_bytes);
        ix->d_dk = dk;
        ix->d_key_s = key;
        ix->d_len_s = len;
        ix->d_ids = id;
        ix->d_codes = codes;
        ix->d_offsets = offs;
        ix->masks = masks;
        ix->d_planes = planes;
        ix->n = (uint32_t)nN;
        ix->total = charsN;
        ix->maxlen = std::max(ix->maxlen, pq.maxlen);
        ix->minlen = std::min(ix->minlen, pq.minlen);
    });
    if (slab && st != EJ_OK) (void)hipStreamSynchronize(ctx->stream);
    slab_give(ctx, slab, slab_bytes);  // the replaced one, or this call's on failure
    for (void *p : fresh) (void)hipFree(p);
    return st;
}

uint64_t ej_query_workspace_estimate(const ej_index *ix, const uint64_t *q_offsets, uint32_t nq,
                                     const uint32_t *Kq) {
    (void)Kq;
    if (!ix || !q_offsets) return 0;
    return estimate(ix, q_offsets[nq] - q_offsets[0], nq);
}

void ej_index_set_hbm_limit(ej_index *ix, uint64_t bytes) {
    if (ix) ix->hbm_limit = bytes;
}

uint32_t ej_index_size(const ej_index *ix) { return ix ? ix->n : 0; }

ej_status ej_query_batch(ej_index *ix, const uint8_t *q, const uint64_t *q_offsets, uint32_t nq,
                         const uint32_t *Kq, ej_qresult *out) {
    if (!ix || !q_offsets || !out || (nq && !Kq)) return EJ_EINVAL;
    ej_ctx *ctx = ix->ctx;
    memset(out, 0, sizeof(*out));
    ej_status st = run_guarded(ctx, [&] {
        for (uint32_t i = 0; i < nq; i++) {
            if (q_offsets[i + 1] < q_offsets[i]) fail(EJ_EINVAL, "query offsets decrease");
            if (verify_lanes_for(Kq[i]) == 0) fail(EJ_EUNSUPPORTED, "query threshold above 2046");
        }
        const uint64_t qbase = q_offsets[0], qtotal = q_offsets[nq] - qbase;
        if (qtotal && !q) fail(EJ_EINVAL, "null query strings");
        // admission by free HBM (or the configured limit)
        size_t freeb = 0, totalb = 0;
        EJ_HIP(hipMemGetInfo(&freeb, &totalb));
        uint64_t avail = ix->hbm_limit ? ix->hbm_limit : (uint64_t)freeb;
        uint32_t Kmax = 0;
        for (uint32_t i = 0; i < nq; i++) Kmax = std::max(Kmax, Kq[i]);
        // admission, checked again as each data-dependent size becomes known
        // and before any of that stage's memory is requested
        uint64_t need = estimate(ix, qtotal, nq);
        auto admit = [&](const char *what) {
            if (need > avail && !ix->hbm_limit && spare_release(ctx)) {
                EJ_HIP(hipMemGetInfo(&freeb, &totalb));
                avail = freeb;
            }
            if (need > avail)
                fail(EJ_ENOMEM, std::string("batch needs ~") + std::to_string(need) +
                                    " bytes (" + what + "), " + std::to_string(avail) +
                                    " admitted");
        };
        admit("before embedding");
        EJ_HIP(hipEventRecord(ctx->timers.ev[0], ctx->stream));
        out->nq = nq;
        out->offsets = (uint64_t *)calloc((size_t)nq + 1, sizeof(uint64_t));
        if (!out->offsets) fail(EJ_ENOMEM, "host allocation failed");
        if (nq == 0) return;
        // upload
        std::vector<uint64_t> reb(q_offsets, q_offsets + nq + 1);
        for (auto &o : reb) o -= qbase;
        uint8_t *dq = ws<uint8_t>(ctx, "q_chars", qtotal + 16);
        uint64_t *dqo = ws<uint64_t>(ctx, "q_off", (uint64_t)nq + 1);
        uint32_t *dK = ws<uint32_t>(ctx, "q_K", nq);
        if (qtotal) EJ_HIP(hipMemcpyAsync(dq, q + qbase, qtotal, hipMemcpyHostToDevice, ctx->stream));
        EJ_HIP(hipMemcpyAsync(dqo, reb.data(), 8ull * (nq + 1), hipMemcpyHostToDevice, ctx->stream));
        EJ_HIP(hipMemcpyAsync(dK, Kq, 4ull * nq, hipMemcpyHostToDevice, ctx->stream));
        // A0-A2 on the queries with the index's alphabet, truncation and randomness
        Prep pq;
        prepare(ctx, dq, dqo, nq, 0, pq, "q", ix->lut, ix->sigma, ix->L);
        const uint32_t T = ix->T;
        uint64_t *qkeys = ws<uint64_t>(ctx, "q_keys", (uint64_t)T * nq);
        embed_keys(ctx, pq, ix->rd, qkeys, nullptr);
        // probe
        const uint64_t tot = (uint64_t)T * nq;
        uint64_t *counts = ws<uint64_t>(ctx, "q_counts", tot);
        uint64_t *d_raw = ws<uint64_t>(ctx, "q_raw", 1);
        uint32_t *first = ws<uint32_t>(ctx, "q_first", tot);
        // codes: the query above B bits of the index position
        const uint32_t B = std::max(1u, bits_for(ix->n ? ix->n - 1 : 0));
        const uint32_t code_bits = B + std::max(1u, bits_for(nq - 1));
        hipLaunchKernelGGL(k_query_count, dim3(grid_for(ctx, tot, 256)), dim3(256), 0, ctx->stream,
                           (const uint64_t *)qkeys, (const uint32_t *)pq.d_len,
                           (const uint32_t *)dK, nq, (const uint32_t *)ix->d_dk,
                           (const uint64_t *)ix->d_key_s, (const uint32_t *)ix->d_len_s, ix->n, T,
                           counts, first);
        EJ_CHECK_LAUNCH();
        scan_exclusive_u64(ctx, counts, counts, tot, d_raw);
        // the shortest text of a pair, over the queries that can have one (while
        // the device counts)
        uint32_t mintext = ix->maxlen;
        for (uint32_t i = 0; i < nq; i++) {
            const uint64_t lq = q_offsets[i + 1] - q_offsets[i];
            const uint64_t least = std::max<uint64_t>(ix->minlen, lq > Kq[i] ? lq - Kq[i] : 0);
            if (least <= ix->maxlen && lq + Kq[i] >= ix->minlen)
                mintext = (uint32_t)std::min<uint64_t>(mintext, std::min(lq, least));
        }
        uint64_t raw = 0;
        read_back(ctx, d_raw, 8, &raw);
        need += probe_bytes(raw);
        admit("with the candidate stage");
        uint64_t cnt = 0;
        uint64_t *pairs = nullptr;
        uint32_t *pk = nullptr;
        if (raw) {
            if (raw >= 0xFFFFFFFFull) fail(EJ_EUNSUPPORTED, "more than 2^32 raw query candidates");
            uint32_t *flags = ws<uint32_t>(ctx, "q_uflags", raw);
            uint32_t *pos = ws<uint32_t>(ctx, "q_upos", raw);
            uint64_t *d_cnt = ws<uint64_t>(ctx, "q_ucnt", 1);
            auto unique_pairs = [&](auto *rb, auto *sorted) {
                using C = std::remove_pointer_t<decltype(rb)>;
                hipLaunchKernelGGL(k_query_emit<C>, dim3(grid_for(ctx, tot, 256)), dim3(256), 0,
                                   ctx->stream, (const uint64_t *)qkeys, nq,
                                   (const uint64_t *)ix->d_key_s, (const uint32_t *)ix->d_ids,
                                   ix->n, T, B, (const uint64_t *)counts,
                                   (const uint32_t *)first, raw, rb);
                EJ_CHECK_LAUNCH();
                if constexpr (sizeof(C) == 4)
                    radix_sort_u32(ctx, rb, nullptr, sorted, nullptr, 1, (uint32_t)raw, code_bits,
                                   ctx->tune.radix_bits);
                else
                    radix_sort_u64(ctx, rb, sorted, raw, code_bits, ctx->tune.radix_bits);
                hipLaunchKernelGGL(k_uniq_flags<C>, dim3(grid_for(ctx, raw, 256)), dim3(256), 0,
                                   ctx->stream, (const C *)sorted, raw, flags);
                EJ_CHECK_LAUNCH();
                scan_exclusive_u32(ctx, flags, pos, raw, d_cnt);
                read_back(ctx, d_cnt, 8, &cnt);
                pairs = ws<uint64_t>(ctx, "q_pairs", cnt);
                pk = ws<uint32_t>(ctx, "q_pk", cnt);
                hipLaunchKernelGGL(k_to_pairs<C>, dim3(grid_for(ctx, raw, 256)), dim3(256), 0,
                                   ctx->stream, (const C *)sorted, raw, B,
                                   (const uint32_t *)flags, (const uint32_t *)pos,
                                   (const uint32_t *)dK, pairs, pk);
                EJ_CHECK_LAUNCH();
            };
            // (32-bit codes up to 65,536 queries on 65,536 strings, and the like)
            uint64_t *rb = ws<uint64_t>(ctx, "q_rawbuf", raw);
            uint64_t *sorted = ws<uint64_t>(ctx, "q_sorted", raw);
            if (code_bits <= 32)
                unique_pairs((uint32_t *)rb, (uint32_t *)sorted);
            else
                unique_pairs(rb, sorted);
        }
        out->n_candidates = cnt;
        const bool new_masks = cnt && !strip_form(ctx) && !ix->masks.words;
        need += verify_bytes(ctx, cnt, qtotal, nq, ix->sigma, Kmax);
        if (new_masks) need += mask_bytes(ix->total, ix->n, ix->sigma);
        admit("with verification");
        out->workspace_bytes = need;
        uint64_t nout = 0;
        uint32_t *per_q = ws<uint32_t>(ctx, "q_perq", nq);
        EJ_HIP(hipMemsetAsync(per_q, 0, 4ull * nq, ctx->stream));
        uint32_t *oids = nullptr;
        int32_t *odist = nullptr;
        if (cnt) {
            int32_t *dist = ws<int32_t>(ctx, "q_dist", cnt);
            VerifySet sx;
            sx.codes = ix->d_codes;
            sx.off = ix->d_offsets;
            sx.n = ix->n;
            sx.total = ix->total;
            sx.maxlen = ix->maxlen;
            sx.tag = "ixm";
            if (new_masks) index_masks(ix);
            sx.masks = ix->masks;
            sx.planes = ix->d_planes;
            const VerifySet sq = verify_set(pq, dqo, "qm");
            verify(ctx, ix->sigma, sx, &sq, pairs, cnt, 0, pk, dist, nullptr, nullptr, nullptr,
                   mintext, Kmax);
            uint32_t *flags = ws<uint32_t>(ctx, "q_oflags", cnt);
            uint32_t *pos = ws<uint32_t>(ctx, "q_opos", cnt);
            uint64_t *d_no = ws<uint64_t>(ctx, "q_nout", 1);
            hipLaunchKernelGGL(k_q_out_flags, dim3(grid_for(ctx, cnt, 256)), dim3(256), 0,
                               ctx->stream, (const int32_t *)dist, (const uint32_t *)pk, cnt, flags);
            EJ_CHECK_LAUNCH();
            scan_exclusive_u32(ctx, flags, pos, cnt, d_no);
            read_back(ctx, d_no, 8, &nout);
            oids = ws<uint32_t>(ctx, "q_oids", nout);
            odist = ws<int32_t>(ctx, "q_odist", nout);
            hipLaunchKernelGGL(k_q_out_compact, dim3(grid_for(ctx, cnt, 256)), dim3(256), 0,
                               ctx->stream, (const uint64_t *)pairs, (const int32_t *)dist, cnt,
                               (const uint32_t *)flags, (const uint32_t *)pos, oids, odist, per_q);
            EJ_CHECK_LAUNCH();
        }
        out->ids = (uint32_t *)malloc(4 * (nout ? nout : 1));
        out->dist = (int32_t *)malloc(4 * (nout ? nout : 1));
        std::vector<uint32_t> hq(nq);
        if (!out->ids || !out->dist) fail(EJ_ENOMEM, "host allocation failed");
        if (nout) {
            EJ_HIP(hipMemcpyAsync(out->ids, oids, 4 * nout, hipMemcpyDeviceToHost, ctx->stream));
            EJ_HIP(hipMemcpyAsync(out->dist, odist, 4 * nout, hipMemcpyDeviceToHost, ctx->stream));
        }
        EJ_HIP(hipMemcpyAsync(hq.data(), per_q, 4ull * nq, hipMemcpyDeviceToHost, ctx->stream));
        EJ_HIP(hipEventRecord(ctx->timers.ev[1], ctx->stream));
        sync(ctx);
        for (uint32_t i = 0; i < nq; i++) out->offsets[i + 1] = out->offsets[i] + hq[i];
        float ms = 0.f;
        EJ_HIP(hipEventElapsedTime(&ms, ctx->timers.ev[0], ctx->timers.ev[1]));
        out->ms_total = ms;
    });
    if (st != EJ_OK) ej_qresult_free(out);
    return st;
}

void ej_qresult_free(ej_qresult *res) {
    if (!res) return;
    free(res->offsets);
    free(res->ids);
    free(res->dist);
    memset(res, 0, sizeof(*res));
}

void ej_index_free(ej_index *ix) {
    if (!ix) return;
    (void)hipSetDevice(ix->device);
    if (*ix->alive) {
        (void)hipStreamSynchronize(ix->ctx->stream);
        slab_give(ix->ctx, ix->slab, ix->slab_bytes);
    } else if (ix->slab) {
        // (the context waited for its stream when it was destroyed)
        (void)hipFree(ix->slab);
    }
    for (void *p : ix->owned) (void)hipFree(p);
    delete ix;
}

}  // extern "C"
