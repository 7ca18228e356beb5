// Stage A5, strip form: threshold edit distance of many pairs, one pair per
// lane, the whole band in the lane's registers, on a band that narrows.
//
// The recurrence is the one of ej_verify.hip (Myers' bit vectors over the
// K + 1 diagonals lo..hi that a path of cost <= K can touch, bit k of the
// state on diagonal k + lo).  Three things differ:
//
//  * The match word of a column is computed from bit planes of the symbol
//    codes instead of being looked up: plane p holds bit p of every code, 32
//    letters to a word, over the concatenated text without regard to string
//    boundaries.  A lane keeps the planes of the rows its band covers in
//    registers and compares them with the column's symbol.  Neither LDS nor a
//    mask array per string and symbol is needed, and there is no lookahead
//    between lanes: 12 instructions per 32 cells and column for alphabets of
//    up to 4 letters, against 17 in the form that spreads a band over lanes.
//    Rows outside the pattern hold some other letter's code.  Above the
//    pattern that changes nothing: there every vertical delta is -1 (Mv set,
//    Pv clear), which fixes the step's outcome whatever the match bit is.
//    Below it, nothing flows back up.
//  * The columns are taken in strips.  A strip's kernel runs every pair that
//    is still undecided for the strip's columns and then drops the words of
//    its band that can no longer matter.  Call a cell good if its value plus
//    its distance from the diagonal d* of the final cell is at most K.  Every
//    cell of a path of cost <= K is good; good cells are computed exactly as
//    long as no good cell was dropped (all cells of their best paths are good
//    too); along a column the sum does not decrease away from d*, nor does it
//    along a diagonal.  So a word beyond the first one without a good cell is
//    dropped for good.  One word past the last good cell is kept at the lower
//    end, whose match bit the step cannot see.
//  * The survivors are grouped by the number of words they keep, and the next
//    strip's waves each take 64 pairs of one width.
//
// A pair is decided as in ej_verify.hip: at the first multiple of 32 columns
// where the value on d* exceeds K, or at its last column.  That value is
// exact whenever it is at most K, so neither the decision nor the column
// where it falls depends on the strips.
#include <algorithm>
#include <string>

#include "ej_bits.h"
#include "ej_internal.h"

namespace ej {

namespace {

// One string set: bit planes (P words per 32 letters, `words` such groups),
// character offsets, the first string's offset.
struct PlaneSet {
    const uint32_t *planes;
    const uint64_t *off;
    uint64_t base;
    uint32_t words;
};

// Band widths the pairs are grouped by: exact up to 8 words, in steps of 2 up
// to 16 and of 8 up to 64.
constexpr uint32_t CLASSES = 18;
constexpr uint32_t CTR = 32;  // counters per strip: [class] pairs of it

__host__ __device__ inline uint32_t width_class(uint32_t words) {
    return words <= 8 ? words : words <= 16 ? 4 + (words + 1) / 2 : 10 + (words + 7) / 8;
}
__host__ __device__ inline uint32_t class_words(uint32_t c) {
    return c <= 8 ? c : c <= 12 ? 2 * (c - 4) : 8 * (c - 10);
}
// The k-th pair of class c in the lists: two classes share an array of `cap`
// entries (a strip's pairs are at most that), one from each end.
__device__ inline uint64_t list_at(uint32_t c, uint64_t k, uint64_t cap) {
    const uint64_t a = (uint64_t)((c - 1) / 2) * cap;
    return (c & 1u) ? a + k : a + cap - 1 - k;
}

// Lanes per pair of a strip with n pairs on a chip that wants `fill` lanes:
// one while the pairs alone fill it, else 2, 4, 8 or 16.
__device__ inline uint32_t strip_lanes(uint32_t n, uint32_t fill) {
    uint32_t k = 1;
    while (k < 16 && (uint64_t)n * k < fill) k *= 2;
    return k;
}

__device__ inline uint32_t clamp_word(int32_t q, uint32_t words) {
    return (uint32_t)min(max(q, 0), (int32_t)words - 1);
}

template <int P>
__device__ inline void load_planes(const uint32_t *planes, uint32_t words, int32_t q,
                                   uint32_t (&out)[P]) {
    const uint32_t *src = planes + (size_t)clamp_word(q, words) * P;
#pragma unroll
    for (int p = 0; p < P; p++) out[p] = src[p];
}

// a += (bit `lane` of c); c = the carry-outs.
__device__ inline void add_mask(uint32_t &a, uint64_t &c) {
    asm("v_addc_co_u32 %0, %1, %0, 0, %1" : "+v"(a), "+s"(c));
}
// The value of the next lane (0 in the last).
__device__ inline uint32_t from_next_lane(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x130, 0xf, 0xf, true);  // wave_shl:1
}

// (a ^ b) | c and a | ~(b | c) in one instruction each.
__device__ inline uint32_t xor_or(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xBE);
}
__device__ inline uint32_t or_nor(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xF1);
}

// Match words w0 .. w0 + N - 1 of column s, from the match bits of the window
// words (cur = those of word w0, which becomes word w0 + N's).
template <int W, int P, int N>
__device__ __forceinline__ void match_bits(int w0, const uint32_t (&Y)[P],
                                           const uint32_t (&X)[P][W + 1], uint32_t (&t)[N]) {
#pragma unroll
    for (int i = 0; i < N; i++)
        if (w0 + i <= W) t[i] = X[0][w0 + i] ^ Y[0];
#pragma unroll
    for (int p = 1; p < P; p++)
#pragma unroll
        for (int i = 0; i < N; i++)
            if (w0 + i <= W) t[i] &= X[p][w0 + i] ^ Y[p];
}

// One column: ty = the inverted text planes of the block, column s of it.
// keep is ~0 in the lanes of a tile that have a next one, 0 in its last;
// more = the mask of those lanes.
//
// A VALU result takes about 10 cycles to reach the next instruction of its
// wave, and one word's step is a chain of 9 instructions, so the words are
// taken in groups of G and each stage is issued for a whole group before the
// next one; the scheduling barriers keep the compiler from going back to one
// word after the other.
template <int W, int P, bool SPLIT, bool AHEAD>
__device__ __forceinline__ void strip_column(uint32_t s, const uint32_t (&ty)[P],
                                             const uint32_t (&X)[P][W + 1], uint32_t (&Pv)[W],
                                             uint32_t (&Mv)[W], uint32_t &Z, uint32_t keep,
                                             uint64_t more) {
    constexpr int G = W < 4 ? W : 4;
    constexpr bool CARRY = W > 1 || SPLIT;
    uint32_t Y[P];  // the symbol's bits, inverted: 0 or all ones
#pragma unroll
    for (int p = 0; p < P; p++) Y[p] = (uint32_t)__builtin_amdgcn_sbfe((int)ty[p], s, 1u);
    uint32_t bits[G + 1], eq[G];
    match_bits<W, P, G + 1>(0, Y, X, bits);
#pragma unroll
    for (int i = 0; i < G; i++) eq[i] = __builtin_amdgcn_alignbit(bits[i + 1], bits[i], s);
    uint32_t Xv[W], sum[W];
    uint64_t cy = 0;
    uint32_t D0[W + 1];
    auto finish = [&](int w) {  // the new state of word w, from D0[w] and D0[w + 1]
        const uint32_t HP = or_nor(Mv[w], D0[w], Pv[w]);
        const uint32_t HN = D0[w] & Pv[w];
        const uint32_t Ds = __builtin_amdgcn_alignbit(D0[w + 1], D0[w], 1);
        if (w == 0) Z += Ds & 1u;
        Pv[w] = or_nor(HN, Ds, HP);
        Mv[w] = HP & Ds;
    };
#pragma unroll
    for (int g = 0; g < W; g += G) {
        const int n = W - g < G ? W - g : G;
        __builtin_amdgcn_sched_barrier(0);
        uint32_t a[G];
#pragma unroll
        for (int i = 0; i < n; i++) {
            Xv[g + i] = eq[i] | Mv[g + i];
            a[i] = eq[i] & Pv[g + i];
        }
        __builtin_amdgcn_sched_barrier(0);
        // the group's carry chain, and meanwhile the next group's match bits
        uint32_t nb[G + 1];
        nb[0] = bits[G];
#pragma unroll
        for (int i = 0; i < n; i++) {
            if (!CARRY)
                sum[g + i] = a[i] + Pv[g + i];
            else if (g + i == 0)
                sum[g + i] = add_carry_mask(a[i], Pv[g + i], cy);
            else
                sum[g + i] = add_carry_chain(a[i], Pv[g + i], cy, cy);
        }
#pragma unroll
        for (int i = 1; i <= G; i++)
            if (g + G + i <= W) nb[i] = X[0][g + G + i] ^ Y[0];
#pragma unroll
        for (int p = 1; p < P; p++)
#pragma unroll
            for (int i = 1; i <= G; i++)
                if (g + G + i <= W) nb[i] &= X[p][g + G + i] ^ Y[p];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < G; i++)
            if (g + G + i < W) eq[i] = __builtin_amdgcn_alignbit(nb[i + 1], nb[i], s);
#pragma unroll
        for (int i = 0; i <= G; i++)
            if (g + G + i <= W) bits[i] = nb[i];
        if (!SPLIT) {
#pragma unroll
            for (int i = 0; i < n; i++) D0[g + i] = xor_or(sum[g + i], Pv[g + i], Xv[g + i]);
            __builtin_amdgcn_sched_barrier(0);
            // the words whose next one is known
#pragma unroll
            for (int i = -1; i < n - 1; i++)
                if (g + i >= 0) finish(g + i);
        }
    }
    if (SPLIT) {
        if (AHEAD) {
            // Large alphabets, and wide bands over many lanes: a lane's words
            // are often all ones (32 rows without a match, or rows outside
            // both strings), so the carries look ahead across the lanes: out =
            // carries out, pass = passes a carry on.
            uint32_t all = sum[0];
#pragma unroll
            for (int w = 1; w < W; w++) all &= sum[w];
            const uint64_t out = cy & more;
            const uint64_t pass = __builtin_amdgcn_ballot_w64(all == 0xFFFFFFFFu) & more;
            uint64_t c = ((out | pass) + out) ^ pass;
#pragma unroll
            for (int w = 0; w < W; w++) add_mask(sum[w], c);
        } else {
            // Up to 4 letters a lane whose first word is all ones, and so
            // carries again, is rare enough for a branch (1 word in 10,000).
            uint64_t c = (cy & more) << 1;
            add_mask(sum[0], c);
            while (__builtin_expect(c != 0, 0)) {
#pragma unroll
                for (int w = 1; w < W; w++) add_mask(sum[w], c);
                c = (c & more) << 1;
                add_mask(sum[0], c);
            }
        }
#pragma unroll
        for (int w = 0; w < W; w++) D0[w] = xor_or(sum[w], Pv[w], Xv[w]);
        D0[W] = from_next_lane(D0[0]) & keep;
#pragma unroll
        for (int w = 0; w < W; w++) finish(w);
    } else {
        D0[W] = 0u;
        finish(W - 1);
    }
    // the state is materialised every column: left free, the compiler
    // re-associates the bit operations across columns and computes the match
    // words of several columns ahead, which costs more registers than it has
#pragma unroll
    for (int w = 0; w < W; w++) asm volatile("" : "+v"(Pv[w]), "+v"(Mv[w]));
    __builtin_amdgcn_sched_barrier(0);
}

// The strip's columns [jbeg, jlim), W band words per lane and KL lanes per
// pair.  Returns, in the pair's first lane, the words the
// pair keeps, or 0 when it is decided.
template <int W, int P, bool SPLIT, bool AHEAD>
__device__ __forceinline__ uint32_t strip_run(
    const PlaneSet &A, const PlaneSet &B, const uint64_t *__restrict__ pairs,
    const uint32_t *__restrict__ Kq, uint32_t K, uint32_t pidx, bool act, uint32_t KL,
    uint32_t jbeg, uint32_t jlim, uint32_t *__restrict__ state, uint32_t SW,
    uint2 *__restrict__ meta, int32_t *__restrict__ dist, unsigned long long &colsum) {
    const uint32_t lane = threadIdx.x;
    const uint32_t l = SPLIT ? lane & (KL - 1) : 0u;
    const uint32_t NW = SPLIT ? W * KL : W;
    const int32_t bit0 = SPLIT ? 32 * W * (int32_t)l : 0;  // the lane's first band bit
    const uint32_t keep = SPLIT && l == KL - 1 ? 0u : 0xFFFFFFFFu;
    const uint64_t more = __builtin_amdgcn_ballot_w64(keep != 0u);
    const uint32_t *px = A.planes, *py = A.planes;
    uint32_t wx = A.words, wy = A.words;
    uint64_t ox = 0, oy = 0;  // first letters, from the set's first one
    uint32_t m = 0, nn = 0, Kp = K;
    if (act) {
        const uint64_t code = pairs[pidx];
        const uint32_t a = (uint32_t)(code >> 32), b = (uint32_t)code;
        const uint64_t oa = A.off[a], ob = B.off[b];
        const uint32_t la = (uint32_t)(A.off[a + 1] - oa), lb = (uint32_t)(B.off[b + 1] - ob);
        if (Kq) Kp = Kq[pidx];
        // the longer string is the pattern (the first one of equal ones)
        const bool first = la >= lb;
        m = first ? la : lb;
        nn = first ? lb : la;
        ox = first ? oa - A.base : ob - B.base;
        oy = first ? ob - B.base : oa - A.base;
        px = first ? A.planes : B.planes;
        py = first ? B.planes : A.planes;
        wx = first ? A.words : B.words;
        wy = first ? B.words : A.words;
    }
    const uint32_t gap = m - nn;
    bool has = act;
    if (act && jbeg == 0 && (gap > Kp || nn == 0)) {
        // decided without a column: length gap above K, or ED = |x|
        if (l == 0) dist[pidx] = (int32_t)min(gap, Kp + 1);
        has = false;
    }
    if (!has) m = nn = 0;
    const uint32_t dstar = has ? gap : 0u;
    // row 0 is at band bit O, d* at bit ks; both move down as low words go
    int32_t O = (int32_t)(has ? (Kp - dstar) / 2 : 0u);
    int32_t ks = O + (int32_t)dstar;
    uint32_t V = (uint32_t)O;  // value on the diagonal of bit 0 (first lane)
    uint32_t woff = 0;
    uint32_t Pv[W], Mv[W];
    if (jbeg == 0) {
        // D[i][0] = |i|: bit k holds row k - O, rows <= 0 have delta -1
#pragma unroll
        for (int w = 0; w < W; w++) {
            const int d = O - bit0 - 32 * w;
            const uint32_t mv = d >= 31 ? 0xFFFFFFFFu : (d < 0 ? 0u : (2u << d) - 1u);
            Mv[w] = mv;
            Pv[w] = ~mv;
        }
    } else {
        const uint2 mt = has ? meta[pidx] : make_uint2(0u, 0u);
        V = mt.x;
        woff = mt.y >> 8;
        const uint32_t nw = mt.y & 0xFFu;  // words kept; above them D grows by 1 per row
        O -= 32 * (int32_t)woff;
        ks -= 32 * (int32_t)woff;
        const uint2 *st = (const uint2 *)(state + (uint64_t)pidx * SW) + l * W;
#pragma unroll
        for (int w = 0; w < W; w++) {
            const uint2 x = l * W + w < nw ? st[w] : make_uint2(~0u, 0u);
            Pv[w] = x.x;
            Mv[w] = x.y;
        }
    }
    // pattern window: word w's bits are pattern letters jb + bit0 + 32 w - O
    // - 1 .. (0-based) of the string, at bit ox + that of the planes
    const int64_t fx = (int64_t)ox + jbeg + bit0 - O - 1;
    const int64_t fy = (int64_t)oy + jbeg;
    int32_t qx = (int32_t)(fx >> 5), qy = (int32_t)(fy >> 5);
    const uint32_t shx = (uint32_t)fx & 31u, shy = (uint32_t)fy & 31u;
    uint32_t X[P][W + 1], rx[P], ry[P];
    load_planes<P>(px, wx, qx, rx);
#pragma unroll
    for (int w = 0; w <= W; w++) {
        uint32_t t[P];
        load_planes<P>(px, wx, qx + w + 1, t);
#pragma unroll
        for (int p = 0; p < P; p++) {
            X[p][w] = __builtin_amdgcn_alignbit(t[p], rx[p], shx);
            rx[p] = t[p];
        }
        if (w % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // few loads' addresses at a time
    }
    uint32_t ny[P];
    load_planes<P>(py, wy, qy, ry);
    load_planes<P>(py, wy, qy + 1, ny);
    qx += W + 2;  // the words fetched during a block
    qy += 2;

    for (uint32_t jb = jbeg; jb < jlim; jb += 32) {
        if (__builtin_amdgcn_ballot_w64(has) == 0) break;
        uint32_t ty[P], tx[P];
#pragma unroll
        for (int p = 0; p < P; p++) {
            ty[p] = ~__builtin_amdgcn_alignbit(ny[p], ry[p], shy);
            ry[p] = ny[p];
        }
        load_planes<P>(px, wx, qx, tx);
        load_planes<P>(py, wy, qy, ny);
        qx++;
        qy++;
        const uint32_t nc = has ? min(nn - jb, 32u) : 32u;
        uint32_t Z = 0;  // columns in which bit 0's diagonal kept its value
        if (__builtin_amdgcn_ballot_w64(nc < 32u) == 0) {
#pragma unroll 2
            for (uint32_t s = 0; s < 32; s++)
                strip_column<W, P, SPLIT, AHEAD>(s, ty, X, Pv, Mv, Z, keep, more);
        } else {
            // a text ends in this block: its lanes stop at its last column
#pragma unroll 1
            for (uint32_t s = 0; s < 32; s++)
                if (s < nc) strip_column<W, P, SPLIT, AHEAD>(s, ty, X, Pv, Mv, Z, keep, more);
        }
        V += nc - Z;
        // keeps the masks below inside the loop (hoisted, they take W registers)
        asm volatile("" : "+v"(ks));
        uint32_t up = 0, dn = 0;
#pragma unroll
        for (int w = 0; w < W; w++) {
            const int d = ks - bit0 - 32 * w;
            uint32_t mk = d >= 31 ? 0xFFFFFFFFu : (d < 0 ? 0u : (2u << d) - 1u);
            if (w == 0 && (!SPLIT || l == 0)) mk &= ~1u;
            up = popc_acc(Pv[w] & mk, up);
            dn = popc_acc(Mv[w] & mk, dn);
        }
        uint32_t Vd = (SPLIT && l != 0 ? 0u : V) + up - dn;
        if (SPLIT)
            for (uint32_t o = 1; o < KL; o <<= 1) Vd += (uint32_t)__shfl_xor((int)Vd, (int)o, 64);
        if (has && (Vd > Kp || jb + 32 >= nn)) {
            if (l == 0) {
                dist[pidx] = (int32_t)min(Vd, Kp + 1);
                colsum += (unsigned long long)min(jb + 32, nn);
            }
            has = false;
        }
#pragma unroll
        for (int p = 0; p < P; p++) {
#pragma unroll
            for (int w = 0; w < W; w++) X[p][w] = X[p][w + 1];
            X[p][W] = __builtin_amdgcn_alignbit(tx[p], rx[p], shx);
            rx[p] = tx[p];
        }
    }
    if (__builtin_amdgcn_ballot_w64(has) == 0) return 0u;

    // the words [w0, w1] still worth keeping.  acc = the value at bit 32 w +
    // 31 of the band: the bit of word w nearest to d* when d* is above the
    // word, and the last one before word w + 1 when it is below.  The words
    // without a good cell are a prefix of those below d*'s and a suffix of
    // those above it, so counting them is enough.
    int32_t acc = 0;
    if (SPLIT) {
        // values at the lanes' first bits
#pragma unroll
        for (int w = 0; w < W; w++) {
            const uint32_t mk = w == 0 && l == 0 ? ~1u : ~0u;
            acc += (int32_t)__builtin_popcount(Pv[w] & mk) -
                   (int32_t)__builtin_popcount(Mv[w] & mk);
        }
        if (l == 0) acc += (int32_t)V;
        const int32_t own = acc;
        for (uint32_t o = 1; o < KL; o <<= 1) {
            const int32_t y = __shfl_up(acc, o, 64);
            if (l >= o) acc += y;
        }
        acc -= own;
        if (l == 0) acc = (int32_t)V;
    } else {
        acc = (int32_t)V;
    }
    const int32_t before = acc;  // at the bit below the lane's first (lane 0: at bit 0)
    uint32_t low = 0, below = 0, high = 0;
#pragma unroll
    for (int w = 0; w < W; w++) {
        const uint32_t mk = w == 0 && (!SPLIT || l == 0) ? ~1u : ~0u;
        acc += (int32_t)__builtin_popcount(Pv[w] & mk) - (int32_t)__builtin_popcount(Mv[w] & mk);
        const int32_t bit = bit0 + 32 * w + 31;
        const bool good = acc + (bit < ks ? ks - bit : bit - ks) <= (int32_t)Kp;
        if (bit < ks) {
            below++;
            low += good ? 0u : 1u;
        } else {
            high += good ? 1u : 0u;
        }
    }
    if (SPLIT)
        for (uint32_t o = 1; o < KL; o <<= 1) {
            low += (uint32_t)__shfl_xor((int)low, (int)o, 64);
            below += (uint32_t)__shfl_xor((int)below, (int)o, 64);
            high += (uint32_t)__shfl_xor((int)high, (int)o, 64);
        }
    if (!has) return 0u;
    // A pair's row holds SW / 2 words, those of the largest threshold; the class
    // it runs in may be wider.  No word past them is kept: the value on a
    // diagonal is at least its distance from the corner's, so beyond bit Kp the
    // sum above exceeds Kp.  The bound keeps the row's end in any case.
    const uint32_t w0 = low, w1 = min(min(below + high, NW - 1), w0 + SW / 2 - 1);
    const uint32_t left = w1 - w0 + 1;
    // the lane of word w0 knows the value on the new bit 0's diagonal
    int32_t v0 = before;
#pragma unroll
    for (int w = 0; w < W; w++) {
        const uint32_t gw = l * W + w;
        uint32_t mk = gw < w0 ? ~0u : gw == w0 ? 1u : 0u;
        if (gw == 0) mk &= ~1u;
        v0 += (int32_t)__builtin_popcount(Pv[w] & mk) - (int32_t)__builtin_popcount(Mv[w] & mk);
    }
    if (l == w0 / W) meta[pidx] = make_uint2((uint32_t)v0, ((woff + w0) << 8) | left);
    uint2 *st = (uint2 *)(state + (uint64_t)pidx * SW) + (int32_t)(l * W) - (int32_t)w0;
#pragma unroll
    for (int w = 0; w < W; w++)
        if (l * W + w >= w0 && l * W + w <= w1) st[w] = make_uint2(Pv[w], Mv[w]);
    return l == 0 ? left : 0u;
}

// Appends the lanes' pairs (width 0: none) to the lists of their widths'
// classes, one atomic per wave and class.
__device__ inline void strip_append(uint32_t width, uint32_t pidx, uint32_t *__restrict__ ctr,
                                    uint32_t *__restrict__ lists, uint64_t cap) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t cls = width_class(width);
    uint64_t left = __builtin_amdgcn_ballot_w64(width != 0);
    while (left) {
        const uint32_t c = readlane_u32(cls, (uint32_t)__builtin_ctzll(left));
        const uint64_t same = __builtin_amdgcn_ballot_w64(width != 0 && cls == c);
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&ctr[c], (uint32_t)__popcll(same));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        if (width != 0 && cls == c)
            lists[list_at(c, at + (uint64_t)__popcll(same & ((1ull << lane) - 1ull)), cap)] = pidx;
        left &= ~same;
    }
}

// Waves per SIMD asked of a kernel with up to `w` band words per lane: what its
// column loop leaves room for.  Outside that loop the instances of 2 planes
// spill (9 to 83 registers up to 8 words, 175 with 16), once a pair and strip.
constexpr int strip_waves(int w, int P) {
    return P == 2 ? (w <= 4 ? 7 : w <= 8 ? 5 : 4)
         : P == 5 ? (w <= 4 ? 4 : w <= 8 ? 3 : 2)
                  : (w <= 4 ? 3 : w <= 8 ? 2 : 1);
}

// Bound by VALU instructions (4.0 to 4.7 cycles each per SIMD at four waves:
// carries, funnel shifts and three-input operations run at half rate).
// 220,300 pairs of 5,000 letters, K = 500: 3.7 ms in five strips, against 4.2
// ms for the two-pass form (masks from LDS, a band over several lanes); 26.9 M
// pairs of 25 letters, 50 to 4,000 of them, K = 100, nearly all in one lane: 5.6
// ms with their order, against 20.4, where that form refilled its mask rows every
// block of columns.  Where that form is the faster one: two_pass_pays.
//
// One strip over the pairs in the classes' lists (null: all pairs are of one
// class, the k-th is order[k], or k), the widest class first, 64 / lanes pairs
// per wave.
// SPLIT = false takes the strip's classes of up to 16 words when the strip has
// pairs enough for one lane each; SPLIT = true takes the others, the band in
// strip_lanes() lanes or as many as MAXW words per lane need.
template <int MAXW, int P, bool SPLIT>
__global__ void __launch_bounds__(64, strip_waves(MAXW, P))
    k_strip(PlaneSet A, PlaneSet B, const uint64_t *__restrict__ pairs,
            const uint32_t *__restrict__ lists, const uint32_t *__restrict__ order, uint64_t cap,
            const uint32_t *__restrict__ ctr, uint32_t fill, const uint32_t *__restrict__ Kq,
            uint32_t K, uint32_t jbeg, uint32_t jlim, uint32_t *__restrict__ state, uint32_t SW,
            uint2 *__restrict__ meta, uint32_t *__restrict__ ctr_next,
            uint32_t *__restrict__ lists_next, int32_t *__restrict__ dist,
            unsigned long long *__restrict__ columns) {
    unsigned long long colsum = 0;
    const uint32_t lane = threadIdx.x;
    // lane c holds class c's count: one load, then reads across lanes
    const uint32_t counts = lane < CTR ? ctr[lane] : 0u;
    uint32_t n = counts;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o, 64);
    n = (uint32_t)__builtin_amdgcn_readfirstlane((int)n);
    const uint32_t lanes = strip_lanes(n, fill);
    for (uint64_t g = blockIdx.x;; g += gridDim.x) {
        // the class of group g and its first group
        uint64_t g0 = 0;
        uint32_t c = SPLIT ? CLASSES : width_class(MAXW), cnt = 0, KL = 1;
        for (; c > 0; c--) {
            if (class_words(c) <= 16 && (lanes != 1) != SPLIT) {
                c = 0;
                break;
            }
            cnt = readlane_u32(counts, c);
            if (cnt == 0) continue;
            if (SPLIT) {
                const uint32_t words = class_words(c);
                // Up to 2 words stay in one lane however few the pairs are: a
                // column's chain through two words takes 71 ns, across two
                // lanes (carry mask, next lane's bit) 80, and 30,000 pairs 90
                // against 107.  With 3 words it is 92 to 81, so they spread.
                KL = words <= 2 ? 1 : lanes;
                while (KL > 1 && KL / 2 >= words) KL /= 2;  // no lane without a word
                while (KL * MAXW < words) KL *= 2;
                // More than 32 words go over up to 64 lanes while the strip has
                // less than a wave per SIMD: 400 pairs of 5,000 letters, K =
                // 2046: 0.89 -> 0.51 ms with 4 letters, 1.06 -> 0.63 with 8 (the
                // two-pass form, a word in each of 64 lanes: 0.67 and 0.69).
                if (words > 32 && lanes == 16)
                    while (KL < 64 && (uint64_t)cnt * KL * 4 <= fill) KL *= 2;
            }
            const uint64_t ng = ((uint64_t)cnt * KL + 63) / 64;
            if (g < g0 + ng) break;
            g0 += ng;
        }
        if (c == 0) break;
        const uint64_t k = (g - g0) * (64 / KL) + (SPLIT ? lane / KL : lane);
        const bool act = k < cnt;
        uint32_t pidx = 0;
        if (act) pidx = lists ? lists[list_at(c, k, cap)] : order ? order[k] : (uint32_t)k;
        const uint32_t words = class_words(c);
        uint32_t width = 0;
#define EJ_STRIP_CASE(N)                                                                   \
    case N:                                                                                \
        if constexpr (N <= MAXW)                                                           \
            width = strip_run<N, P, SPLIT, (P > 2)>(A, B, pairs, Kq, K, pidx, act, KL,     \
                                                    jbeg, jlim, state, SW, meta, dist,     \
                                                    colsum);                               \
        break;
// Up to 4 letters, bands over 16 words in 16 lanes and more: the instance that
// looks ahead (400 pairs of 1,500 letters, K = 700: 298 -> 241 us; on 4 or 8
// lanes the branch is up to 10% faster).
#define EJ_STRIP_WIDE(N)                                                                   \
    case 32 + N:                                                                           \
        if constexpr (SPLIT && P == 2 && MAXW == 8)                                        \
            width = strip_run<N, P, SPLIT, true>(A, B, pairs, Kq, K, pidx, act, KL, jbeg,  \
                                                 jlim, state, SW, meta, dist, colsum);     \
        break;
#define EJ_STRIP_ONE(N)                                                                    \
    case 16 + N:                                                                           \
        if constexpr (SPLIT)                                                               \
            width = strip_run<N, P, false, false>(A, B, pairs, Kq, K, pidx, act, KL, jbeg, \
                                                  jlim, state, SW, meta, dist, colsum);    \
        break;
        const uint32_t form = !SPLIT ? 0 : KL == 1 ? 16 : P == 2 && words > 16 && KL >= 16 ? 32 : 0;
        switch ((words + KL - 1) / KL + form) {
            EJ_STRIP_ONE(1)
            EJ_STRIP_ONE(2)
            EJ_STRIP_WIDE(1)
            EJ_STRIP_WIDE(2)
            EJ_STRIP_WIDE(3)
            EJ_STRIP_WIDE(4)
            EJ_STRIP_WIDE(5)
            EJ_STRIP_WIDE(6)
            EJ_STRIP_WIDE(7)
            EJ_STRIP_WIDE(8)
            EJ_STRIP_CASE(1)
            EJ_STRIP_CASE(2)
            EJ_STRIP_CASE(3)
            EJ_STRIP_CASE(4)
            EJ_STRIP_CASE(5)
            EJ_STRIP_CASE(6)
            EJ_STRIP_CASE(7)
            EJ_STRIP_CASE(8)
            EJ_STRIP_CASE(9)
            EJ_STRIP_CASE(10)
            EJ_STRIP_CASE(11)
            EJ_STRIP_CASE(12)
            EJ_STRIP_CASE(13)
            EJ_STRIP_CASE(14)
            EJ_STRIP_CASE(15)
            EJ_STRIP_CASE(16)
        }
#undef EJ_STRIP_CASE
#undef EJ_STRIP_ONE
#undef EJ_STRIP_WIDE
        if (ctr_next) strip_append(width, pidx, ctr_next, lists_next, cap);
    }
    if (columns) {
        for (int o = 32; o > 0; o >>= 1) colsum += __shfl_xor(colsum, o, 64);
        if (lane == 0 && colsum) atomicAdd(columns, colsum);
    }
}

// Clears the strips' counters; with one threshold for all pairs the first
// strip's class is known (cls), and so its count: the pairs [first, first +
// count) of those that are there.
__global__ void k_strip_init(uint32_t *__restrict__ ctr, uint32_t n, uint32_t cls, uint64_t first,
                             uint64_t count, const uint64_t *__restrict__ count_dev) {
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
        uint32_t v = 0;
        if (cls && i == cls) {
            const uint64_t live = count_dev ? *count_dev : first + count;
            v = live > first ? (uint32_t)min(live - first, count) : 0u;
        }
        ctr[i] = v;
    }
}

// Sort keys of the pairs' order: the longest text first, in blocks of 32 << sh
// columns (at most 254 of them); pairs past a count on the device last.
__global__ void k_strip_order(const uint64_t *__restrict__ offA, const uint64_t *__restrict__ offB,
                              const uint64_t *__restrict__ pairs, uint64_t first, uint64_t count,
                              const uint64_t *__restrict__ count_dev, uint32_t sh,
                              uint32_t *__restrict__ key, uint32_t *__restrict__ val) {
    uint64_t live = count;
    if (count_dev) live = *count_dev > first ? min(*count_dev - first, count) : 0;
    for (uint64_t k = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; k < count;
         k += (uint64_t)gridDim.x * blockDim.x) {
        uint32_t kk = 255;
        if (k < live) {
            const uint64_t code = pairs[k];
            const uint32_t a = (uint32_t)(code >> 32), b = (uint32_t)code;
            const uint64_t la = offA[a + 1] - offA[a], lb = offB[b + 1] - offB[b];
            kk = 254 - (uint32_t)((((la < lb ? la : lb) + 31) >> 5) >> sh);
        }
        key[k] = kk;
        val[k] = (uint32_t)k;
    }
}

// Thresholds per pair: the class of each pair's own threshold.  A workgroup
// counts its 1,024 pairs in LDS and takes its places in the lists with one
// atomic per class (one per wave and class took 26 us for 50,000 pairs: the
// counters share two cache lines).
__global__ void __launch_bounds__(1024)
    k_strip_widths(const uint32_t *__restrict__ Kq, uint64_t first, uint64_t count,
                   const uint64_t *__restrict__ count_dev, const uint32_t *__restrict__ order,
                   uint32_t *__restrict__ ctr, uint32_t *__restrict__ lists, uint64_t cap) {
    __shared__ uint32_t cnt[CTR], at[CTR];
    uint64_t live = count;
    if (count_dev) live = *count_dev > first ? min(*count_dev - first, count) : 0;
    for (uint64_t b = (uint64_t)blockIdx.x * 1024; b < live; b += (uint64_t)gridDim.x * 1024) {
        if (threadIdx.x < CTR) cnt[threadIdx.x] = 0;
        __syncthreads();
        const uint64_t k = b + threadIdx.x;
        const uint32_t v = order && k < live ? order[k] : (uint32_t)k;
        const uint32_t c = k < live ? width_class((Kq[v] + 33u) / 32u) : 0u;
        const uint32_t rank = c ? atomicAdd(&cnt[c], 1u) : 0u;
        __syncthreads();
        if (threadIdx.x < CTR && cnt[threadIdx.x])
            at[threadIdx.x] = atomicAdd(&ctr[threadIdx.x], cnt[threadIdx.x]);
        __syncthreads();
        if (c) lists[list_at(c, (uint64_t)at[c] + rank, cap)] = v;
        __syncthreads();
    }
}

// Bit planes of a code array (padded with 64 zero bytes): thread g turns codes
// 32 g .. 32 g + 31 into P words.  Reads 32 B and writes 4 P B per 32 letters.
template <int P>
__global__ void __launch_bounds__(256)
    k_planes(const uint8_t *__restrict__ codes, uint64_t total, uint64_t words,
             uint32_t *__restrict__ planes) {
    for (uint64_t g = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; g < words;
         g += (uint64_t)gridDim.x * blockDim.x) {
        uint32_t out[P];
#pragma unroll
        for (int p = 0; p < P; p++) out[p] = 0;
        if (32 * g < total) {
            const uint4 *src = (const uint4 *)(codes + 32 * g);
            const uint4 u = src[0], v = src[1];
            const uint32_t d[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
            for (int q = 0; q < 8; q++)
#pragma unroll
                for (int p = 0; p < P; p++) {
                    // bits 0, 8, 16, 24 of the dword to bits 0 .. 3
                    const uint32_t x = (d[q] >> p) & 0x01010101u;
                    const uint32_t t = x | (x >> 7);
                    out[p] |= ((t | (t >> 14)) & 0xFu) << (4 * q);
                }
        }
#pragma unroll
        for (int p = 0; p < P; p++) planes[g * P + p] = out[p];
    }
}

uint32_t grid_for(ej_ctx *ctx, uint64_t work, uint32_t block) {
    uint64_t g = (work + block - 1) / block;
    uint64_t cap = (uint64_t)ctx->num_cu * 16;
    if (g > cap) g = cap;
    if (g == 0) g = 1;
    return (uint32_t)g;
}

using StripKernel = decltype(&k_strip<4, 2, false>);

template <int P>
StripKernel strip_kernel(uint32_t words, bool split) {
    if (split) return words <= 16 ? k_strip<4, P, true> : k_strip<8, P, true>;
    return words <= 4 ? k_strip<4, P, false> : words <= 8 ? k_strip<8, P, false>
                                                          : k_strip<16, P, false>;
}

}  // namespace

uint32_t plane_count(uint32_t sigma) { return sigma <= 4 ? 2u : sigma <= 32 ? 5u : 8u; }

void build_planes(ej_ctx *ctx, const uint8_t *d_codes, uint64_t total, uint32_t sigma,
                  uint32_t *d_planes) {
    const uint64_t words = plane_words(total);
    const uint32_t P = plane_count(sigma);
    auto launch = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid_for(ctx, words, 256)), dim3(256), 0, ctx->stream,
                           d_codes, total, words, d_planes);
        EJ_CHECK_LAUNCH();
    };
    if (P == 2)
        launch(k_planes<2>);
    else if (P == 5)
        launch(k_planes<5>);
    else
        launch(k_planes<8>);
}

// Pairs per batch: bounds the state and the lists.
static uint64_t strip_batch(uint64_t count, uint32_t NW) {
    return std::min<uint64_t>(count, NW <= 16 ? 1u << 24 : 1u << 23);
}

uint64_t strip_bytes(uint64_t count, uint32_t Kmax) {
    const uint32_t NW = (Kmax + 33u) / 32u, sets = (width_class(NW) + 1) / 2;
    return strip_batch(count, NW) * (8ull * NW + 8 + 2 * 4 * sets + 4);
}

void verify_strips(ej_ctx *ctx, uint32_t sigma, const StripSet &A, const StripSet &B,
                   const uint64_t *d_pairs, uint64_t count, uint32_t K, const uint32_t *d_Kq,
                   uint32_t Kmax, uint32_t mtext, bool uneven, int32_t *d_dist,
                   unsigned long long *d_columns, const uint64_t *d_count) {
    const uint32_t P = plane_count(sigma);
    const uint32_t NW = (Kmax + 33u) / 32u;
    const uint32_t ncls = width_class(NW);
    const PlaneSet SA{A.planes, A.off, A.base, (uint32_t)plane_words(A.total)};
    const PlaneSet SB{B.planes, B.off, B.base, (uint32_t)plane_words(B.total)};
    // The strips' ends.  The first is where unrelated strings are decided
    // (random texts of 4 letters differ in about half of the columns, of 20
    // and more in 4 of 5, and the value has to pass K), the others by halves: a
    // strip costs a launch and the state's way through memory (16 W bytes a
    // pair), steps of 512, 1024 and 2048 columns measured within 2%.
    std::vector<uint32_t> end;
    const uint64_t first = ((sigma <= 4 ? 2ull * Kmax : 5ull * Kmax / 4) + 95) & ~31ull;
    // Lanes that fill the chip: two waves per SIMD.  One wave alone issues every
    // 5 cycles, two together every 4: with 96 lanes per SIMD the strips
    // of the survivors ran at one wave each, 4.15 ms for the workload above
    // against 3.94; 256 lanes measured the same as 128.
    const uint32_t fill = (uint32_t)ctx->num_cu * 4 * 128;
    // Thresholds per pair: also at a half and a quarter of the first end, for
    // the pairs of smaller thresholds, down to 256 columns (49,000 pairs,
    // thresholds of 90 to 550: 1.27 -> 1.06 ms; of 10 to 180, strips of 96 and
    // 192 columns cost 40 us more than they saved).
    uint64_t e = first;
    for (int i = 0; i < 2 && d_Kq && e >= 512; i++) e = (e / 2 + 31) & ~31ull;
    for (;; e = e < first ? std::min(2 * e, first)
                          : e + std::max<uint64_t>(1024, (e / 2) & ~31ull)) {
        // (a band in 16 lanes gains nothing from being narrower)
        if (e >= mtext || count * 16 <= fill) {
            end.push_back(0xFFFFFFFFu);
            break;
        }
        end.push_back((uint32_t)e);
    }
    const uint32_t ns = (uint32_t)end.size();
    const uint32_t SW = 2 * NW;
    const uint64_t batch = strip_batch(count, NW);
    const bool listed = ns > 1 || d_Kq;
    uint32_t *ctr = ws<uint32_t>(ctx, "vs_ctr", (uint64_t)(ns + 1) * CTR);
    uint32_t *state = ns > 1 ? ws<uint32_t>(ctx, "vs_state", batch * SW) : nullptr;
    uint2 *meta = ns > 1 ? ws<uint2>(ctx, "vs_meta", batch) : nullptr;
    uint32_t *lists[2] = {nullptr, nullptr};
    const uint64_t entries = batch * ((ncls + 1) / 2);
    if (listed) lists[0] = ws<uint32_t>(ctx, "vs_lists0", entries);
    if (ns > 1) lists[1] = ws<uint32_t>(ctx, "vs_lists1", entries);
    // A wave runs a strip until its longest text ends, so pairs of texts of
    // unlike lengths go in length order (one pass of 8-bit digits; the strips
    // hand their survivors on in about the order they got them).  26.9 M pairs
    // of 50 to 4,000 letters, 10.8 -> 10.0 ms for the join; 60,000 pairs of 500
    // to 5,000, K = 60 to 500: 1.1 to 1.4 times as fast.  The sort is five
    // launches, 25 us, so not for little work: 30,011 pairs of 100 to 1,500
    // letters in 8 words took 312 us without and 336 with it.
    const bool by_len = uneven && count * 16 > fill && count * NW * mtext > 1ull << 29;
    uint32_t sh = 0;
    while (((mtext + 31) / 32 >> sh) > 254) sh++;
    uint32_t *okey = nullptr, *okey2 = nullptr, *oval = nullptr, *order = nullptr;
    if (by_len) {
        // the sort's scratch is the state, which the first strip writes after it
        uint32_t *tmp = ns > 1 ? state : ws<uint32_t>(ctx, "vs_state", 2 * batch);
        okey = tmp;
        oval = tmp + batch;
        okey2 = (uint32_t *)(ns > 1 ? meta : ws<uint2>(ctx, "vs_meta", batch));
        order = ws<uint32_t>(ctx, "vs_order", batch);
    }
    auto kernel = [&](bool split) {
        return P == 2 ? strip_kernel<2>(NW, split)
             : P == 5 ? strip_kernel<5>(NW, split) : strip_kernel<8>(NW, split);
    };
    uint32_t launches = 0;
    for (uint64_t b0 = 0; b0 < count; b0 += batch) {
        const uint64_t n = std::min(batch, count - b0);
        hipLaunchKernelGGL(k_strip_init, dim3(1), dim3(256), 0, ctx->stream, ctr, (ns + 1) * CTR,
                           d_Kq ? 0u : ncls, b0, n, d_count);
        EJ_CHECK_LAUNCH();
        const uint32_t *kq = d_Kq ? d_Kq + b0 : nullptr;
        if (by_len) {
            hipLaunchKernelGGL(k_strip_order, dim3(grid_for(ctx, n, 256)), dim3(256), 0,
                               ctx->stream, SA.off, SB.off, d_pairs + b0, b0, n, d_count, sh, okey,
                               oval);
            EJ_CHECK_LAUNCH();
            radix_sort_u32(ctx, okey, oval, okey2, order, 1, (uint32_t)n, 8, 8);
        }
        if (d_Kq) {
            hipLaunchKernelGGL(k_strip_widths, dim3(grid_for(ctx, n, 1024)), dim3(1024), 0,
                               ctx->stream, kq, b0, n, d_count, (const uint32_t *)order, ctr,
                               lists[0], batch);
            EJ_CHECK_LAUNCH();
        }
        uint32_t jbeg = 0;
        for (uint32_t i = 0; i < ns; i++) {
            uint32_t *c = ctr + (uint64_t)i * CTR;
            const bool known = i == 0 && !d_Kq && !d_count;  // the strip's pairs are n
            for (int split = 0; split < 2; split++) {
                if (!split && n < fill) continue;  // never enough pairs for a lane each
                if (known && split && n >= fill && NW <= 16) continue;
                uint64_t lanes = split ? n * 16 : n;
                if (split && NW > 32) lanes = std::max(lanes, std::min<uint64_t>(n * 64, fill));
                const uint64_t waves = (lanes + 63) / 64 + ncls;
                const uint32_t grid =
                    (uint32_t)std::min<uint64_t>(waves, (uint64_t)ctx->num_cu * 32);
                hipLaunchKernelGGL(kernel(split), dim3(grid), dim3(64), 0, ctx->stream, SA, SB,
                                   d_pairs + b0,
                                   (const uint32_t *)(i > 0 || d_Kq ? lists[i & 1] : nullptr),
                                   (const uint32_t *)order, batch, (const uint32_t *)c, fill, kq,
                                   K, jbeg, end[i], state, SW, meta,
                                   i + 1 < ns ? c + CTR : nullptr, lists[(i + 1) & 1],
                                   d_dist + b0, d_columns);
                EJ_CHECK_LAUNCH();
                launches++;
            }
            jbeg = end[i];
        }
    }
    if (ctx->timers.on) ctx->timers.more += launches - 1;
}

}  // namespace ej
